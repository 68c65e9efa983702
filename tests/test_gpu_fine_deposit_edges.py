"""GPU: tile densities, bit for bit, on states with runs of empty cells, cells
fuller than a workgroup's first pass, and counts that need 64-bit sums, for
both coarse ratios and for a mesh with a partial column."""

import numpy as np
import pytest
import torch

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

# particles per side, tiles, coarse ratio, buffer, split radius; tile boxes of 64, 48, 96 and 160 cells
BOXES = {"r4": (64, 4, 4, 16, 12), "r4_48": (64, 4, 4, 8, 5), "r8": (64, 2, 8, 16, 12), "r8_160": (128, 2, 8, 16, 12)}


def _state(box, dense, seed):
    """Most cells empty, the others of every size, one (in two corners) with `dense` particles."""
    from oracle.codec import State
    rng = np.random.default_rng(seed)
    n, cells = box.n_side ** 3, box.n_cells
    filled = rng.random(cells) < 0.3
    w = np.where(filled, rng.exponential(1.0, cells), 0.0)
    fixed = np.zeros(cells, dtype=np.int64)
    fixed[[0, cells - 1]] = dense
    w[[0, cells - 1]] = 0.0
    counts = fixed + np.floor(w / w.sum() * (n - fixed.sum())).astype(np.int64)
    left = n - int(counts.sum())
    counts[np.flatnonzero(filled)[1:1 + left]] += 1
    counts[np.flatnonzero(filled)[2]] += n - int(counts.sum())
    m = rng.integers(0, 256, size=(3, n), dtype=np.uint8)
    m[:, ::7] = rng.choice([0, 31, 32, 127, 128, 255], size=(3, m[:, ::7].shape[1])).astype(np.uint8)
    return State(box, counts, m, np.zeros((3, n), np.int8), 1.0, 0, np.arange(n, dtype=np.uint32))


@pytest.mark.parametrize("dense", [50, 3000, 20000])
@pytest.mark.parametrize("name", list(BOXES))
def test_tile_density_is_exact(name, dense):
    import oracle
    from oracle import cic, pm
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, nt, r, b, a = BOXES[name]
    spec = BoxSpec(name, n, nt, 2, r, b, a, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    ref = _state(box, dense, dense + n)
    Q, off = ref.quanta(), ref.offsets()
    with CubeBox(spec, with_ids=True) as g:
        g.set_state(ref.counts, ref.m, ref.u, ref.s, ref.M, ref.ids)
        for t in (0, box.n_tiles // 2, box.n_tiles - 1):
            idx, origin = pm.tile_sources(box, ref.counts, off, t)
            X = pm.tile_box_coords(box, Q[idx], origin)
            rho = cic.deposit(X, box.F, periodic=False) / box.h ** 3 - 1.0
            got = g.debug_mesh(2, t).cpu().numpy()
            assert np.array_equal(got, rho.transpose(2, 1, 0).astype(np.float32)), f"tile {t}"
