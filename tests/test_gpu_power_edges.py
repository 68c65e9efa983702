"""GPU: the power spectrum's mesh at every ratio of diagnostic cells per coarse
cell, with 32- and 64-bit accumulators, and the moments of extreme codes."""

import numpy as np
import pytest
import torch

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

# particles per side, fine cells per spacing, coarse ratio (one periodic tile of 64 or 128 fine cells)
BOXES = {1: (32, 4, 4), 2: (32, 2, 4), 4: (64, 2, 8), 8: (128, 1, 8)}


def _state(box, dense, seed):
    from oracle.codec import State
    rng = np.random.default_rng(seed)
    n, cells = box.n_side ** 3, box.n_cells
    counts = np.full(cells, n // cells, dtype=np.int64)
    if dense:                                  # enough for 64-bit sums at 2 and 4 cells per coarse cell
        counts[5] += 3000
        counts[np.arange(cells - 3000, cells) if n // cells < 16 else np.arange(cells - 300, cells)] -= \
            1 if n // cells < 16 else 10
    m = rng.integers(0, 256, size=(3, n), dtype=np.uint8)
    u = rng.integers(-127, 128, size=(3, n)).astype(np.int8)
    u[:, :2] = [[-127, 127]] * 3
    return State(box, counts, m, u, 0.25, 127, np.arange(n, dtype=np.uint32))


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("ratio", list(BOXES))
def test_power_and_moments(ratio, dense):
    import oracle
    from oracle import diag
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, f, r = BOXES[ratio]
    spec = BoxSpec(f"diag{ratio}", n, 1, f, r, 0, 12, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    ref = _state(box, dense, n + dense)
    k_o, p_o, n_o = diag.power_spectrum(ref)
    mo = diag.moments(ref)
    with CubeBox(spec, with_ids=True) as g:
        g.set_state(ref.counts, ref.m, ref.u, ref.s, ref.M, ref.ids)
        k, p, modes = g.power_spectrum()
        d = g.diagnostics()
    assert np.array_equal(modes, n_o) and np.allclose(k, k_o, rtol=1e-12)
    # FP32 transform: about log2(n^3) roundings of 6e-8 of the rms amplitude,
    # shells within a factor ten of the mean power
    assert np.max(np.abs(p / p_o - 1.0)) <= 1e-5
    # sums of integers times powers of two are exact
    assert np.array_equal(d["momentum"], mo["momentum"]) and d["kinetic"] == mo["kinetic"] and d["mass"] == ref.n
