"""GPU: the coarse deposit against an exact integer deposit, on every shape of
its dispatch (cubes of 4, 8 and 16 cells, one lane or four per cell), with
cells around the 32 particles that fit one 32-bit sum, and empty ones."""

import numpy as np
import pytest
import torch

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

# particles per side, tiles, fine cells per spacing, coarse ratio, buffer
SHAPES = {
    "cubes4": (32, 1, 2, 4, 0), "cubes4_48": (96, 2, 2, 4, 16), "cubes4_full": (64, 1, 2, 8, 0),
    "cubes8": (128, 2, 2, 4, 16), "cubes8_80": (160, 2, 2, 4, 16), "cubes16": (256, 4, 2, 4, 16),
    "cubes16_quads": (512, 8, 2, 8, 16),
}


def _counts(n, cells, seed):
    """Poisson-like counts of n particles with runs of empty cells and cells of 31, 32, 33, 64, 65 and 300."""
    rng = np.random.default_rng(seed)
    mean = n // cells
    c = np.full(cells, mean, dtype=np.int64)
    moved = rng.integers(0, mean + 1, size=cells // 2)
    c[0::2] += moved
    c[1::2] -= moved
    for at, k in zip(rng.choice(cells // 2, size=6, replace=False) * 2, (31, 32, 33, 64, 65, 300)):
        c[at] = k
    c[-1] = 37
    c[0] = 33
    extra = int(c.sum()) - n
    for i in range(3, cells - 1):                    # settle the total on ordinary cells
        if extra == 0:
            break
        if c[i] in (31, 32, 33, 64, 65, 300):
            continue
        d = min(extra, int(c[i])) if extra > 0 else -min(-extra, 5)
        c[i] -= d
        extra -= d
    assert c.sum() == n and c.min() >= 0
    return c.astype(np.int32)


def _exact(box, counts, m):
    """Density - 1 in units of 2^-27 particles summed as integers, rounded once."""
    cells = counts.size
    canon = torch.repeat_interleave(torch.arange(cells, device="cuda"), torch.from_numpy(counts).cuda().long())
    tc, nt, nc = box.Tc, box.tiles_per_dim, box.n_coarse
    tile, local = canon // tc ** 3, canon % tc ** 3
    c = (tile % nt * tc + local % tc, tile // nt % nt * tc + local // tc % tc, tile // nt ** 2 * tc + local // tc ** 2)
    low, w = [], []
    for k in range(3):
        p = 2 * (256 * c[k] + torch.from_numpy(m[k]).cuda().long()) + 1 - 256      # in 1/512 of a cell
        low.append(p >> 9)
        w.append(p & 511)
    acc = torch.zeros(cells, dtype=torch.int64, device="cuda")
    for s in range(8):
        d = (s & 1, s >> 1 & 1, s >> 2)
        at = [(low[k] + d[k]) % nc for k in range(3)]
        ww = [w[k] if d[k] else 512 - w[k] for k in range(3)]
        acc.index_add_(0, (at[2] * nc + at[1]) * nc + at[0], ww[0] * ww[1] * ww[2])
    return (acc.double() * (2.0 ** -27 / box.H ** 3) - 1.0).float().view(nc, nc, nc)


@pytest.mark.parametrize("shape", list(SHAPES))
def test_coarse_density_equals_integer_deposit(shape):
    import oracle
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, nt, f, r, b = SHAPES[shape]
    spec = BoxSpec(shape, n, nt, f, r, b, 12, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec)
    rng = np.random.default_rng(n)
    counts = _counts(n ** 3, box.n_cells, n)
    m = rng.integers(0, 256, size=(3, n ** 3), dtype=np.uint8)
    m[:, :4] = [0, 127, 128, 255]                    # the bytes at which a slot changes
    with CubeBox(spec, tiles_per_batch=1) as gpu:
        gpu.set_state(counts, m, np.zeros((3, n ** 3), np.int8), 1.0, 0)
        got = gpu.debug_mesh(0)
    assert torch.equal(got, _exact(box, counts, m))
