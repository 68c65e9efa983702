"""GPU: decoding where a workgroup's cells hold nothing, less than a round of
1024 particles, exactly one or several, and for each size of its groups of
cells (1 to 512 particles a cell on average)."""

import ctypes

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# side, tiles, fine cells per spacing, coarse ratio, buffer
BOXES = {"1": (48, 2, 4, 4, 16), "8": (64, 2, 2, 4, 16), "64": (64, 1, 2, 8, 0), "512": (128, 1, 1, 8, 0)}


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("mean", sorted(BOXES))
def test_groups_of_cells(mean, aligned):
    import oracle
    from oracle.codec import State
    from paper_2003_03931_amd import CubeBox
    from paper_2003_03931_amd._lib import check
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, tiles, f, r, b = BOXES[mean]
    spec = BoxSpec(mean, n, tiles, f, r, b, 12, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    rng = np.random.default_rng(int(mean))
    cells, left = box.n_cells, n ** 3
    counts = np.zeros(cells, np.int64)
    counts[:4] = [1024, 0, 1023, 1025]                    # rounds' edges, in groups of one cell too
    counts[cells // 2] = 4 * 1024 + 3
    counts[cells // 2 + 1] = left // 3                    # many rounds
    left -= int(counts.sum())
    counts[cells * 3 // 4:] += rng.multinomial(left, np.full(cells - cells * 3 // 4, 1.0 / (cells - cells * 3 // 4)))
    m = rng.integers(0, 256, size=(3, n ** 3), dtype=np.uint8)
    u = rng.integers(-127, 128, size=(3, n ** 3)).astype(np.int8)
    ref = State(box, counts, m, u, 0.5, 127, np.arange(n ** 3, dtype=np.uint32))
    with CubeBox(spec) as g:
        g.set_state(counts, m, u, 0.5, 127)
        out = [torch.zeros(3 * n ** 3 + 4, device="cuda")[0 if aligned else 1:][:3 * n ** 3].view(-1, 3) for _ in range(2)]
        assert (out[0].data_ptr() % 16 == 0) == aligned
        check(g.lib.cube_decompress(g.ctx, *(ctypes.c_void_p(o.data_ptr()) for o in out), g.n, 1))
    assert np.array_equal(out[0].cpu().numpy().astype(np.float64), ref.positions())
    assert np.array_equal(out[1].cpu().numpy().astype(np.float64), ref.velocities())
