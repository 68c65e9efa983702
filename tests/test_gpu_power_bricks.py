"""GPU: the power spectrum's mesh where some of its large bricks hold so many
particles that small ones take them, with 32- and 64-bit accumulators."""

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# diagnostic cells per coarse cell: side, tiles, fine cells per spacing, coarse ratio, buffer, cells of a full row, particles of each
BOXES = {2: (128, 2, 2, 4, 16, 12, 2000), 4: (128, 2, 2, 8, 16, 6, 6000), 8: (128, 1, 1, 8, 0, 4, 20000)}


@pytest.mark.parametrize("ratio,narrow", [(2, False), (4, False), (8, False), (8, True)])
def test_full_bricks(ratio, narrow):
    import oracle
    from oracle import diag
    from oracle.codec import State
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, tiles, f, r, b, cells, each = BOXES[ratio]
    spec = BoxSpec(f"bricks{ratio}", n, tiles, f, r, b, 12, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    rng = np.random.default_rng(ratio)
    counts = np.zeros(box.n_cells, np.int64)
    if narrow:                                        # a full window without a full 2 x 2 x 2 block: 32-bit sums
        x, y, z = np.indices((6, 6, 6)).reshape(3, -1) + 5
        counts[box.canon(x, y, z)] = 1600
    for at in () if narrow else (0, box.n_cells - cells, *rng.integers(0, box.n_cells // 16 - 1, 4) * 16):
        counts[at:at + cells] = each                  # consecutive cells of an x row
    left = n ** 3 - int(counts.sum())
    counts += rng.multinomial(left, np.full(box.n_cells, 1.0 / box.n_cells))
    m = rng.integers(0, 256, size=(3, n ** 3), dtype=np.uint8)
    ref = State(box, counts, m, np.zeros((3, n ** 3), np.int8), 1.0, 0, np.arange(n ** 3, dtype=np.uint32))
    k_o, p_o, n_o = diag.power_spectrum(ref)
    with CubeBox(spec, tiles_per_batch=1) as g:
        g.set_state(counts, m, ref.u, 1.0, 0)
        k, p, modes = g.power_spectrum()
    assert np.array_equal(modes, n_o) and np.allclose(k, k_o, rtol=1e-12)
    # FP32 transform: some 20 roundings of 6e-8 of the rms amplitude, shells
    # within a factor ten of the mean power
    assert np.max(np.abs(p / p_o - 1.0)) <= 1e-5
