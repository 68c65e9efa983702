"""GPU: pair forces of rows of other lengths than 8 and 16 cells: 4, the
shortest, 24, between two powers of two, and 32."""

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOXES = {4: BoxSpec("r4", 32, 4, 4, 8, 8, 5, DT, 2.0, -2.0, 0.2, 1, 1),
         24: BoxSpec("r24", 48, 2, 4, 4, 16, 12, DT, 2.0, -2.0, 0.2, 1, 1),
         32: BoxSpec("r32", 32, 1, 4, 4, 0, 12, DT, 2.0, -2.0, 0.2, 1, 1)}


@pytest.mark.parametrize("cells", [4, 24, 32])
@pytest.mark.parametrize("npp", [2, 4])
def test_pair_forces_of_row_lengths(cells, npp):
    import oracle
    from oracle import pm
    from oracle.codec import State
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = BOXES[cells].with_(pp_range=npp)
    box = oracle.Box.from_spec(spec).validate()
    assert box.Tc == cells
    # nine cells in ten empty, the last cell of every row well filled
    rng = np.random.default_rng(cells)
    n = box.n_side ** 3
    w = np.where(rng.random(box.n_cells) < 0.1, rng.exponential(1.0, box.n_cells), 0.0)
    w[box.Tc - 1::box.Tc] += 0.5
    counts = np.bincount(rng.choice(box.n_cells, n, p=w / w.sum()), minlength=box.n_cells)
    m = rng.integers(0, 256, size=(3, n), dtype=np.uint8)
    st = State(box, counts.astype(np.int64), m, np.zeros((3, n), np.int8), 1.0, 0, np.arange(n, dtype=np.uint32))
    with CubeBox(spec, with_ids=True) as g:
        g.set_state(st.counts, st.m, st.u, st.s, st.M, st.ids, st.step)
        got = g.forces().cpu().numpy()
    # FP32 sums of some tens of pairs, the bound of the forces elsewhere
    assert rel_l2(got, pm.Solver(box).forces(st, workers=1)) <= 1e-5
