"""GPU: pair forces where the runs of partners end at row ends, the next rows
are nearly empty, cells hold more pairs in reach than a thread lists at a time
and positions lie on the cells' faces."""

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# rows of 16 cells of one periodic tile, of 8 cells of 2^3 tiles, and of 16
# cells of which some rows hold so many particles that they are staged in pieces
BOXES = {"p16": BoxSpec("p16", 32, 1, 2, 4, 0, 12, DT, 2.0, -2.0, 0.2, 1, 1),
         "b8": BoxSpec("b8", 32, 2, 2, 4, 8, 5, DT, 2.0, -2.0, 0.2, 1, 1),
         "slab": BoxSpec("slab", 32, 1, 2, 4, 0, 12, DT, 2.0, -2.0, 0.2, 1, 1)}


def _state(spec, box):
    """Particles in some of the cells, the most of them in the end cells of the tiles' rows."""
    from oracle.codec import State
    rng = np.random.default_rng(spec.pp_range)
    n, cells = box.n_side ** 3, box.n_cells
    w = np.where(rng.random(cells) < 0.25, rng.exponential(1.0, cells), 0.0)
    x = np.arange(cells) % box.Tc                   # a row's cells are consecutive
    w[(x == 0) | (x == box.Tc - 1)] *= 3.0
    if spec.name == "slab":
        w[:] = 0.1 * w.mean()
        w.reshape(16, 16, 16)[3:7, 3:7] = rng.uniform(2.0, 8.0, (4, 4, 16))
    counts = np.floor(w / w.sum() * n).astype(np.int64)
    counts[rng.choice(np.flatnonzero(w), n - int(counts.sum()), replace=False)] += 1
    m = rng.integers(0, 256, size=(3, n), dtype=np.uint8)
    m[:, ::5] = rng.choice([0, 1, 127, 128, 254, 255], size=m[:, ::5].shape).astype(np.uint8)
    return State(box, counts, m, np.zeros((3, n), np.int8), 1.0, 0, np.arange(n, dtype=np.uint32))


@pytest.mark.parametrize("name,npp", [("p16", 4), ("b8", 1), ("b8", 4), ("slab", 4)])
def test_pair_forces_at_row_ends(name, npp):
    import oracle
    from oracle import pm
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = BOXES[name].with_(pp_range=npp)
    box = oracle.Box.from_spec(spec).validate()
    st = _state(spec, box)
    with CubeBox(spec, with_ids=True) as g:
        g.set_state(st.counts, st.m, st.u, st.s, st.M, st.ids, st.step)
        got = g.forces().cpu().numpy()
    # FP32 sums of some tens of pairs, the bound of the forces elsewhere
    assert rel_l2(got, pm.Solver(box).forces(st, workers=1)) <= 1e-5
