"""GPU: pair forces of rows too full to be staged at once: several batches of
particles, neighbour rows staged in groups of nine to one, single rows that
exceed the stage, and nearly empty rows beside them."""

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOXES = {"p16": BoxSpec("p16", 32, 1, 2, 4, 0, 12, DT, 2.0, -2.0, 0.2, 1, 1),
         "b8": BoxSpec("b8", 32, 2, 2, 4, 8, 5, DT, 2.0, -2.0, 0.2, 1, 1)}


def _counts(box):
    """Cells of 40, 80 and 300 particles in 3 x 3 rows each, a few of 1300 in a row, some in all others."""
    rng = np.random.default_rng(3)
    nc = box.n_coarse
    mesh = np.zeros((nc, nc, nc), np.int64)               # z, y, x
    mesh[1:4, 1:4] = rng.poisson(40, (3, 3, nc))
    mesh[6:9, 6:9] = rng.poisson(80, (3, 3, nc))
    mesh[12:14, 12:14, :6] = rng.poisson(300, (2, 2, 6))
    mesh[13, 3, 5:9] = 1300
    left = box.n_side ** 3 - int(mesh.sum())
    assert left > 0
    free = np.flatnonzero(mesh.reshape(-1) == 0)
    mesh.reshape(-1)[free] += rng.multinomial(left, np.full(free.size, 1.0 / free.size))
    z, y, x = np.indices(mesh.shape)
    counts = np.zeros(box.n_cells, np.int64)
    counts[box.canon(x.reshape(-1), y.reshape(-1), z.reshape(-1))] = mesh.reshape(-1)
    return counts


@pytest.mark.parametrize("name,npp", [("p16", 4), ("p16", 1), ("b8", 4), ("b8", 2)])
def test_pair_forces_of_dense_rows(name, npp):
    import oracle
    from oracle import pm
    from oracle.codec import State
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = BOXES[name].with_(pp_range=npp)
    box = oracle.Box.from_spec(spec).validate()
    n = box.n_side ** 3
    rng = np.random.default_rng(npp)
    m = rng.integers(0, 256, size=(3, n), dtype=np.uint8)
    m[:, ::7] = rng.choice([0, 1, 127, 128, 254, 255], size=m[:, ::7].shape).astype(np.uint8)
    st = State(box, _counts(box), m, np.zeros((3, n), np.int8), 1.0, 0, np.arange(n, dtype=np.uint32))
    with CubeBox(spec, with_ids=True) as g:
        g.set_state(st.counts, st.m, st.u, st.s, st.M, st.ids, st.step)
        got = g.forces().cpu().numpy()
    # FP32 sums of up to some hundreds of pairs, the bound of the forces elsewhere
    assert rel_l2(got, pm.Solver(box).forces(st, workers=1)) <= 1e-5
