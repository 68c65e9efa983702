"""GPU: the radix sort where its last tile is partial (numbers of particles
that are no multiple of a tile's 8192): in encoding, and in the sorted
compaction of a step."""

import numpy as np
import pytest

from cube_inputs.configs import DT, BoxSpec
from tests.gpu_common import check_compaction

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# four fine cells per spacing: one particle per coarse cell
BOXES = {"48": BoxSpec("48", 48, 2, 4, 4, 16, 12, DT, 2.0, -2.0, 0.5, 1, 1),
         "80": BoxSpec("80", 80, 5, 4, 4, 16, 12, DT, 2.0, -2.0, 0.5, 1, 1)}


@pytest.mark.parametrize("name", sorted(BOXES))
def test_partial_last_tile(name):
    import oracle
    from oracle import codec
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = BOXES[name]
    n, side = spec.n_side ** 3, spec.n_side
    assert n % 8192
    rng = np.random.default_rng(side)
    pos = rng.uniform(0, side, size=(n, 3)).astype(np.float32)
    pos[pos >= side] = 0.0
    pos[: n // 4] = rng.uniform(0.0, 3.9, size=(n // 4, 3)).astype(np.float32)     # long runs of equal keys
    vel = rng.normal(scale=0.1, size=(n, 3)).astype(np.float32)
    perm = rng.permutation(n)
    pos, vel = pos[perm], vel[perm]
    box = oracle.Box.from_spec(spec).validate()
    ref = codec.compress(box, pos, vel, with_ids=True)
    with CubeBox(spec, with_ids=True) as g:
        g.compress(pos, vel)
        before = g.get_state()
        g.debug_force(2, 1)                          # the sorted compaction
        g.step(1)
        after = g.get_state()
    assert np.array_equal(before["counts"], ref.counts.astype(np.int32))
    assert np.array_equal(before["ids"], ref.ids)
    assert np.array_equal(before["m"], ref.m) and np.array_equal(before["u"], ref.u)
    check_compaction(box, before, after)
