"""GPU: the fine potential of tiles whose transforms have each of the supported
radix plans, periodic and buffered, from the density the device holds against the oracle's solve."""

import numpy as np
import pytest
import torch

from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu

# cells per side of the tile box: particles per side, tiles, coarse ratio, buffer, split radius
BOXES = {"p64": (32, 1, 4, 0, 5), "b48": (64, 4, 4, 8, 5), "b64": (64, 4, 4, 16, 12), "b96": (64, 2, 4, 16, 12),
         "p128": (64, 1, 4, 0, 12), "b160": (128, 2, 4, 16, 12), "p192": (96, 1, 4, 0, 12),
         "b192": (160, 2, 4, 16, 12)}


@pytest.mark.parametrize("name", list(BOXES))
def test_potential_of_the_held_density(name):
    import oracle
    from oracle import green, pm
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, nt, r, b, a = BOXES[name]
    spec = BoxSpec(name, n, nt, 2, r, b, a, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    assert box.F == int(name[1:])
    rng = np.random.default_rng(n)
    pos = rng.uniform(0, n, size=(n ** 3, 3)).astype(np.float32)
    pos[pos >= n] = 0.0
    vel = np.zeros((n ** 3, 3), np.float32)
    with CubeBox(spec) as g:
        g.compress(pos, vel)
        t = box.n_tiles - 1
        rho = g.debug_mesh(2, t).cpu().numpy()
        got = g.debug_mesh(3, t).cpu().numpy()
    ref = pm.solve(rho.transpose(2, 1, 0).astype(np.float64), green.fine_green(box)).transpose(2, 1, 0)
    # about 2 log2(F^3) roundings of 6e-8 each
    assert np.linalg.norm(got - ref) < 3e-6 * np.linalg.norm(ref)
