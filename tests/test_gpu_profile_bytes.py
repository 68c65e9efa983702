"""GPU: the bytes that the stage profile charges the coarse solve are those of
the sweeps it makes: three where an xy plane of the mesh fits LDS, else five,
each reading and writing the complex mesh once."""

import pytest

from cube_inputs import config

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("name,sweeps", [("c1", 3), ("c3cpu", 5)])
def test_coarse_solve_bytes(name, sweeps):
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = config(name)
    at = torch.arange(spec.n_side, device="cuda") + 0.5
    pos = torch.stack(torch.meshgrid(at, at, at, indexing="ij"), -1).flip(-1).reshape(-1, 3).contiguous()
    with CubeBox(spec) as g:
        g.compress(pos, torch.zeros_like(pos))
        g.profile(True)
        g.forces()
        stage = {s["name"]: s for s in g.profile_read()}["coarse_fft_green"]
        assert stage["launches"] == 1
        assert stage["bytes"] == 16.0 * sweeps * g.n_cells
