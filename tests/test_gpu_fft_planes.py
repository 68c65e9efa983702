"""GPU: the plane transforms of small cubes (every size up to the largest whose
xy plane is kept in LDS, and the smallest above) against numpy, both ways."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 80, 96, 112, 128])
def test_plane_transforms(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_03931_amd import fft3d
    rng = np.random.default_rng(n)
    x = (rng.standard_normal((n, n, n)) + 1j * rng.standard_normal((n, n, n))).astype(np.complex64)
    for inverse in (False, True):
        d = torch.from_numpy(x).cuda()
        fft3d(d, inverse=inverse)
        ref = np.fft.ifftn(x.astype(np.complex128)) * n ** 3 if inverse else np.fft.fftn(x.astype(np.complex128))
        # about log2(n^3) roundings of 6e-8 each
        assert np.linalg.norm(d.cpu().numpy() - ref) < 2e-6 * np.linalg.norm(ref)
