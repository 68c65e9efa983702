"""GPU: compress and decompress against the oracle where their kernels can go
wrong: shuffled input, cells with more particles than a workgroup walks,
positions outside the box, nothing moving, arrays that are not 16-byte
aligned, and a box whose tiles per side are no power of two."""

import ctypes

import numpy as np
import pytest
import torch

from cube_inputs import config
from cube_inputs.configs import DT, BoxSpec

pytestmark = pytest.mark.gpu


def _input(case, spec):
    n, L = spec.n_side ** 3, spec.n_side
    rng = np.random.default_rng(7)
    pos = rng.uniform(0, L, size=(n, 3)).astype(np.float32)
    pos[pos >= L] = 0.0
    vel = rng.normal(size=(n, 3)).astype(np.float32)
    if case == "dense":                        # two thirds of all particles in two cells
        pos[: n // 3] = rng.uniform(0.0, 1.9, size=(n // 3, 3)).astype(np.float32)
        pos[n // 3: 2 * (n // 3)] = (L - 2 + rng.uniform(0.1, 1.9, size=(n // 3, 3))).astype(np.float32)
        perm = rng.permutation(n)
        pos, vel = pos[perm], vel[perm]
    elif case == "outside":
        pos[::3] -= np.float32(L)
        pos[1::5] += np.float32(2 * L)
        pos[0] = [-0.0, L, -1e-6]
    elif case == "still":
        vel[:] = 0.0
    return np.ascontiguousarray(pos), np.ascontiguousarray(vel)


def _shifted(a):
    """The same values on the device, one float past a 16-byte boundary."""
    buf = torch.empty(a.size + 4, device="cuda")
    v = buf[1:1 + a.size].view(a.shape)
    v.copy_(torch.from_numpy(a))
    assert v.data_ptr() % 16 == 4
    return v


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("case", ["uniform", "dense", "outside", "still"])
@pytest.mark.parametrize("name", ["c1", "ragged"])
def test_codec_edges(name, case, aligned):
    import oracle
    from oracle import codec
    from paper_2003_03931_amd import CubeBox
    from paper_2003_03931_amd._lib import check
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = config("c1") if name == "c1" else BoxSpec("ragged", 96, 6, 2, 4, 16, 12, DT, 2.0, -2.0, 0.5, 1, 1)
    box = oracle.Box.from_spec(spec).validate()
    pos, vel = _input(case, spec)
    ref = codec.compress(box, pos, vel, with_ids=True)
    put = (lambda a: torch.from_numpy(a).cuda()) if aligned else _shifted
    with CubeBox(spec, with_ids=True, tiles_per_batch=1) as g:
        g.compress(put(pos), put(vel))
        st = g.get_state()
        x, v = put(np.zeros_like(pos)), put(np.zeros_like(vel))
        check(g.lib.cube_decompress(g.ctx, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(v.data_ptr()), g.n, 1))
    assert st["s"] == ref.s and st["M"] == ref.M
    assert np.array_equal(st["counts"], ref.counts.astype(np.int32))
    assert np.array_equal(st["ids"], ref.ids)
    assert np.array_equal(st["m"], ref.m) and np.array_equal(st["u"], ref.u)
    assert np.array_equal(x.cpu().numpy().astype(np.float64), ref.positions())
    assert np.array_equal(v.cpu().numpy().astype(np.float64), ref.velocities())
