"""GPU: a box without particles (new, or after a state that was refused) has
no mass, momentum or energy, whatever its particle planes hold."""

import numpy as np
import pytest

from cube_inputs import config
from tests.gpu_common import ics

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _is_empty(d):
    return d["mass"] == 0 and not d["momentum"].any() and d["kinetic"] == 0.0 and d["potential"] == 0.0


@pytest.mark.parametrize("vel_codec", [0, 1])
def test_diagnostics_of_an_empty_box(vel_codec):
    from paper_2003_03931_amd import CubeBox
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pos, vel = ics("c1")
    with CubeBox(config("c1").with_(vel_codec=vel_codec)) as g:
        assert _is_empty(g.diagnostics())
        g.compress(pos, vel)
        st = g.get_state()
        full = g.diagnostics()
        assert full["mass"] == g.n and full["kinetic"] > 0.0
        counts = st["counts"].copy()
        counts[0] += 1                               # do not sum to the particles
        with pytest.raises(Exception):
            g.set_state(counts, st["m"], st["u"], st["s"], st["M"], vc=st["vc"])
        assert _is_empty(g.diagnostics())
        g.set_state(st["counts"], st["m"], st["u"], st["s"], st["M"], vc=st["vc"])
        again = g.diagnostics()
    assert again["kinetic"] == full["kinetic"] and np.array_equal(again["momentum"], full["momentum"])
