"""The step autotuner advances a simulation only where it is said to choose: one
solid on walled axes with at most 11 layers.  Any other context keeps its
options, its step count and its state."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def _cfg(nx, ny, **kw):
    return workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.0 if kw.get("periodic_y") else 0.05,
                          solid=dict(cx=0.5 * nx, cy=0.5 * ny, R=10.0, G=0.01, rho_s=1.2), **kw)


@pytest.mark.parametrize("cfg", [
    _cfg(96, 64, periodic_x=True),
    _cfg(64, 96, periodic_y=True),
    _cfg(90, 96, periodic_x=True, periodic_y=True),
    _cfg(64, 64, periodic_x=True),   # a period narrower than a tile's copy
    _cfg(64, 64, layers=12),
], ids=["x", "y", "both", "short", "12 layers"])
def test_a_context_without_the_choice_is_left_alone(cfg):
    from paper_2402_12696_amd import Sim
    from paper_2402_12696_amd import lbrmt as B
    sim = Sim(device="cuda:0", precision="f64", **cfg).init()
    sim.step(8)
    before = _state(sim)
    mode, ms = sim.autotune_steps(6)
    assert (mode, ms) == (-1, 0.0)
    assert sim.step_count == 8 and sim.get_option(B.LBRMT_OPT_FUSED_FIT) == -1
    assert _equal(before, _state(sim))
    sim.close()
