"""The lattice update outside the window as blocks of the force pass (small
grids) against the launch beside the chain and against one stream without
overlap: the whole state bitwise, on grids of ragged tile counts, windows that
cover the grid and windows that cover little of it, runs of lengths that split
the captured sequences."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def _cfg(nx, ny, R, **kw):
    return workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.0 if kw.get("periodic_y") else 0.05,
                          solid=dict(cx=0.45 * nx, cy=0.55 * ny, R=R, G=0.01, rho_s=1.2), **kw)


def _run(cfg, prec, steps, opts):
    from paper_2402_12696_amd import Sim
    sim = Sim(device="cuda:0", precision=prec, **cfg)
    for o, v in opts.items():
        sim.set_option(o, v)
    sim.init()
    for n in steps:
        sim.step(n)
    out = _state(sim)
    sim.close()
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,cfg", [
    ("window over the grid", _cfg(33, 31, 9.0)),
    ("ragged", _cfg(259, 67, 12.0)),
    ("periodic", _cfg(513, 130, 20.0, periodic_x=True, periodic_y=True)),
    ("small solid", _cfg(640, 385, 4.0, layers=3)),
])
def test_update_along_the_force_pass_is_bitwise_the_launch_beside(name, cfg, prec):
    from paper_2402_12696_amd import lbrmt as B
    steps = (1, 5, 4, 13, 2)
    got = _run(cfg, prec, steps, {})
    assert _equal(got, _run(cfg, prec, (25,), {})), name
    assert _equal(got, _run(cfg, prec, steps, {B.LBRMT_OPT_GRAPH: 0})), name
    assert _equal(got, _run(cfg, prec, steps, {B.LBRMT_OPT_BULK_EARLY: 0})), name
    assert _equal(got, _run(cfg, prec, steps, {B.LBRMT_OPT_OVERLAP: 0})), name
