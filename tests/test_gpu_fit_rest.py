"""The block that finishes the tiles their copies cannot serve, where its list of
targets has edges: every layer at once, a few layers at a time (more targets
than the list has room for), and one layer by shares of the tiles (a layer of
its own larger than the list).  Long solids whose every tile is left to it, by
the check mode or by their wide scan windows, against one launch per layer: the
whole state bitwise."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def _long(nx, ny, R, b, theta=0.0, **kw):
    return workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.05,
                          solid=dict(cx=0.5 * nx, cy=0.5 * ny, R=R, b=b, theta=theta,
                                     shape="ellipse", G=0.01, rho_s=1.2), **kw)


def _run(cfg, prec, opt):
    from paper_2402_12696_amd import Sim, lbrmt as B
    sim = Sim(device="cuda:0", precision=prec, **cfg)
    sim.set_option(B.LBRMT_OPT_FUSED_FIT, opt)
    sim.init(workloads.cellular_velocity(cfg["nx"], cfg["ny"], 0.04, 3, 5))
    sim.step(3)
    out = _state(sim)
    sim.close()
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,cfg,opt", [
    ("all layers at once", _long(180, 64, 70.0, 1.0, 0.1), 512),
    ("seven layers", _long(180, 64, 70.0, 1.0, 0.1, layers=7), 512),
    ("a few layers at a time", _long(1500, 64, 700.0, 1.5), 1),
    ("a few layers, wide windows", _long(1400, 200, 660.0, 1.0, 0.1), 512),
    ("half of a disc's fits wide", _long(128, 120, 40.0, 40.0, det_rel=0.33), 512),
    ("all of a disc's fits wide", _long(128, 120, 40.0, 40.0, det_rel=0.6), 256),
    ("half of a disc's fits fail", _long(128, 120, 40.0, 40.0, det_rel=0.3, r_max=2), 512),
    ("a layer by shares (FP32: 11554 entries)", _long(6100, 64, 2960.0, 1.5), 1),
])
def test_left_tiles_are_bitwise_the_per_layer_path(name, cfg, opt, prec):
    assert _equal(_run(cfg, prec, 0), _run(cfg, prec, opt)), (name, prec)
