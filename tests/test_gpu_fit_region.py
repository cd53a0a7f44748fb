"""The block-wide extrapolation (every layer of a tile, or of a whole solid,
from a copy in LDS) where its dispatch and its copy have edges: one solid
against the one-launch-per-layer path, bitwise (the copy of a periodic axis
just as wide as the period, one node too wide, windows that meet themselves
across the seam, layer counts whose margins differ); several solids at the
copy's capacity against the FP64 oracle at the bar of the parity tests."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _run
from test_gpu_multibody import _run as _run_mb

pytestmark = pytest.mark.gpu


def _channel(nx, ny, R, layers=11, px=True, py=False, b=None, r_max=8):
    shape = {} if b is None else dict(shape="ellipse", b=b, theta=0.5)
    return workloads.make(nx=nx, ny=ny, tau=0.9, periodic_x=px, periodic_y=py,
                          lid_ux=0.0 if py else 0.03, gravity=(2e-5, 1e-5 if py else 0.0),
                          layers=layers, r_max=r_max,
                          solid=dict(cx=0.5 * nx, cy=0.5 * ny, R=R, G=0.005, rho_s=1.2, **shape))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,cfg", [
    ("period 76, the copy's width", _channel(76, 64, 14.0)),
    ("period 75, one launch per layer", _channel(75, 64, 14.0)),
    ("window next to the seam", _channel(80, 96, 25.5)),
    ("window across the whole period", _channel(80, 120, 28.5)),
    ("both axes periodic", _channel(97, 83, 22.0, py=True)),
    ("one layer", _channel(90, 70, 12.0, layers=1)),
    ("two layers", _channel(90, 70, 12.0, layers=2, px=False)),
    ("three layers", _channel(90, 70, 12.0, layers=3, px=False)),
    ("ten layers", _channel(90, 70, 12.0, layers=10)),
    ("fits that fail for good", _channel(96, 80, 20.0, b=1.2, r_max=2)),
])
def test_region_extrapolation_is_bitwise_the_per_layer_path(name, cfg, prec):
    ref = _run(cfg, prec, 0, 40)
    for opt in (512, 256, 1):
        assert _equal(ref, _run(cfg, prec, opt, 40)), (name, prec, opt)


@pytest.mark.parametrize("R", [28.0, 29.0, 33.0])
def test_several_solids_at_the_copy_capacity_match_oracle(R):
    # the window of R = 28 fits the 7168-node copy, that of R = 29 does not
    # (every layer on the maps); each beside a small solid
    _run_mb(workloads.make(nx=150, ny=110, tau=0.9, lid_ux=0.03,
                           solids=[dict(cx=45.0, cy=52.0, R=R, G=0.005, rho_s=1.2),
                                   dict(cx=115.0, cy=60.0, R=11.0, G=0.005, rho_s=1.1)]), (1, 40))
