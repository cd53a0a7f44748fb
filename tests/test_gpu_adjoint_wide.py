"""The extrapolation's adjoint of steps that some fit's scan window makes go over
the fields in memory, whose shares the blocks of one launch take in order:
windows of few and of many shares, a grid of fewer blocks than shares, layers
below the most, fits that fail for good, a periodic axis, and a snapshot taken
on the other path, which leaves the windows unknown.  Against the launches per
layer, at the bar of test_gpu_adjoint_fits (1e-12 of the largest component,
1e4 roundings)."""
import numpy as np
import pytest

import workloads
from test_gpu_adjoint_fits import _gradient

pytestmark = pytest.mark.gpu


def _thin(nx, ny, R, b=1.2, **kw):
    shape = {} if b is None else dict(shape="ellipse", b=b, theta=0.4)
    return workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.05,
                          solid=dict(cx=0.45 * nx, cy=0.55 * ny, R=R, G=0.01, rho_s=1.2, **shape),
                          **kw)


def _same(got, ref):
    assert abs(got[0] - ref[0]) <= 1e-12 * abs(ref[0]), (got[0], ref[0])
    assert abs(got[1] - ref[1]) <= 1e-12 * abs(ref[1]), (got[1], ref[1])
    assert np.max(np.abs(got[2] - ref[2])) <= 1e-12 * np.max(np.abs(ref[2]))


@pytest.mark.parametrize("cfg", [
    _thin(40, 36, 12.0, layers=3),
    _thin(64, 48, 18.0, layers=1),
    _thin(260, 200, 90.0),
    _thin(517, 413, 180.0, b=2.0),
    _thin(128, 128, 30.0, r_max=2),
    _thin(160, 90, 40.0, periodic_x=True),
    _thin(150, 131, 30.0, b=None, det_rel=0.33),
    _thin(139, 133, 30.0, b=None, det_rel=0.3, r_max=2),
], ids=lambda c: f"{c['nx']}x{c['ny']}")
def test_shared_layers_match_launches_per_layer(cfg):
    _same(_gradient(cfg, 512), _gradient(cfg, 0))


def test_snapshots_of_the_other_path():
    import torch
    from paper_2402_12696_amd import Sim, lbrmt as B
    cfg = _thin(131, 117, 21.0, b=None)
    out = []
    for back in (0, 512):
        sim = Sim(device="cuda:0", precision="f64", **cfg)
        sim.set_option(B.LBRMT_OPT_FUSED_FIT, 0)
        sim.init(workloads.cellular_velocity(131, 117, 0.03, 2, 7))
        snaps = [torch.empty(B.lbrmt_snapshot_bytes(sim.ctx), dtype=torch.uint8, device="cuda:0")
                 for _ in range(5)]
        adj = torch.empty(B.lbrmt_adjoint_bytes(sim.ctx), dtype=torch.uint8, device="cuda:0")
        for s in snaps:
            B.lbrmt_step_snapshot(sim.ctx, s)
        sim.set_option(B.LBRMT_OPT_FUSED_FIT, back)
        B.lbrmt_adjoint_zero(sim.ctx, adj)
        B.lbrmt_adjoint_loss(sim.ctx, adj, snaps[-1], 1, [50.0, 60.0, 0.1, -0.2, 0.3, -0.7, 0.9, 0.2])
        for s in reversed(snaps):
            B.lbrmt_adjoint_step(sim.ctx, adj, s)
        u0 = torch.empty(2, 117, 131, dtype=torch.float64, device="cuda:0")
        gG, gU = B.lbrmt_adjoint_init(sim.ctx, adj, snaps[0], u0)
        out.append((gG, gU, u0.cpu().numpy()))
        sim.close()
    _same(out[1], out[0])
