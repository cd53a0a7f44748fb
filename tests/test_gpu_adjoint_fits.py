"""The extrapolation's adjoint in one launch (tiles with recomputed margins,
one block where a scan window is wider than 2) against the launches per layer,
where its tiling has edges: windows of one tile and of several, layer counts
whose margins differ, a periodic axis narrower than a tile's copy, a thin
solid with wide windows.  Both sum the same terms in orders that atomics leave
open: 1e-12 of the largest component, 1e4 roundings."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _cfg(nx, ny, R, b=None, **kw):
    shape = {} if b is None else dict(shape="ellipse", b=b, theta=0.4)
    return workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.05,
                          solid=dict(cx=0.45 * nx, cy=0.55 * ny, R=R, G=0.01, rho_s=1.2, **shape),
                          **kw)


def _gradient(cfg, fused, T=7):
    import torch
    from paper_2402_12696_amd import Sim, lbrmt as B
    nx, ny = cfg["nx"], cfg["ny"]
    sim = Sim(device="cuda:0", precision="f64", **cfg)
    sim.set_option(B.LBRMT_OPT_FUSED_FIT, fused)
    sim.init(workloads.cellular_velocity(nx, ny, 0.03, 2, 7))
    ctx = sim.ctx
    snaps = [torch.empty(B.lbrmt_snapshot_bytes(ctx), dtype=torch.uint8, device="cuda:0")
             for _ in range(T)]
    adj = torch.empty(B.lbrmt_adjoint_bytes(ctx), dtype=torch.uint8, device="cuda:0")
    B.lbrmt_adjoint_zero(ctx, adj)
    for s in snaps:
        B.lbrmt_step_snapshot(ctx, s)
    coef = [0.4 * nx, 0.5 * ny, 0.1, -0.2, 0.3, -0.7, 0.9, 0.2]
    B.lbrmt_adjoint_loss(ctx, adj, snaps[-1], 1, coef)
    for n in reversed(range(T)):
        if n:
            B.lbrmt_adjoint_loss(ctx, adj, snaps[n], 0, coef)
        B.lbrmt_adjoint_step(ctx, adj, snaps[n])
    u0 = torch.empty(2, ny, nx, dtype=torch.float64, device="cuda:0")
    gG, gU = B.lbrmt_adjoint_init(ctx, adj, snaps[0], u0)
    sim.close()
    return gG, gU, u0.cpu().numpy()


@pytest.mark.parametrize("name,cfg", [
    ("one tile", _cfg(40, 36, 4.0, layers=3)),
    ("ragged tiles", _cfg(131, 117, 21.0)),
    ("one layer", _cfg(90, 80, 14.0, layers=1)),
    ("seven layers", _cfg(90, 80, 14.0, layers=7)),
    ("period 77", _cfg(77, 90, 13.0, periodic_x=True)),
    ("wide scan windows", _cfg(128, 128, 30.0, b=1.2)),
])
def test_one_launch_matches_launches_per_layer(name, cfg):
    ref, got = _gradient(cfg, 0), _gradient(cfg, 512)
    assert abs(got[0] - ref[0]) <= 1e-12 * abs(ref[0]), (name, got[0], ref[0])
    assert abs(got[1] - ref[1]) <= 1e-12 * abs(ref[1]), (name, got[1], ref[1])
    assert np.max(np.abs(got[2] - ref[2])) <= 1e-12 * np.max(np.abs(ref[2])), name
