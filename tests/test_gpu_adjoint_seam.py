"""The extrapolation's adjoint in one launch on periodic axes where the last
tile of the window runs over the seam and holds images of the window's first
columns or rows: each node must be one tile's own.  Against the launches per
layer, at the bar of test_gpu_adjoint_fits (1e-12 of the largest component,
1e4 roundings)."""
import numpy as np
import pytest

import workloads
from test_gpu_adjoint_fits import _gradient

pytestmark = pytest.mark.gpu


def _periodic(nx, ny, R, px=True, py=False):
    return workloads.make(nx=nx, ny=ny, tau=0.8, periodic_x=px, periodic_y=py,
                          lid_ux=0.0 if py else 0.05, gravity=(2e-5, 1e-5),
                          solid=dict(cx=0.5 * nx, cy=0.5 * ny, R=R, G=0.01, rho_s=1.2))


@pytest.mark.parametrize("cfg", [
    _periodic(80, 120, 24.0),                   # window 5 .. 74, tiles to 100
    _periodic(80, 96, 25.5),                    # 4 .. 75
    _periodic(80, 120, 28.5),                   # 1 .. 78, layers up to the seam
    _periodic(110, 96, 38.0),                   # four tiles, 6 .. 103
    _periodic(96, 80, 25.5, px=False, py=True),
    _periodic(80, 80, 24.0, py=True),           # both seams
    _periodic(80, 110, 28.0, py=True),          # one tile row to spare along y
    _periodic(128, 96, 33.0),                   # no tile over the seam
], ids=lambda c: f"{c['nx']}x{c['ny']}")
def test_nodes_next_to_the_seam_count_once(cfg):
    ref, got = _gradient(cfg, 0), _gradient(cfg, 512)
    assert abs(got[0] - ref[0]) <= 1e-12 * abs(ref[0]), (got[0], ref[0])
    # (no lid where y is periodic)
    assert abs(got[1] - ref[1]) <= 1e-12 * abs(ref[1]), (got[1], ref[1])
    assert np.max(np.abs(got[2] - ref[2])) <= 1e-12 * np.max(np.abs(ref[2]))
