"""Layer numbers at the edges of the distance transform's forms (rows as words
up to 16 layers, scans beyond, up to 31), one launch per layer, against the
FP64 oracle: the node sets exactly, the maps within what L layers of
extrapolations can make of rounding (each at most about doubles it)."""
import pytest

import workloads
from oracle import Oracle
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers", [12, 16, 17, 31])
@pytest.mark.parametrize("nx,ny,px,R,b", [(131, 117, False, 17.0, 6.0), (150, 140, True, 2.2, 2.2)])
def test_layer_counts_match_oracle(layers, nx, ny, px, R, b):
    from paper_2402_12696_amd import Sim
    cfg = workloads.make(nx=nx, ny=ny, tau=0.8, lid_ux=0.05, periodic_x=px, layers=layers,
                         solid=dict(cx=0.43 * nx, cy=0.55 * ny, R=R, G=0.01, rho_s=1.1,
                                    shape="ellipse", b=b, theta=0.7))
    u0 = workloads.cellular_velocity(nx, ny, 0.05, 2, 3)
    sim = Sim(device="cuda:0", **cfg).init(u0)
    ref = Oracle(**cfg).init(u0)
    for n in (1, 3, 12):
        sim.step(n)
        ref.step(n)
        compare(sim, ref, tol=max(1e-10, 2.0 ** (layers - 52)), what=f"{layers} layers, +{n}")
    sim.close()
