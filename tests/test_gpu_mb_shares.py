"""Several solids where the sharing-out of their work changes: extrapolation by
tiles for a few solids, by solid for many, and both at once when one of many
does not fit a block's copy; thin solids whose fits need wide scan windows on
either way.  Against the FP64 oracle at the bar of the parity tests."""
import pytest

import workloads
from test_gpu_multibody import _run as _run_mb

pytestmark = pytest.mark.gpu


def _many(n, extra=(), b=None, px=False):
    # n solids of nine tiles each, eight to a row (more than 56 of them are
    # extrapolated by solid), and the extra ones beside them
    shape = {} if b is None else dict(shape="ellipse", b=b, theta=0.6)
    solids = [dict(cx=30.0 + 48.0 * (k % 8), cy=28.0 + 48.0 * (k // 8), R=22.0, G=0.005,
                   rho_s=1.1, **shape) for k in range(n)]
    return workloads.make(nx=512, ny=48 * ((n + 7) // 8) + 60, tau=0.9, lid_ux=0.03,
                          periodic_x=px,
                          solids=solids + [dict(cx=455.0, cy=54.0, G=0.005, rho_s=1.2, **e)
                                           for e in extra])


@pytest.mark.parametrize("name,cfg", [
    ("few: by tiles", _many(5)),
    ("few, thin: by tiles", _many(5, b=0.9)),
    ("many: by solid", _many(60)),
    ("many, thin: by solid", _many(60, b=0.9)),
    ("many and a large one", _many(60, extra=[dict(R=38.0)])),
    ("many and a large thin one, moving windows",
     _many(60, extra=[dict(R=36.0, shape="ellipse", b=1.2, theta=1.2)], px=True)),
])
def test_shares_match_oracle(name, cfg):
    _run_mb(cfg, (1, 5))
