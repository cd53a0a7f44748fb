"""The batch extrapolation's blocks where their shape changes: FP32 members of few
tiles in all (blocks of 512 threads), and of more (two blocks of 256 on a unit),
with the option set and read back, and members whose zone grows past the blocks
launched for it; and where captured steps become two groups of members (48, or
4 million nodes).  Against each member alone: the same bits."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def _cfg(nx, R, **kw):
    return workloads.make(nx=nx, ny=nx, tau=0.8, lid_ux=0.08,
                          solid=dict(cx=0.5 * nx, cy=0.55 * nx, R=R, G=0.002, rho_s=1.1), **kw)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,cfgs", [
    ("few tiles", [_cfg(64, 12.0), _cfg(96, 21.0), _cfg(64, 5.0)]),
    ("512 tiles", [_cfg(256, 50.0)] * 32),
    ("513 and more", [_cfg(256, 50.0)] * 32 + [_cfg(64, 4.0)]),
    ("47 members", [_cfg(64 + 8 * (k % 3), 9.0 + k % 5) for k in range(47)]),
    ("48 members, two groups", [_cfg(64 + 8 * (k % 3), 9.0 + k % 5) for k in range(48)]),
    ("4 million nodes, two groups", [_cfg(1424, 60.0), _cfg(1424, 70.0), _cfg(64, 9.0)]),
    ("a layer", [_cfg(64, 12.0, layers=1)] * 2),
])
def test_members_equal_single_contexts(name, cfgs, prec):
    from paper_2402_12696_amd import Batch, Sim
    b = Batch(cfgs, precision=prec, device="cuda:0")
    b.init()
    b.step(26)
    for k in (0, len(cfgs) // 2, len(cfgs) - 1):
        one = Sim(device="cuda:0", precision=prec, **cfgs[k]).init()
        one.step(26)
        assert _equal(_state(b.member(k)), _state(one)), (name, k)
        one.close()
    b.close()
