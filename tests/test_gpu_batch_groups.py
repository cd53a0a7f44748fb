"""A batch large enough to run its captured steps as two groups of members side
by side, against the same batch stepped eagerly (one group, one stream): every
member's state bitwise.  Members of uneven sizes, so that the groups differ in
number, and a run whose steps are partly captured, partly not."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def _run(cfgs, prec, graph, steps):
    from paper_2402_12696_amd import Batch, lbrmt as B
    b = Batch(cfgs, precision=prec, device="cuda:0")
    B.lbrmt_batch_set_option(b.batch, B.LBRMT_OPT_GRAPH, 1 if graph else 0)
    b.init()
    for n in steps:
        b.step(n)
    out = [_state(m) for m in b.members]
    b.close()
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [24, 31])
def test_two_groups_are_bitwise_one(n, prec):
    cfgs = []
    for k in range(n):
        L = 64 + 24 * (k * k % 5)
        cfgs.append(workloads.make(nx=L, ny=L + 8 * (k % 3), tau=0.8, lid_ux=0.05,
                                   solid=dict(cx=0.5 * L, cy=0.5 * L, R=(0.1 + 0.01 * (k % 9)) * L,
                                              G=0.01, rho_s=1.0 + 0.1 * (k % 2))))
    a = _run(cfgs, prec, True, (7, 12, 6, 1, 9))
    b = _run(cfgs, prec, False, (35,))
    assert all(_equal(x, y) for x, y in zip(a, b))
