"""The batch's extrapolation option: an untouched batch reads the default, -1,
and setting back what was read, or any other mode, keeps every bit."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu


def test_an_untouched_batch_reads_the_default_and_takes_it_back():
    from paper_2402_12696_amd import Batch, lbrmt as B
    cfgs = [workloads.make(nx=n, ny=n + 5, tau=0.8, lid_ux=0.05, periodic_x=n > 80,
                           solid=dict(cx=0.5 * n, cy=0.5 * n, R=0.15 * n, G=0.01, rho_s=1.1))
            for n in (48, 64, 90)]
    states = []
    for mode in (None, "read", 0, 1024):
        b = Batch(cfgs, precision="f64", device="cuda:0")
        assert b.get_option(B.LBRMT_OPT_FUSED_FIT) == -1
        if mode is not None:
            for o in (B.LBRMT_OPT_FUSED_FIT, B.LBRMT_OPT_GRAPH, B.LBRMT_OPT_LB_VARIANT):
                b.set_option(o, b.get_option(o))
            assert b.get_option(B.LBRMT_OPT_FUSED_FIT) == -1
        if isinstance(mode, int):
            b.set_option(B.LBRMT_OPT_FUSED_FIT, mode)
            assert b.get_option(B.LBRMT_OPT_FUSED_FIT) == mode
        b.init()
        b.step(14)
        states.append([_state(m) for m in b.members])
        b.close()
    for other in states[1:]:
        assert all(_equal(x, y) for x, y in zip(states[0], other))
