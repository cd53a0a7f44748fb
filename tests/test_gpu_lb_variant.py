"""The lattice tile shape on lattices small enough that the force pass takes the
update along: a shape that was asked for is a launch of its own, the one that
the autotuner chose is not, and the state has the same bits on every route."""
import pytest

import workloads
from test_gpu_fused_fit import _equal, _state

pytestmark = pytest.mark.gpu

CFG = workloads.make(nx=131, ny=70, tau=0.8, lid_ux=0.05,
                     solid=dict(cx=60.0, cy=36.0, R=11.0, G=0.01, rho_s=1.2))


def _run(prec, prepare):
    from paper_2402_12696_amd import Sim
    sim = Sim(device="cuda:0", precision=prec, **CFG).init()
    sim.step(7)
    prepare(sim)
    sim.step(13)
    out = _state(sim)
    sim.close()
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_every_tile_shape_gives_the_same_bits(prec):
    from paper_2402_12696_amd import lbrmt as B
    ref = _run(prec, lambda sim: None)
    default = 3 if prec == "f64" else 5

    def ask(v):
        def f(sim):
            sim.set_option(B.LBRMT_OPT_LB_VARIANT, v)
            assert sim.get_option(B.LBRMT_OPT_LB_VARIANT) == v
        return f

    for v in (0, 1, 7, default):
        assert _equal(ref, _run(prec, ask(v))), v

    def there_and_back(sim):
        ask(1)(sim)
        sim.step(2)
        ask(default)(sim)

    def same_steps(sim):
        sim.step(2)

    assert _equal(_run(prec, same_steps), _run(prec, there_and_back))

    def tune(sim):
        v, _ = sim.autotune(2)
        assert sim.get_option(B.LBRMT_OPT_LB_VARIANT) == v

    assert _equal(ref, _run(prec, tune))
