"""Solids among several whose fits need wide scan windows, or fail for good: by
tiles, by solid, on windows that a block's copy holds and that it does not,
with periodic axes that wrap inside the copy.  Their maps after one step from a
moving fluid (densities alike, so that nothing but the solid itself decides
them) against contexts of that solid alone with one launch per layer: the same
bits, and as many fits that fail."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _row(n, R, b, pitch=48, theta=0.6):
    # eight to a row; every third turned by another angle
    return [dict(cx=30.0 + pitch * (k % 8), cy=28.0 + pitch * (k // 8) + 0.3 * (k % 5), R=R,
                 G=0.005, rho_s=1.0, shape="ellipse", b=b, theta=theta + 0.7 * (k % 3))
            for k in range(n)]


def _many(n, R=22.0, b=0.9, **kw):
    kw.setdefault("layers", 11)
    return dict(nx=512, ny=48 * ((n + 7) // 8) + 60, solids=_row(n, R, b), **kw)


CASES = {
    "few: by tiles, then whole": _many(5),
    "many: by solid": _many(60),
    "many, a line of nodes": _many(60, b=0.45),
    "many, r_max 2": _many(60, r_max=2),
    "many, r_max 3": _many(60, b=0.6, r_max=3),
    "many, five layers": _many(60, layers=5),
    "many, the large ones last": dict(nx=512, ny=450, solids=_row(56, 22.0, 0.9) + [
        dict(cx=455.0, cy=60.0, R=40.0, G=0.005, rho_s=1.0, shape="ellipse", b=1.2, theta=1.2),
        dict(cx=440.0, cy=180.0, R=38.0, G=0.005, rho_s=1.0),
        dict(cx=452.0, cy=330.0, R=90.0, G=0.005, rho_s=1.0, shape="ellipse", b=1.1, theta=1.5)]),
    "by tiles, a large one among small": dict(nx=400, ny=300, solids=[
        dict(cx=20.0 + 30.0 * k, cy=30.0, R=4.0, G=0.005, rho_s=1.0) for k in range(5)] + [
        dict(cx=220.0, cy=170.0, R=80.0, G=0.005, rho_s=1.0),
        dict(cx=90.0, cy=120.0, R=40.0, G=0.005, rho_s=1.0, shape="ellipse", b=1.0, theta=1.4)]),
    "beyond the copy": dict(nx=300, ny=260, solids=[
        dict(cx=150.0, cy=90.0, R=100.0, G=0.005, rho_s=1.0, shape="ellipse", b=1.2, theta=0.1),
        dict(cx=140.0, cy=190.0, R=90.0, G=0.005, rho_s=1.0, shape="ellipse", b=0.8, theta=0.9)]),
    "a period as wide as the copy": dict(nx=96, ny=300, periodic_x=True, solids=[
        dict(cx=48.0, cy=60.0 + 80.0 * k, R=33.5, G=0.005, rho_s=1.0, shape="ellipse", b=1.1,
             theta=0.05) for k in range(3)]),
    "a short period": dict(nx=70, ny=120, periodic_x=True, layers=5, solids=[
        dict(cx=35.0, cy=30.0 + 50.0 * k, R=27.5, G=0.005, rho_s=1.0, shape="ellipse", b=1.1,
             theta=0.05) for k in range(2)]),
    "more layers than one launch": _many(5, layers=13),
    # (a disc's fits at half-width 2 have det / (sum w)^3 between 0.2 and 0.5)
    "few, some fits wide": _many(5, b=22.0, det_rel=0.25),
    "few, half of the fits wide": _many(5, b=22.0, det_rel=0.33),
    "many, half of the fits wide": _many(60, b=22.0, det_rel=0.33),
    "few, all wide: more than the list holds": _many(5, b=22.0, det_rel=0.6),
    "many, all wide: more than the list holds": _many(60, b=22.0, det_rel=0.6),
    "few, half of the fits fail": _many(5, b=22.0, det_rel=0.3, r_max=2),
    "many, half of the fits fail": _many(60, b=22.0, det_rel=0.3, r_max=2),
    "few, thirteen layers, half fail": _many(4, R=15.0, b=15.0, layers=13, det_rel=0.3, r_max=2),
    "twenty layers, round": _many(5, R=12.0, b=12.0, layers=20),
    "thirteen layers, r_max 2": _many(5, R=15.0, layers=13, r_max=2),
}


def check_maps(cfg, prec, sample=None):
    """The maps of the sampled solids (all by default) after one step."""
    from paper_2402_12696_amd import Sim, lbrmt as B
    cfg = dict(cfg)
    solids = cfg.pop("solids")
    base = workloads.make(tau=0.9, lid_ux=0.03, **cfg)
    u0 = workloads.cellular_velocity(base["nx"], base["ny"], 0.05, 3, 11)
    many = Sim(device="cuda:0", precision=prec, **dict(base, solids=solids)).init(u0)
    many.step(1)
    fails = 0
    for k in sample or range(len(solids)):
        one = Sim(device="cuda:0", precision=prec, **dict(base, solid=solids[k]))
        one.set_option(B.LBRMT_OPT_FUSED_FIT, 0)
        one.init(u0)
        one.step(1)
        for a, b in zip(many.refmap(k), one.refmap()):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy(), equal_nan=True), k
        fails += one.diag(raise_unstable=False)["health"]["extrap_fail"]
        one.close()
    if sample is None:
        assert many.diag(raise_unstable=False)["health"]["extrap_fail"] == fails
    many.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", CASES)
def test_maps_are_bitwise_those_of_the_solid_alone(name, prec):
    n = len(CASES[name]["solids"])
    check_maps(CASES[name], prec, None if n < 8 else [*range(0, 56, 7), *range(56, n)])
