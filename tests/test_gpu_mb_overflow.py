"""Force blocks that more solids meet than a block holds (32): the first 32 in
index order count, the others are counted in the capacity health counter, and
no order in which a block finds them changes that, also beyond the 256 that are
put in order at once.  Two heaps of solids of alike regions, the indices of one
spread so that the threads that find its first solids come to them late;
against a context of the first 32 of each heap: the same bits."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _solid(k, heap):
    # (centres apart by far less than a node: alike regions)
    return dict(cx=(12.25 if heap else 46.25) + 1e-5 * k, cy=15.5, R=5.0,
                G=0.001 * (1 + k % 7), rho_s=1.0 + 0.1 * (k % 5))


def _run(solids):
    from paper_2402_12696_amd import Sim
    cfg = workloads.make(nx=60, ny=32, tau=0.8, lid_ux=0.05, layers=3, gravity=(0.0, -1e-5),
                         eta=0.5, solids=solids)
    sim = Sim(device="cuda:0", precision="f64", **cfg).init()
    sim.step(3)
    out = [t.cpu().numpy() for t in sim.force() + sim.macro()]
    health = sim.diag(raise_unstable=False)["health"]
    sim.close()
    return out, health


@pytest.mark.parametrize("n", [40, 256, 300, 2400])
def test_the_first_solids_by_index_count(n):
    near = [k >= 960 and (k < 992 or k % 256 < 64) if n > 1000 else k % 2 == 0 for k in range(n)]
    solids = [_solid(k, h) for k, h in enumerate(near)]
    heap = lambda h: [s for s, q in zip(solids, near) if q == h][:32]  # noqa: E731
    first = sorted(heap(True) + heap(False), key=solids.index)
    got, over = _run(solids)
    ref, _ = _run(first)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    assert (over["list_overflow"] > 0) == (n > 64)
