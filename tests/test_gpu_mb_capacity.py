"""A block's copy of a whole solid at its capacity (7168 nodes of window and rim):
solids just inside, exactly at and just beyond it, among enough others that they
are extrapolated by solid (more than 512 tiles in all; fewer solids go by
tiles, whatever their size).  Maps after one step against each solid alone, as
test_gpu_mb_wide compares them."""
import pytest

from test_gpu_mb_wide import check_maps

pytestmark = pytest.mark.gpu

FB, LIMIT = 11 + 2, 7168  # layers and rim on each side


def _others():
    # 60 discs of 3 x 3 tiles
    return [dict(cx=30.0 + 48.0 * (k % 8), cy=28.0 + 48.0 * (k // 8), R=22.0, G=0.005, rho_s=1.0)
            for k in range(60)]


def _nodes(a, b):
    # window and rim of an axis-parallel ellipse at a whole node's corner
    return (2 * int(a) + 2 * FB) * (2 * int(b) + 2 * FB)


def _solid(cy, a, b):
    return dict(cx=452.0, cy=cy, R=a, b=b, theta=0.0, shape="ellipse", G=0.005, rho_s=1.0)


def test_the_sizes_lie_about_the_capacity():
    assert _nodes(28, 28) <= LIMIT - 200 and _nodes(29, 29) <= LIMIT
    assert _nodes(19, 43) == LIMIT and _nodes(19, 44) > LIMIT and _nodes(30, 30) > LIMIT
    assert 60 * 9 > 512


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("extra", [
    [_solid(60.0, 28.0, 28.0), _solid(160.0, 29.0, 29.0), _solid(260.0, 19.0, 43.0)],
    [_solid(60.0, 30.0, 30.0), _solid(160.0, 19.0, 44.0), _solid(300.0, 33.0, 33.0)],
    [_solid(100.0, 19.0, 43.0), _solid(250.0, 38.0, 38.0)],
], ids=["within", "beyond", "both"])
def test_solids_at_the_copys_capacity(extra, prec):
    solids = _others() + extra
    check_maps(dict(nx=512, ny=444, solids=solids), prec, [0, 33, *range(60, len(solids))])
