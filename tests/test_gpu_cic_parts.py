"""Cloud-in-cell with few particles to a tile: the reduction takes a tile, or parts
of a tile of many records, to a workgroup.  Clouds whose particles lie in one
tile, in two, in a row of them and everywhere, with counts around the multiples of
a part, below and above the mean from which it takes equal shares, against the
oracle with the bars of the other tests of this entry point."""
import pytest

import workloads as W
from test_gpu_cic import _check, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("shape", ["even", "one", "two", "row"])
@pytest.mark.parametrize("n, count", [((200, 190), 4 * 4225 * 3 - 1), ((200, 190), 4 * 4225 * 3), ((200, 190), 60000),
                                      ((200, 190), 16 * 4225 * 3 + 1), ((50, 41, 37), 2601 * 9 + 1),
                                      ((50, 41, 37), 90001), ((200, 190), 16 * 4225 + 77), ((170, 160, 140), 1377 * 30)])
def test_parts(ctx, prec, shape, n, count):  # noqa: F811
    dim = len(n)
    cloud = W.abc_cloud(count, seed=43, jacobian=False)
    if dim == 2:
        cloud.x, cloud.v, cloud.ug = (t[:2].contiguous() for t in (cloud.x, cloud.v, cloud.ug))
    if shape == "one":
        cloud.x = 0.43 + cloud.x / 64
    elif shape == "two":
        cloud.x = cloud.x / 40
        cloud.x[:, ::3] += 0.94
    elif shape == "row":
        cloud.x[1:] = 0.3 + cloud.x[1:] / 50
    m = W.Mesh(dim, n, (0.0,) * dim, (1.0,) * dim, (True, False, True)[:dim])
    _check(ctx, m, cloud, prec, 0.7, f"parts {shape} {count}")
