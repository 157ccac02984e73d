"""The general-mesh gather at the edges of its batches: numbers of records
around one, two and three batches of 64 (odd and even), work items of one cell
up to more than both sets of 64, one bucket and many, and boxes that lie in one
periodic image of a record or straddle two (kernels narrow and wide against the
box, closed and periodic axes mixed).  Against the oracle with the bars of the
other general-mesh tests: binary64 1e-12, binary32 1e-5, since a binary32 sum
runs over no more than a batch (64 x 6e-8 = 4e-6 at the worst) before it is
carried in binary64; pair counts exact."""
import pytest

import oracle  # noqa: F401  (the reference the helper compares with)
import workloads as W
import torch
from test_gpu_cells import _check, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def _some(wl, n):
    wl.traj = wl.traj.subset(torch.arange(n))
    return wl


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("records", [1, 2, 63, 64, 65, 127, 128, 193])
def test_records_around_a_batch(ctx, prec, records):  # noqa: F811
    """Every record reaches every cell of 5^3 in one bucket."""
    cells = W.scattered_cells(3, 5, (0.0,) * 3, (1.0,) * 3, (False,) * 3, seed=71)
    wl = _some(W.small_random_3d(400, 8, seed=72, periodic=False, h0=0.3), records)
    _check(ctx, cells, wl, prec, f"{records} records", per_bucket=1000)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dim,n,per_bucket", [(2, 1, 4), (2, 8, 64), (2, 9, 200), (2, 23, 130), (3, 4, 64), (3, 6, 300),
                                              (3, 9, 20), (3, 11, 129)])
@pytest.mark.parametrize("h0", [0.004, 0.05, 0.2])
@pytest.mark.parametrize("wrap", ["open", "periodic", "mixed"])
def test_items_and_images(ctx, prec, dim, n, per_bucket, h0, wrap):  # noqa: F811
    periodic = {"open": (False,) * 3, "periodic": (True,) * 3, "mixed": (True, False, True)}[wrap][:dim]
    cells = W.scattered_cells(dim, n, (0.0,) * dim, (1.0,) * dim, periodic, seed=73 + n)
    if dim == 3:
        wl = _some(W.small_random_3d(700, 8, seed=74, periodic=True, h0=h0), 331)
    else:
        wl = W.taylor_green_2d(per_axis=19, mesh_n=16, seed=75)
        wl.h0 = h0
    _check(ctx, cells, wl, prec, f"{dim}-D n={n} per_bucket={per_bucket} h0={h0} {wrap}", per_bucket=per_bucket)
