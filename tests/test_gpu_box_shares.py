"""The reductions of the box-counting comparators where their work division
and their rounding change: particle counts around the one from which the
integer words stay below 2^50, clouds that leave most tiles empty or put
everything into one or two of them (shares of the records that end inside a
tile, or span many), meshes of one tile, of a few and of more than the sorted
scatter takes, ragged.  Against the oracle with the bars of the other tests of
these entry points: binary64 1e-12, and binary32 1e-5, since a term's binary32
arithmetic is good to a few ulps (5e-7) and the integer sums add nothing."""
import pytest

import oracle
import workloads as W
from helpers import as_precision, assert_fields_close, gpu_run
from test_gpu_cic import TOL, _check, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def _cloud(n, shape):
    cloud = W.abc_cloud(n, seed=41, jacobian=False)
    if shape == "one":            # within a sixteenth of the box
        cloud.x = 0.43 + cloud.x / 16
    elif shape == "two":          # two clumps at opposite corners, the rest empty
        cloud.x = cloud.x / 20
        cloud.x[:, ::3] += 0.94
    return cloud


MESHES = {"one tile": (9, 5, 7), "few": (37, 21, 19), "many": (170, 160, 140), "flat": (150, 70)}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("count", [1, 1025, 4095, 4096, 60001])
@pytest.mark.parametrize("shape", ["even", "one", "two"])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_shares(ctx, prec, count, shape, mesh):  # noqa: F811
    n = MESHES[mesh]
    dim = len(n)
    if mesh == "many" and count < 4096:
        count += 40000
    m = W.Mesh(dim, n, (0.0,) * dim, (1.0,) * dim, (True, False, True)[:dim])
    cloud = _cloud(count, shape)
    if dim == 2:
        cloud.x, cloud.v, cloud.ug = (t[:2].contiguous() for t in (cloud.x, cloud.v, cloud.ug))
    _check(ctx, m, cloud, prec, 0.7, f"{mesh} {shape} {count}")
    wl = W.small_random_3d(10, 4, seed=1) if dim == 3 else W.taylor_green_2d(per_axis=4, mesh_n=4, seed=1)
    wl.mesh = m
    S, den, st = gpu_run(ctx, wl, prec=prec, psicell_cloud=as_precision(cloud, prec), weight=0.7)
    Sref, counts, out, nf = oracle.psicell(m, as_precision(cloud, prec), 0.7, wl.rho_d, wl.mu, wl.delta,
                                          split=True)
    assert_fields_close(S, Sref, TOL[prec], f"box counts {mesh} {shape} {count} {prec}")
    assert (den == counts).all() and st["outside"] == out and st["skipped"] == nf
