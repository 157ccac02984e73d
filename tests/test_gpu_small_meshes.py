"""Small meshes, whose tiles are shared by several workgroups, against the
batched entry point, which has one workgroup per tile or part: bit for bit (a
share evaluates its own cells of the same staged records in the same order) and
with the same pair totals, at numbers of tiles around those where the sharing
changes (the workgroups that fit 256 compute units, their half and quarter),
ragged, closed and periodic."""
import pytest
import torch

import workloads as W
from helpers import device_traj

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("n", [(5, 3, 9), (16, 16, 16), (31, 33, 40), (64, 32, 32), (65, 32, 32), (64, 64, 32),
                               (65, 64, 32), (64, 64, 64), (66, 61, 63), (17, 5), (64, 64), (128, 256), (130, 256),
                               (256, 256), (257, 256), (512, 256), (500, 257)])
def test_shares_keep_the_bits(ctx, prec, periodic, n):
    import paper_2512_20829_amd as F
    dim = len(n)
    if dim == 3:
        wl = W.small_random_3d(9000, 20, seed=61, periodic=periodic)
    else:
        wl = W.taylor_green_2d(per_axis=75, mesh_n=64, seed=62)
    mesh = W.Mesh(dim, n, (0.0,) * dim, (1.0,) * dim, (periodic,) * dim)
    dt = torch.float64 if prec == "f64" else torch.float32
    tr, keep = device_traj(wl.traj, prec)
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff, count_pairs=True)
    print(f"[case] small {n} periodic={periodic} {prec}", flush=True)
    one = F.alloc_fields(mesh.cells, dim, dt, DEV)
    ctx.project_sources(F.mesh_of(mesh), tr, p, *one)
    torch.cuda.synchronize()
    pairs = ctx.stats()["pairs"]
    many = F.alloc_fields(mesh.cells, dim, dt, DEV)
    ctx.project_batch([F.mesh_of(mesh)], [tr], [p], [many])
    torch.cuda.synchronize()
    assert ctx.stats()["pairs"] == pairs > 0
    for a, b in zip([one[0], *one[1], one[2]], [many[0], *many[1], many[2]]):
        assert torch.equal(a, b)
