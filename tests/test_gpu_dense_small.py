"""Binary32 3-D meshes of few tiles with many records each, which four workgroups
to a tile share, alone and in a batch: bit for bit what the same snapshot gives in
a batch with a mesh of a thousand tiles (one workgroup per tile), with the same
pairs in every cell, and the oracle's fields within the parity bar; just below the
number of records where the sharing begins, at it and above, with batches of
every remainder, ragged, closed, periodic and stretched."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import as_precision, assert_fields_close, device_traj, gpu_run

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
PER_TILE = 1280


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


def _tiles(n):
    return int(np.prod([(k + 7) // 8 for k in n]))


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("n, extra, h", [((5, 3, 7), 0, 1.0), ((8, 8, 8), 1, 2.5), ((20, 20, 20), -1, 1.0),
                                         ((20, 20, 20), 0, 1.0), ((20, 20, 20), 33, 4.0), ((17, 9, 30), 517, 0.5),
                                         ((40, 33, 35), 77, 1.0), ((64, 64, 40), 5, 0.8), ((72, 64, 64), 3, 0.8)])
def test_split_keeps_the_bits(ctx, n, extra, h, periodic):
    import paper_2512_20829_amd as F
    N = PER_TILE * _tiles(n) + extra
    wl = W.small_random_3d(N, 20, seed=101, periodic=periodic)
    wl.h0 *= h
    wl.mesh = W.Mesh(3, n, (0.0,) * 3, (1.0,) * 3, (periodic,) * 3)
    tr, keep = device_traj(wl.traj, "f32")
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff, count_pairs=True)
    q = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff)
    big = F.make_mesh(3, (80, 80, 80), [0.0] * 3, [1.0] * 3, [True] * 3)
    btr, bkeep = device_traj(W.small_random_3d(200, 20, seed=103).traj, "f32")
    print(f"[case] dense small {n} N={N} periodic={periodic}", flush=True)
    for edges in (None, [W.stretched_edges(k, 0.0, 1.0, 1.1).to(DEV) for k in n]):
        mesh = F.make_mesh(3, n, [0.0] * 3, [1.0] * 3, [periodic] * 3, None, edges)
        one, many, few, two = (F.alloc_fields(wl.mesh.cells, 3, torch.float32, DEV) for _ in range(4))
        cp = [torch.full((wl.mesh.cells,), -1, dtype=torch.int32, device=DEV) for _ in range(2)]
        ctx.project_sources(mesh, tr, p, *one, pairs=cp[0])
        torch.cuda.synchronize()
        pairs = ctx.stats()["pairs"]
        large = F.alloc_fields(80 ** 3, 3, torch.float32, DEV)
        ctx.project_batch([mesh, big], [tr, btr], [p, q], [many, large])
        torch.cuda.synchronize()
        total = ctx.stats()["pairs"]
        ctx.project_sources(big, btr, p, *large)
        torch.cuda.synchronize()
        assert total - ctx.stats()["pairs"] == pairs == int(cp[0].sum()) > 0
        ctx.project_batch([mesh], [tr], [p], [few])
        ctx.project_batch([mesh, mesh], [tr, tr], [q, q], [few, two])
        torch.cuda.synchronize()
        for other in (many, few, two):
            for a, b in zip([one[0], *one[1], one[2]], [other[0], *other[1], other[2]]):
                assert torch.equal(a, b)
        plain = F.alloc_fields(wl.mesh.cells, 3, torch.float32, DEV)
        ctx.project_sources(mesh, tr, q, *plain)
        torch.cuda.synchronize()
        for a, b in zip([one[0], *one[1], one[2]], [plain[0], *plain[1], plain[2]]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("mode", ["nw", "deposit"])
def test_split_matches_the_oracle(ctx, mode):
    import paper_2512_20829_amd as F
    n = (20, 18, 23)
    wl = W.small_random_3d(PER_TILE * _tiles(n) + 13, 20, seed=102)
    wl.mesh = W.Mesh(3, n, (0.0,) * 3, (1.0,) * 3, (True, False, True))
    print(f"[case] dense small against the oracle {mode}", flush=True)
    S, den, st = gpu_run(ctx, wl, prec="f32", cell_pairs=True, mode=F.FLA_DEPOSIT if mode == "deposit" else F.FLA_NW)
    tr = as_precision(wl.traj, "f32")
    ref, t = oracle.project_box(wl.mesh, tr, wl.rho_d, wl.mu, wl.delta, wl.h0, cutoff=wl.cutoff, f32_decision=True)
    if mode == "deposit":
        Sref = oracle.deposit_scatter(wl.mesh, tr.x, t, tr.seed_volume, f32_decision=True)[0]
    else:
        Sref = ref.S
        np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
    assert_fields_close(S, Sref, 1e-5, f"dense small {mode}")
