"""2-D binary64 meshes with few records to a tile, which are gathered in whole tiles,
and with more, in halves: the oracle's pairs in every cell and its fields within
1e-12 on both sides of the number of records where that changes, ragged, closed
and periodic, and the same bits from the batched entry point, whose rule looks at
the whole batch."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import assert_fields_close, device_traj, gpu_run

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
PER_TILE = 128


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("n, records", [((270, 275), 40), ((270, 275), -1), ((270, 275), 0), ((16, 16), -1),
                                        ((9, 33), -2), ((530, 261), 1500)])
def test_whole_and_half_tiles(ctx, n, records, periodic):
    import paper_2512_20829_amd as F
    tiles = int(np.prod([(k + 15) // 16 for k in n]))
    N = records if records > 0 else PER_TILE * tiles + records
    x0 = W.random_points(2, N, 111)
    xp, J, v, ug = W.from_map(x0, "tg", {"amp": 0.1})
    tr = W.Trajectories(xp, J, v, ug, W.radius_uniform(N, 112, 5.0, 20.0), 1e10, 1.0 / N)
    wl = W.Workload("tg", W.Mesh(2, n, (0.0,) * 2, (1.0,) * 2, (periodic,) * 2), tr, N ** -0.5, "f64")
    print(f"[case] 2-D f64 {n} N={N} periodic={periodic}", flush=True)
    S, den, st = gpu_run(ctx, wl, prec="f64", cell_pairs=True)
    ref, _ = oracle.project_box(wl.mesh, tr, wl.rho_d, wl.mu, wl.delta, wl.h0, cutoff=wl.cutoff)
    np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
    assert_fields_close(S, ref.S, 1e-12, f"2-D f64 {n}")
    # beside a snapshot of 20000 records on one tile, and one of 300^2 cells with 50
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff)
    dev, keep = device_traj(tr, "f64")
    for m, k in ((16, 20000), (300, 50)):
        y, K, w, ue = W.from_map(W.random_points(2, k, 113), "tg", {"amp": 0.05})
        other, keep2 = device_traj(W.Trajectories(y, K, w, ue, W.radius_uniform(k, 114, 5.0, 20.0), 1e10, 1.0 / k), "f64")
        mesh = F.make_mesh(2, (m, m), [0.0] * 2, [1.0] * 2, [False] * 2)
        out, rest = F.alloc_fields(wl.mesh.cells, 2, torch.float64, DEV), F.alloc_fields(m * m, 2, torch.float64, DEV)
        q = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=k ** -0.5, cutoff=wl.cutoff)
        ctx.project_batch([F.mesh_of(wl.mesh), mesh], [dev, other], [p, q], [out, rest])
        torch.cuda.synchronize()
        assert np.array_equal(torch.stack([out[0], *out[1]]).cpu().numpy(), S)
        assert np.array_equal(out[2].cpu().numpy(), den)
