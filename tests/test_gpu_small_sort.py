"""The one-launch sort of few keys and the short blocks of a middling one
against the long blocks: a call alone and as the first snapshot of a batch,
whose keys are sorted together, agree bit for bit and in their statistics, at
the numbers of keys where the sorts change over (1024, 4096 and 8192 keys, 2^18
with the second snapshot beyond it) and with few, many and very many buckets."""
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


@pytest.mark.parametrize("count,n", [(1, 12), (2, 12), (63, 12), (1023, 20), (1024, 20), (1025, 20), (4095, 40),
                                     (4096, 70), (4097, 70), (8191, 40), (8192, 80), (8192, 90), (8193, 40),
                                     (20000, 30), (1 << 18, 40), ((1 << 18) + 1, 40)])
def test_sorts_agree(ctx, count, n):
    import paper_2512_20829_amd as F
    wl = W.small_random_3d(count, 20, seed=63, periodic=True, h0=max(0.02, 0.7 * count ** (-1 / 3)) if count > 8 else 0.1)
    mesh = W.Mesh(3, (n,) * 3, (0.0,) * 3, (1.0,) * 3, (True,) * 3)
    tr, keep = device_traj(wl.traj, "f32")
    more, keep2 = device_traj(W.small_random_3d(300, 20, seed=64).traj, "f32")
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff, count_pairs=True)
    print(f"[case] sort {count} keys, {n}^3 cells", flush=True)
    outs = [F.alloc_fields(mesh.cells, 3, torch.float32, DEV) for _ in range(4)]
    stats = []
    for o, t in ((outs[0], tr), (outs[1], more)):
        ctx.project_sources(F.mesh_of(mesh), t, p, *o)
        torch.cuda.synchronize()
        stats.append(ctx.stats())
    ctx.project_batch([F.mesh_of(mesh)] * 2, [tr, more], [p] * 2, outs[2:])
    torch.cuda.synchronize()
    st = ctx.stats()
    assert st["pairs"] == stats[0]["pairs"] + stats[1]["pairs"] > 0
    assert st["max_class"] == max(s["max_class"] for s in stats)
    for one, many in zip(outs[:2], outs[2:]):
        for a, b in zip([one[0], *one[1], one[2]], [many[0], *many[1], many[2]]):
            assert torch.equal(a, b)
