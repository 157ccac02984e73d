"""Every gather plan code on meshes above the size that one launch of all parts
takes (where the codes are different kernels), against the oracle: included pairs
of every cell exact, fields within the parity bars (binary64 1e-12, binary32
1e-5); and the same bits under every code of one shape."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import as_precision, assert_fields_close, device_traj, gpu_run

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


def _workload(n):
    """729 tiles in 3-D, 1496 in 2-D: binary32 puts 512 and 1024 workgroups on 256
    compute units at once, binary64 fewer."""
    dim = len(n)
    wl = W.small_random_3d(5000, 20, seed=91) if dim == 3 else W.taylor_green_2d(per_axis=70, mesh_n=64, seed=92)
    wl.mesh = W.Mesh(dim, n, (0.0,) * dim, (1.0,) * dim, (dim == 3,) * dim)
    return wl


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(70, 66, 68), (700, 530)])
def test_every_code_matches_the_oracle(ctx, prec, n):
    import paper_2512_20829_amd as F
    wl, dim = _workload(n), len(n)
    pr = F.FLA_F64 if prec == "f64" else F.FLA_F32
    ref, _ = oracle.project_box(wl.mesh, as_precision(wl.traj, prec), wl.rho_d, wl.mu, wl.delta, wl.h0,
                                cutoff=wl.cutoff, f32_decision=prec == "f32")
    base = {}
    for code in range(F.GATHER_CONFIGS if dim == 3 else F.GATHER_PLANS):
        print(f"[case] plan code {code} {n} {prec}", flush=True)
        ctx.set_plan(dim, pr, code)
        try:
            S, den, st = gpu_run(ctx, wl, prec=prec, cell_pairs=True)
            plain, pden, _ = gpu_run(ctx, wl, prec=prec, count_pairs=False)
        finally:
            ctx.set_plan(dim, pr, -1)
        np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
        assert st["pairs"] == int(ref.pairs.sum())
        assert_fields_close(S, ref.S, TOL[prec], f"plan code {code} {n} {prec}")
        S0, den0 = base.setdefault(code // F.GATHER_PLANS, (S, den))
        for a, b in ((S, S0), (den, den0), (plain, S0), (pden, den0)):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(70, 66, 68), (700, 530)])
def test_batch_keeps_the_bits(ctx, prec, n):
    import paper_2512_20829_amd as F
    wl, dim = _workload(n), len(n)
    dt = torch.float64 if prec == "f64" else torch.float32
    tr, keep = device_traj(wl.traj, prec)
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff, count_pairs=True)
    print(f"[case] batch of one {n} {prec}", flush=True)
    one, many = (F.alloc_fields(wl.mesh.cells, dim, dt, DEV) for _ in range(2))
    ctx.project_sources(F.mesh_of(wl.mesh), tr, p, *one)
    torch.cuda.synchronize()
    pairs = ctx.stats()["pairs"]
    ctx.project_batch([F.mesh_of(wl.mesh)], [tr], [p], [many])
    torch.cuda.synchronize()
    assert ctx.stats()["pairs"] == pairs > 0
    for a, b in zip([one[0], *one[1], one[2]], [many[0], *many[1], many[2]]):
        assert torch.equal(a, b)
