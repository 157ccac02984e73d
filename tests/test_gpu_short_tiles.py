"""Periodic axes whose last tile (or a whole run of buckets) is short: a
support that spans less than the axis can wrap past it and end in its home
tile again.  Per-cell pair counts against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import as_precision, assert_fields_close, device_traj, gpu_run, oracle_run

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(9, 9, 9), (10, 12, 15)])
def test_cartesian_3d(ctx, n, prec):
    wl = W.small_random_3d(400, 8, seed=210, periodic=True, h0=0.11, amp=0.02)
    wl.mesh = W.Mesh(3, n, (0.0,) * 3, (1.0,) * 3, (True,) * 3)
    print(f"[case] mesh={n} prec={prec}", flush=True)
    S, _, st = gpu_run(ctx, wl, prec=prec, cell_pairs=True)
    ref, _ = oracle_run(wl, prec=prec)
    np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
    assert_fields_close(S, ref.S, TOL[prec], f"mesh {n}")


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_cartesian_2d(ctx, prec):
    wl = W.taylor_green_2d(per_axis=20)
    wl.mesh = W.Mesh(2, (17, 21), (0.0,) * 2, (1.0,) * 2, (True,) * 2)
    wl.h0 = 0.1
    S, _, st = gpu_run(ctx, wl, prec=prec, cell_pairs=True)
    ref, _ = oracle_run(wl, prec=prec)
    np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
    assert_fields_close(S, ref.S, TOL[prec], "2-D")


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_general_mesh(ctx, prec):
    """Cells clustered at both ends of every axis: one bucket spans most of it."""
    import paper_2512_20829_amd as F
    cells = W.rectilinear_cells([W.stretched_edges(12, 0.0, 1.0, 3.0)] * 3, (True,) * 3)
    wl = W.small_random_3d(400, 8, seed=211, periodic=True, h0=0.11, amp=0.02)
    dev, dt = torch.device("cuda", 0), torch.float64 if prec == "f64" else torch.float32
    cs, keep = F.cells_of(cells, dev)
    ix = ctx.cell_index(cs, 64)
    print(f"[case] buckets={ix.shape()} prec={prec}", flush=True)
    tr, keep2 = device_traj(wl.traj, prec)
    S_mass, S_mom, den = F.alloc_fields(cells.count, 3, dt, dev)
    pairs = torch.full((cells.count,), -1, dtype=torch.int32, device=dev)
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff)
    ctx.project_cells(ix, tr, p, S_mass, S_mom, den, pairs=pairs)
    torch.cuda.synchronize()
    ix.close()
    ref, _ = oracle.project_points(cells, as_precision(wl.traj, prec), wl.rho_d, wl.mu, wl.delta, wl.h0,
                                   cutoff=wl.cutoff, f32_decision=(prec == "f32"))
    np.testing.assert_array_equal(pairs.cpu().numpy().astype(np.int64), ref.pairs)
    assert_fields_close(torch.stack([S_mass, *S_mom]).double().cpu().numpy(), ref.S, TOL[prec], "cells")
