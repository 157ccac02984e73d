"""Trajectories whose weights q/h are beyond the range of the call's precision (a
tiny |det J|, or an enormous number density): cells that do not include them
keep the values they have without them, on general and on Cartesian meshes.

Bars: those of the parity tests (binary64 1e-12, binary32 1e-5 of the largest
magnitude of a field) against the oracle; pair counts exact."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import as_precision, device_traj, gpu_run

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
TOL = {"f64": 1e-12, "f32": 1e-5}
KINDS = ["cells2", "cells3", "mesh2", "mesh3", "mesh3 deposit"]


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


def _workload(kind):
    dim = 2 if "2" in kind else 3
    if dim == 2:
        wl = W.taylor_green_2d(per_axis=40, mesh_n=37, seed=71)
    else:
        wl = W.small_random_3d(3000, 22, seed=72)
    cells = W.scattered_cells(dim, 15 if dim == 3 else 40, (0.0,) * dim, (1.0,) * dim, (dim == 3,) * dim, seed=73)
    return wl, cells


def _project(ctx, kind, wl, cells, tr, prec):
    """Fields (C, M), pair counts (M) or None."""
    import paper_2512_20829_amd as F
    if "cells" not in kind:
        S, _, st = gpu_run(ctx, wl, prec=prec, traj=tr, cell_pairs=True,
                           mode=F.FLA_DEPOSIT if "deposit" in kind else F.FLA_NW)
        return S, st["cell_pairs"]
    dt = torch.float64 if prec == "f64" else torch.float32
    cs, keep = F.cells_of(cells, DEV)
    ix = ctx.cell_index(cs)
    t, keep2 = device_traj(tr, prec)
    mass, mom, den = F.alloc_fields(cells.count, cells.dim, dt, DEV)
    pairs = torch.full((cells.count,), -1, dtype=torch.int32, device=DEV)
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff, count_pairs=True)
    ctx.project_cells(ix, t, p, mass, mom, den, pairs=pairs)
    torch.cuda.synchronize()
    ix.close()
    return torch.stack([mass, *mom]).double().cpu().numpy(), pairs.cpu().numpy().astype(np.int64)


def _reference(kind, wl, cells, tr, prec):
    tr = as_precision(tr, prec)
    args = (wl.rho_d, wl.mu, wl.delta, wl.h0)
    if "deposit" in kind:
        t = oracle.trajectory_terms(tr, *args)
        return oracle.deposit(wl.mesh, tr.x, t, tr.seed_volume, f32_decision=prec == "f32")[0], None
    if "cells" in kind:
        ref, _ = oracle.project_points(cells, tr, *args, cutoff=wl.cutoff, f32_decision=prec == "f32")
    else:
        ref, _ = oracle.project(wl.mesh, tr, *args, cutoff=wl.cutoff, f32_decision=prec == "f32")
    return ref.S, ref.pairs


def _close(S, ref, at, tol, what):
    for k in range(ref.shape[0]):
        off = np.abs(S[k][at] - ref[k][at])
        assert np.all(np.isfinite(S[k][at])), f"{what} field {k}: {np.sum(~np.isfinite(S[k][at]))} cells are not finite"
        worst = float(off.max()) / float(np.abs(ref[k][at]).max())
        print(f"[case] {what} field {k}: {worst:.2e} of the largest", flush=True)
        assert worst <= tol


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("kind", [k for k in KINDS if "deposit" not in k])
def test_a_record_that_reaches_no_centre_changes_nothing(ctx, kind, prec):
    wl, cells = _workload(kind)
    tr = wl.traj
    some = torch.arange(5, tr.count, 37)
    J = tr.J.clone()
    J[:, some] = 0.0
    for a in range(tr.dim):
        J[a * (tr.dim + 1), some] = 1e-20 if a == 0 else 1.0
    n0 = torch.full((tr.count,), 1e10, dtype=torch.float64)
    if prec == "f64":
        n0[some] = 1e288
    tr = W.Trajectories(tr.x, J, tr.v, tr.ug, tr.r, n0, tr.seed_volume)
    print(f"[case] weight overflow, no reach: {kind} {prec}", flush=True)
    S, pairs = _project(ctx, kind, wl, cells, tr, prec)
    ref, refpairs = _reference(kind, wl, cells, tr, prec)
    _close(S, ref, np.ones(ref.shape[1], bool), TOL[prec], f"no reach {kind} {prec}")
    np.testing.assert_array_equal(pairs, refpairs)


@pytest.mark.parametrize("kind", KINDS)
def test_only_the_cells_that_include_it_see_an_overflow(ctx, kind):
    prec = "f32"
    wl, cells = _workload(kind)
    tr = wl.traj
    one = 17
    n0 = torch.full((tr.count,), 1e10, dtype=torch.float64)
    n0[one] = 1e60
    full = W.Trajectories(tr.x, tr.J, tr.v, tr.ug, tr.r, n0, tr.seed_volume)
    rest = W.Trajectories(tr.x, tr.J, tr.v, tr.ug, tr.r, 1e10, tr.seed_volume).subset(
        torch.tensor([i for i in range(tr.count) if i != one]))
    alone = W.Trajectories(tr.x, tr.J, tr.v, tr.ug, tr.r, 1e10, tr.seed_volume).subset(torch.tensor([one]))
    print(f"[case] weight overflow, some reach: {kind} {prec}", flush=True)
    S, pairs = _project(ctx, kind, wl, cells, full, prec)
    if "cells" in kind:
        seen = oracle.project_points(cells, as_precision(alone, prec), wl.rho_d, wl.mu, wl.delta, wl.h0,
                                     cutoff=wl.cutoff, f32_decision=True)[0].pairs > 0
    else:
        seen = oracle.project(wl.mesh, as_precision(alone, prec), wl.rho_d, wl.mu, wl.delta, wl.h0, cutoff=wl.cutoff,
                              f32_decision=True)[0].pairs > 0
    assert 0 < seen.sum() < seen.size
    ref, refpairs = _reference(kind, wl, cells, rest, prec)
    _close(S, ref, ~seen, TOL[prec], f"some reach {kind} {prec}")
    assert not np.any(np.isfinite(S[0][seen]))
    if refpairs is not None:
        np.testing.assert_array_equal(pairs, refpairs + seen)
