"""The binary32 3-D gather at the edges of its tiles, batches and thresholds:
meshes around one tile of 8^3 cells, record counts around its batches of 32
and groups of two, and cutoffs from a hair above zero to supports that span
the box, against the oracle (fields within the binary32 bar of 1e-5, the
included pairs of every cell exactly)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import as_precision, assert_fields_close, gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2512_20829_amd as F
    c = F.Context(0)
    yield c
    c.close()


def _case(n_traj, mesh, periodic, h0, cutoff, seed):
    wl = W.small_random_3d(n_traj, 8, seed=seed, periodic=periodic, h0=h0)
    wl.mesh = W.Mesh(3, mesh, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (periodic,) * 3)
    wl.cutoff = cutoff
    return wl


@pytest.mark.parametrize("mesh", [(1, 1, 1), (7, 8, 9), (8, 8, 8), (17, 5, 16)])
@pytest.mark.parametrize("n_traj", [1, 2, 31, 33, 129])
def test_tiles_and_batches(ctx, mesh, n_traj):
    for periodic in (True, False):
        print(f"[case] mesh={mesh} N={n_traj} periodic={periodic}", flush=True)
        wl = _case(n_traj, mesh, periodic, 0.15, 4.0, 200 + n_traj)
        S, den, st = gpu_run(ctx, wl, prec="f32", cell_pairs=True)
        ref, _ = oracle_run(wl, prec="f32")
        np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
        assert st["pairs"] == int(ref.pairs.sum())
        assert_fields_close(S, ref.S, 1e-5, "planes")
        assert rel_l2(den, ref.den) <= 1e-5


@pytest.mark.parametrize("cutoff", [1e-3, 0.3, 1.0, np.sqrt(3.0), 7.7, 30.0, 999.0])
def test_cutoffs(ctx, cutoff):
    """Squares of the cutoff of either parity in binary32, far below and far
    above the usual 16 (the largest cutoff is below 1000)."""
    wl = _case(700, (19, 16, 11), True, 0.06, float(cutoff), 300)
    print(f"[case] cutoff={cutoff}", flush=True)
    S, den, st = gpu_run(ctx, wl, prec="f32", cell_pairs=True)
    ref, _ = oracle_run(wl, prec="f32")
    np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
    if int(ref.pairs.sum()):
        # the weights of a cell that only far records reach are subnormal
        near = ref.den > 1e-20 * ref.den.max()
        assert_fields_close(np.where(near, S, 0.0), np.where(near, ref.S, 0.0), 1e-5, "cutoff")
        assert rel_l2(den, ref.den) <= 1e-5


def test_ties_at_the_cutoff(ctx):
    """Trajectories on cell centres with undistorted supports: s is a sum of
    squares of whole numbers, many of them exactly the squared cutoff."""
    n = 24
    wl = W.abc_lattice_3d(per_axis=n, mesh_n=n, amp=0.0)
    for cutoff in (3.0, 4.0, 5.0):
        wl.cutoff = cutoff
        S, den, st = gpu_run(ctx, wl, prec="f32", cell_pairs=True)
        ref, _ = oracle_run(wl, prec="f32")
        np.testing.assert_array_equal(st["cell_pairs"], ref.pairs)
        assert_fields_close(S, ref.S, 1e-5, f"ties at {cutoff}")


def test_deposit_over_whole_axes_and_lone_cells(ctx):
    """Deposition with supports that reach no centre (the whole amount goes to
    the home cell) beside supports that span the box."""
    wl = _case(400, (13, 9, 20), True, 0.05, 4.0, 310)
    hf = torch.ones(400, dtype=torch.float32)
    hf[::3] = 1e-4
    hf[1::7] = 6.0
    S, _, st = gpu_run(ctx, wl, prec="f32", mode=1, h_factor=hf)
    assert st["zero_support"] > 0
    tr = as_precision(wl.traj, "f32")
    _, terms = oracle.project(wl.mesh, tr, wl.rho_d, wl.mu, wl.delta, wl.h0, f32_decision=True,
                              h_factor=hf.double().numpy())
    S_ref, _ = oracle.deposit(wl.mesh, tr.x, terms, tr.seed_volume, f32_decision=True)
    assert_fields_close(S, S_ref, 1e-5, "deposit")
