"""The tuner on a mesh whose parts all have a workgroup at once: projections there
take a launch that no plan code changes, so fla_autotune times the launch that
the codes differ in, each distinct kernel once, and what it keeps for larger
meshes is a measured choice."""
import os
import re

import numpy as np
import pytest
import torch

import workloads as W
from helpers import device_traj

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
SAME = {("f32", 3): [0, 0, 2, 3, 0, 0, 2, 3], ("f64", 3): [0, 1, 2, 2, 4, 5, 6, 7],
        ("f32", 2): [0, 1, 1, 1], ("f64", 2): [0, 1, 1, 1]}


def _traced():
    import paper_2512_20829_amd as F
    os.environ["FLA_TRACE"] = "1"
    try:
        return F.Context(0)
    finally:
        os.environ["FLA_TRACE"] = "0"


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_tuner_times_the_kernels_that_the_codes_name(capfd, prec, dim):
    import paper_2512_20829_amd as F
    wl = W.small_random_3d(3000, 20, seed=81) if dim == 3 else W.taylor_green_2d(per_axis=40, mesh_n=50, seed=82)
    tr, keep = device_traj(wl.traj, prec)
    dt = torch.float64 if prec == "f64" else torch.float32
    out = F.alloc_fields(wl.mesh.cells, dim, dt, DEV)
    p = F.Params(rho_d=wl.rho_d, mu=wl.mu, delta=wl.delta, h0=wl.h0, cutoff=wl.cutoff)
    same, pr = SAME[prec, dim], F.FLA_F64 if prec == "f64" else F.FLA_F32
    print(f"[case] tuner on a small mesh {dim}-D {prec}", flush=True)
    ctx = _traced()
    try:
        capfd.readouterr()
        times = ctx.autotune(F.mesh_of(wl.mesh), tr, p, *out)
        tuned = capfd.readouterr().err
        ctx.project_sources(F.mesh_of(wl.mesh), tr, p, *out)
        torch.cuda.synchronize()
        plain = capfd.readouterr().err
        assert ctx.get_plan(dim, pr) == int(np.argmin(times[: len(same)]))
        batch = ctx.autotune_batch([F.mesh_of(wl.mesh)], [tr], [p], [out])
        torch.cuda.synchronize()
        batched = capfd.readouterr().err
    finally:
        ctx.close()
        F.Context(0).close()          # the log is per process: off again
    count = lambda log, k: len(re.findall(r"launch [(]*" + k + r"\b", log))
    distinct = len(set(same))
    assert count(tuned, "k_gather_small") == 0 and count(tuned, "k_gather") == 2 * distinct
    assert count(plain, "k_gather_small") == 1 and count(plain, "k_gather") == 0
    assert count(batched, "k_gather_batch") == 2 * distinct * F.BATCH_CHUNKS
    for code, first in enumerate(same):
        assert times[code] == times[first] > 0
        for c in range(F.BATCH_CHUNKS):
            assert batch[code * F.BATCH_CHUNKS + c] == batch[first * F.BATCH_CHUNKS + c] > 0
    assert all(t == -1 for t in times[len(same):])
