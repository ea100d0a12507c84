"""nif_query in stages (launches of many rays) against the fused kernels: blocks of 16 rays (the same rays
in pieces below the staged size) and waves of 16 (dealt pose by pose), held to the oracle in
test_gpu_query.py.  A ray's outputs depend on none of them, so all are the same, bit for bit, as are the
ray, evaluation and degenerate-test counts.  Cases: rays that go on
past their first segment, more segments than the list has room for, an occlusion bound, several poses
with an empty one."""
import dataclasses

import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, offsets, say

pytestmark = pytest.mark.gpu

_TORUS, _SPHERES = S.workload("torus16").model, S.workload("spheres64").model
MODELS = {"torus": _TORUS, "spheres": _SPHERES, "wide": dataclasses.replace(_SPHERES, hidden_width=128, n_materials=1)}


@pytest.mark.parametrize("name,prec,view,n,bound", [
    ("torus", 0, "random", 40003, False), ("spheres", 2, "inside", 70001, True), ("spheres", 0, "inside", 150001, False),
    ("wide", 1, "random", 33000, False)])
def test_staged_query_equals_the_fused_one(name, prec, view, n, bound):
    import torch
    import paper_2604_24666_amd as P
    m = MODELS[name]
    say(f"query stages: {name} prec={prec} {view} n={n} bound={bound}")
    tab, prm, _ = model_params(m, 21, 1e3)
    model = P.Model(m)
    model.set_params(tab, prm)
    w = S.workload("spheres64")
    N = 40
    occ = torch.zeros(N ** 3, dtype=torch.uint8, device="cuda")
    P.nif_voxelize(w.scene_kind, S.scene_params(w.scene_kind, w.seed), N, occ)
    if n > 100000:
        occ.fill_(1)                                 # every ray has a segment: more than the list holds
    kinds, strengths = [S.TWIST, S.BEND, S.TAPER], [1.0, 0.5, 0.75]
    grid = P.Grid(occ, N, kinds, strengths)
    o, d = (dev_f32(v) for v in (S.rays_random(n, 6) if view == "random" else S.rays_inside(n, 6, lo=0.2, hi=0.8)))
    tmax = torch.rand(n, device="cuda") * 0.5 if bound else None
    half = n // 3
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    whole = grid.query(model, o, d, offsets([half, 0, n - half]), precision=prec, tmax=tmax, stats=stats)
    whole = {k: v.clone() for k, v in whole.items()}
    sums = torch.zeros_like(stats)
    size = 16000
    for at in range(0, n, size):
        c = min(size, n - at)
        first = max(0, min(c, half - at))
        part = grid.query(model, o[:, at:at + c].contiguous(), d[:, at:at + c].contiguous(), offsets([first, 0, c - first]),
                          precision=prec, tmax=None if tmax is None else tmax[at:at + c].contiguous(), stats=sums)
        torch.cuda.synchronize()
        for k, v in part.items():
            assert torch.equal(v, whole[k][at:at + c]), (at, k)
    say(f"  counts {stats[:3].tolist()}  hits {float(whole['hit'].float().mean()):.3f}  most {int(whole['n_queried'].max())}")
    assert torch.equal(stats, sums) and int(stats[0]) == n
    waves = P.alloc_hits(n, "cuda")
    sums.zero_()
    P.nif_query(model.h, grid.h, P.make_rays(o, d, offsets([half, 0, n - half]), tmax), n, P.hits_struct(waves),
                P.Q_POSE_ORDER, prec, sums)
    torch.cuda.synchronize()
    for k, v in waves.items():
        assert torch.equal(v, whole[k]), k
    assert torch.equal(stats, sums)
    assert bool(whole["hit"].any()) and int(whole["n_queried"].max()) > 1
