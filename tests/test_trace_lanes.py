"""The lanes that share a ray in the traversal must keep together and find what one lane finds alone,
also where a lane meets more segments in a bin than it has slots for (its ray then goes over the bin's
list again): coarse bins and filled occupancies.  On the CPU the library's own traversal header runs
lane by lane (tests/lanes) against repeated one-lane steps, bit for bit, as do the lanes of a wave that takes rays; on the GPU nif_trace on grids
whose rays spill, 8 and 16 lanes a ray, must give the segments of fine bins and of the oracle."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, offsets, say

_HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("lanes") / "liblanes.so")
    src = os.path.join(_HERE, "lanes")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-Wno-unknown-pragmas", "-I" + src,
                    "-I" + os.path.join(_HERE, "..", "paper_2604_24666_amd", "csrc"), "-o", so, os.path.join(src, "lanes.cpp")],
                   check=True)
    return C.CDLL(so)


@pytest.fixture(scope="module")
def lanes(lib):
    def check(N, occ, kind, s, bins, sub, o, d):
        o, d = (np.ascontiguousarray(v, dtype=np.float32) for v in (o, d))
        n = o.shape[1]
        res, spilled = np.zeros(6, np.int64), np.zeros(n, np.uint8)
        rc = lib.lanes_check(C.c_int(N), occ.ctypes.data_as(C.c_void_p), C.c_int(kind), C.c_float(s), C.c_int(bins), C.c_int(sub),
                           C.c_int64(n), o.ctypes.data_as(C.c_void_p), d.ctypes.data_as(C.c_void_p),
                           res.ctypes.data_as(C.c_void_p), spilled.ctypes.data_as(C.c_void_p))
        assert rc == 0
        return dict(zip(("spilled", "apart", "other", "next_apart", "next_other", "segments"), res.tolist())), spilled
    return check


def _rays(n, seed):
    a, b = S.rays_random(n, seed), S.rays_inside(n, seed + 1, lo=0.1, hi=0.9)
    return np.concatenate([a[0], b[0]], 1), np.concatenate([a[1], b[1]], 1)


@pytest.mark.parametrize("sub", [2, 4, 8, 16])
@pytest.mark.parametrize("N,kind,s,bins", [(21, S.TWIST, 1.0, 1), (24, S.TAPER, 0.7, 2), (33, S.IDENTITY, 0.0, 4),
                                           (16, S.BEND, 1.0, 0), (24, S.TWIST_BEND, 1.0, 5)])
def test_lanes_of_a_ray_keep_together_on_filled_grids(lanes, N, kind, s, bins, sub):
    occ = np.ones(N ** 3, np.uint8)
    got, _ = lanes(N, occ, kind, s, bins, sub, *_rays(40, 3))
    say(f"lanes {sub}, N={N} kind={kind} bins={bins}: {got}")
    assert got["segments"] > 0 and (got["spilled"] > 0 or bins not in (1, 2))
    assert not (got["apart"] or got["other"] or got["next_apart"] or got["next_other"])


@pytest.mark.parametrize("sub", [8, 16])
@pytest.mark.parametrize("bins", [1, 4])
def test_lanes_of_a_ray_keep_together_on_a_surface(lanes, orc, bins, sub):
    w = S.workload("torus16")
    N = 40
    occ = orc.voxelize(w.scene_kind, S.scene_params(w.scene_kind, w.seed), N)
    got, _ = lanes(N, occ, S.TWIST, 1.0, bins, sub, *_rays(400, 5))
    say(f"lanes {sub}, torus surface bins={bins}: {got}")
    assert got["segments"] > 0
    assert not (got["apart"] or got["other"] or got["next_apart"] or got["next_other"])


@pytest.mark.parametrize("look", [0, 1])
def test_lanes_of_a_wave_take_the_same_tickets(lib, look):
    """The counter moves past the end of the range while the wave takes its rays: all lanes must hold the
    same tickets (some would else leave out or repeat rays), and none is taken twice."""
    lib.lanes_take.restype = C.c_int64
    for size in (0, 1, 40, 1000):
        for at in sorted({0, max(0, size - 70), max(0, size - 1), size, size + 5}):
            for n in (1, 4, 64):
                for leader in (0, 4, 63):
                    for others in (0, 1, 3, 64):
                        base = lib.lanes_take(C.c_int64(at), C.c_int64(size), n, leader, look, C.c_int64(others))
                        assert base >= min(at, size), (size, at, n, leader, others, base)


@pytest.mark.gpu
@pytest.mark.parametrize("N,kind,s,coarse", [(24, S.TWIST, 1.0, (1, 2)), (20, S.BEND, 1.0, (1,))])
def test_trace_of_spilling_rays(lanes, orc, N, kind, s, coarse):
    import torch
    import paper_2604_24666_amd as P
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 33      # 8 lanes per ray
    few, looked = 2001, 150                                                      # 16 lanes; rays emulated on the host
    o, d = S.rays_inside(n, 6, lo=0.1, hi=0.9)
    occ = np.ones(N ** 3, np.uint8)
    max_seg = 4 * N
    fine = P.Grid(torch.as_tensor(occ).cuda(), N, [kind], [s], bins_per_axis=2 * N).trace(
        dev_f32(o), dev_f32(d), offsets([n]), max_seg=max_seg)
    torch.cuda.synchronize()
    for bins in coarse:
        for m, sub in ((n, 8), (few, 16)):
            got, _ = lanes(N, occ, kind, s, bins, sub, o[:, :looked], d[:, :looked])
            say(f"trace of spilling rays: N={N} kind={kind} bins={bins} lanes={sub}: {got['spilled']} of {looked} spill")
            assert got["spilled"] > 0
            grid = P.Grid(torch.as_tensor(occ).cuda(), N, [kind], [s], bins_per_axis=bins)
            out = grid.trace(dev_f32(o[:, :m]), dev_f32(d[:, :m]), offsets([m]), max_seg=max_seg)
            torch.cuda.synchronize()
            for k, v in out.items():
                assert torch.equal(v, fine[k][:, :m] if k in ("x0", "x1") else fine[k][:m]), (bins, sub, k)
    V = orc.lattice_vertices(kind, float(np.float32(s)), N)
    m = 500
    rc, _, _, rcnt, fl = orc.trace(N, occ, V, o[:, :m], d[:, :m], brute=False, max_out=max_seg)
    cnt, cell = fine["count"].cpu().numpy(), fine["cell"].cpu().numpy()
    ok = fl == 0
    assert ok.sum() > m // 2 and np.array_equal(cnt[:m][ok], rcnt[ok])
    for r in np.nonzero(ok)[0]:
        assert np.array_equal(cell[r, :rcnt[r]], rc[r, :rcnt[r]]), r
