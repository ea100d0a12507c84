"""nif_trace over its launch forms: 16 lanes per ray (small launches) and 8 (large ones), bins of few
and of many voxels.  A ray's segments depend on none of them, so every output must be the same, bit
for bit, in all; one form is held to the oracle in test_gpu_geometry.py."""
import pytest

import nif_synth as S
from _helpers import dev_f32, offsets, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,s,N,max_seg", [(S.TWIST, 1.0, 33, 64), (S.BEND, 0.8, 64, 3)])
def test_segments_do_not_depend_on_the_launch_form(kind, s, N, max_seg):
    import torch
    import paper_2604_24666_amd as P
    w = S.workload("blobs128")
    occ = torch.zeros(N ** 3, dtype=torch.uint8, device="cuda")
    P.nif_voxelize(w.scene_kind, S.scene_params(w.scene_kind, w.seed), N, occ)
    say(f"trace forms: kind={kind} N={N} max_seg={max_seg}")
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 33      # 8 lanes per ray
    o, d = (dev_f32(v) for v in S.rays_inside(n, 6, lo=0.1, hi=0.9))
    whole = P.Grid(occ, N, [kind], [s], bins_per_axis=N // 2).trace(o, d, offsets([n]), max_seg=max_seg)
    assert int(whole["count"].max()) > 3
    for bins, size in ((N // 2, 4097), (5, 2049)):   # 16 lanes per ray; bins of more voxels than one LDS sort holds
        grid = P.Grid(occ, N, [kind], [s], bins_per_axis=bins)
        for at in (0, size, n - size):
            part = grid.trace(o[:, at:at + size].contiguous(), d[:, at:at + size].contiguous(), offsets([size]),
                              max_seg=max_seg)
            torch.cuda.synchronize()
            for k, v in part.items():
                u = whole[k][:, at:at + size] if k in ("x0", "x1") else whole[k][at:at + size]
                assert torch.equal(v, u), (bins, at, k)
