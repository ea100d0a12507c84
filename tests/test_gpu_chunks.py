"""The backward of a batch that spans several chunks (and more than one table-gradient round)
against the same samples in calls of one chunk each, whose gradients accumulate.

Tolerance: both sides are FP32 sums of the same terms in another order; the d heads are random, so
no sum is much smaller than sqrt(terms) of one term and the rounding of the partial sums stays
below 1e-5 of each tensor's norm (sqrt(1024) 2^-24 = 2e-6 for the longest run of a partial)."""
import dataclasses

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, say

pytestmark = pytest.mark.gpu

_SMALL = dataclasses.replace(S.workload("torus16").model, levels=4, res=[16, 32, 64, 128], pe_freqs=2, hidden_width=32)
MODELS = {
    "two_features": _SMALL,
    "concat": dataclasses.replace(_SMALL, concat_encoding=1),
    "three_features": dataclasses.replace(S.workload("spheres32_paper").model, log2_table=14, hidden_width=16),
    "width64_per_sample": dataclasses.replace(_SMALL, hidden_width=64, per_sample_tables=1),
}


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("B", [(1 << 18) + 77])
def test_backward_over_chunks_equals_accumulated_calls(name, B):
    import torch
    import paper_2604_24666_amd as P
    m = MODELS[name]
    say(f"backward over chunks: {name} B={B}")
    tab, prm, _ = model_params(m, 5, 1e3)
    x0, x1 = (dev_f32(v) for v in S.random_points(B, 6))
    dh = dev_f32(np.random.default_rng(7).normal(size=(B, m.n_heads)))
    got = []
    for cuts in ([0, B], [0, 100000, 200003, B]):
        model = P.Model(m, max_batch=max(b - a for a, b in zip(cuts, cuts[1:])))
        model.set_params(tab, prm)
        dx = [[], []]
        for k, (a, b) in enumerate(zip(cuts, cuts[1:])):
            y0, y1 = x0[:, a:b].contiguous(), x1[:, a:b].contiguous()
            d0, d1 = torch.empty_like(y0), torch.empty_like(y1)
            P.nif_backward(model.h, y0, y1, b - a, dh[a:b].contiguous(), d0, d1, accumulate=k > 0)
            dx[0].append(d0)
            dx[1].append(d1)
        g = model.get_grads()
        torch.cuda.synchronize()
        got.append([g[0], g[1], torch.cat(dx[0], 1), torch.cat(dx[1], 1)])
    for what, u, v in zip(("tables", "mlp", "dx0", "dx1"), *got):
        u, v = u.double(), v.double()
        off = float((u - v).norm() / v.norm())
        say(f"  {what}: {off:.2e}")
        assert float(v.norm()) > 0 and off <= 1e-5, what
