"""nif_backward with one of the two points' gradients asked for: it is the one that a call for both
writes, and the other points' buffer is not needed.  Tolerance 1e-6 of the largest: with three features
the levels' parts are added by FP32 atomics in any order, at most 16 of them."""
import dataclasses

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, say

pytestmark = pytest.mark.gpu

_TORUS = dataclasses.replace(S.workload("torus16").model, hidden_width=32)
MODELS = {"two_features": _TORUS, "concat": dataclasses.replace(_TORUS, concat_encoding=1),
          "three_features": dataclasses.replace(S.workload("spheres32_paper").model, log2_table=14, hidden_width=16)}


@pytest.mark.parametrize("name", list(MODELS))
def test_either_points_gradient_alone(name):
    import torch
    import paper_2604_24666_amd as P
    m, B = MODELS[name], 3001
    say(f"backward, one point's gradient: {name}")
    tab, prm, _ = model_params(m, 5, 1e3)
    model = P.Model(m, max_batch=B)
    model.set_params(tab, prm)
    x0, x1 = (dev_f32(v) for v in S.random_points(B, 6))
    dh = dev_f32(np.random.default_rng(7).normal(size=(B, m.n_heads)))

    def backward(want):
        dx = [torch.full((3, B), float("nan"), device="cuda") if w else None for w in want]
        P.nif_backward(model.h, x0, x1, B, dh, *dx)
        torch.cuda.synchronize()
        return dx
    both = backward((True, True))
    for k in (0, 1):
        one = backward((k == 0, k == 1))[k]
        assert float(both[k].abs().max()) > 0
        assert float((one - both[k]).abs().max()) <= 1e-6 * float(both[k].abs().max()), k
