"""nif_forward over the panel path's launch forms: the block-per-16-pairs and wave MLPs, chunks, the
level-by-level and LDS encodings.  Heads do not depend on the form, so a batch must give, bit for
bit, what its pieces give on other forms; one form is held to the oracle in test_gpu_network.py."""
import dataclasses

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, say

pytestmark = pytest.mark.gpu

_TORUS, _SPHERES = S.workload("torus16").model, S.workload("spheres64").model
MODELS = {
    "torus_w16": dataclasses.replace(_TORUS, hidden_width=16),
    "torus_w32_f16": dataclasses.replace(_TORUS, hidden_width=32, table_dtype=S.TABLE_F16, n_materials=8),
    "spheres_w64": _SPHERES,
    "spheres_w128_l12_per_sample": dataclasses.replace(_SPHERES, levels=12, res=S.level_resolutions(12, 16, 700), hidden_width=128,
                                                       log2_table=15, per_sample_tables=1, pe_freqs=3),
    "identity_pe": dataclasses.replace(_SPHERES, pe_freqs=0, hidden_width=128, levels=4, res=[16, 64, 200, 801]),
}


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("name", list(MODELS))
def test_forward_does_not_depend_on_the_launch_form(name, prec):
    import torch
    import paper_2604_24666_amd as P
    m = MODELS[name]
    n = 140003                                       # two or more chunks, waves of several columns
    say(f"forward launch forms: {name} prec={prec}")
    tab, prm, _ = model_params(m, 11, 1e3)
    model = P.Model(m)
    model.set_params(tab, prm)
    x0, x1 = (dev_f32(v) for v in S.random_points(n, 12))
    whole = model.forward(x0, x1, prec)
    at = 0
    for size in (1, 15, 16, 17, 241, 4099, 10241, 12345, 33001):
        part = model.forward(x0[:, at:at + size].contiguous(), x1[:, at:at + size].contiguous(), prec)
        assert torch.equal(part, whole[at:at + size]), size
        at += size
    assert bool(torch.isfinite(whole).all()) and float(whole.std()) > 0


@pytest.mark.parametrize("name", list(MODELS))
def test_encode_does_not_depend_on_the_launch_form(name):
    """Rows of nif_encode: chunks, level-by-level and LDS lookups, an output that is aligned to 4 bytes only."""
    import torch
    import paper_2604_24666_amd as P
    m = MODELS[name]
    n = 140003
    say(f"encode launch forms: {name}")
    tab, prm, _ = model_params(m, 13, 1e3)
    model = P.Model(m)
    model.set_params(tab, prm)
    x, _ = (dev_f32(v) for v in S.random_points(n, 14))
    whole = model.encode(x)
    at = 0
    for size in (1, 63, 64, 65, 300, 5003, 20011, 70001):
        part = x[:, at:at + size].contiguous()
        out = torch.full((size * whole.shape[1] + 1,), float("nan"), device="cuda")
        P.nif_encode(model.h, part, size, out[1:])
        torch.cuda.synchronize()
        assert torch.equal(out[1:].view(size, -1), whole[at:at + size]), size
        at += size
    assert bool(torch.isfinite(whole).all()) and float(whole.std()) > 0
