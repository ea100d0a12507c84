"""nif_forward of small networks: few pairs go through the fused kernel, more through panels.  Heads depend
on neither, so the pieces of a batch on both sides of each line equal the batch, bit for bit; a
fused piece is also held to the oracle (bar of test_gpu_network.py)."""
import dataclasses

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, say
from test_gpu_network import _fp32_close

pytestmark = pytest.mark.gpu

_BASE = S.workload("spheres64").model


def _model(**kw):
    L = kw["levels"]
    return dataclasses.replace(_BASE, hidden_layers=2, res=S.level_resolutions(L, 16, 512), **kw)


MODELS = {       # batches of the first layer x width: fused up to 2^16 pairs, up to 2^14, up to 2^16
    "l8_no_pe_w64": _model(levels=8, pe_freqs=0, hidden_width=64, log2_table=14, table_dtype=S.TABLE_F32),
    "l4_f3_w32": _model(levels=4, pe_freqs=3, hidden_width=32, log2_table=16),
    "l4_f1_w16_per_sample": _model(levels=4, pe_freqs=1, hidden_width=16, log2_table=14, per_sample_tables=1),
}


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("name", list(MODELS))
def test_forward_on_both_sides_of_the_line(orc, name, prec):
    import torch
    import paper_2604_24666_amd as P
    m = MODELS[name]
    n = 120003                                       # panels, in chunks of more pairs than the lines
    say(f"forward of a small network: {name} prec={prec}")
    tab, prm, seen = model_params(m, 11, 1e3)
    model = P.Model(m)
    model.set_params(tab, prm)
    pts = S.random_points(n, 12)
    x0, x1 = (dev_f32(v) for v in pts)
    whole = torch.empty((n, m.n_heads), device="cuda")
    at = 0
    for size in (1, 15, 17, 64, 65, 4097, 1 << 14, (1 << 14) + 1, 65536):
        part = model.forward(x0[:, at:at + size].contiguous(), x1[:, at:at + size].contiguous(), prec)
        whole[at:at + size] = part
        at += size
    assert at <= n
    assert torch.equal(model.forward(x0, x1, prec)[:at], whole[:at])
    assert bool(torch.isfinite(whole[:at]).all()) and float(whole[:at].std()) > 0
    if prec == 0:
        p0, p1 = (v[:, :162] for v in pts)           # the first five pieces
        ref = orc.forward(m, seen, prm.astype(np.float64), p0.T.astype(np.float64), p1.T.astype(np.float64))
        _fp32_close(orc, m, seen, prm, p0, p1, whole[:162].cpu().numpy().astype(np.float64), ref,
                    np.sqrt(np.mean(ref ** 2, axis=0, keepdims=True)), "fused")
