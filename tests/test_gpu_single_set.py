"""Table sets per sample where a point has one sample (no positional encoding, or the concatenated form):
both points of a pair then read one set, whose additions meet in the fill's batches.  Gradients against
the oracle, bar as in test_gpu_train.py (1e-4 norm-wise and element-wise), at table sizes of one, few and
many buckets; every table size takes records here, as no model with sets per sample is summed in LDS."""
import dataclasses

import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, say
from test_gpu_train import _batch, _grad_close

pytestmark = pytest.mark.gpu

_BASE = dataclasses.replace(S.workload("torus16").model, hidden_width=32, per_sample_tables=1)


@pytest.mark.parametrize("log2_table", [11, 14, 19])
@pytest.mark.parametrize("form", [dict(pe_freqs=0), dict(concat_encoding=1)], ids=["no_pe", "concat"])
def test_backward_with_one_table_set_matches_oracle(orc, form, log2_table):
    import torch
    import paper_2604_24666_amd as P
    m = dataclasses.replace(_BASE, log2_table=log2_table, **form)
    say(f"backward, one table set per sample: {form} log2_table={log2_table}")
    tab, prm, seen = model_params(m, 15, scale_tables=300.0)
    B = 1500 + 37
    x0, x1, hit, t, nr, al, mt = _batch(m, B, 16)
    s = np.array([0.2, -0.1, 0.3, 0.1, -0.2])
    _, gt, gp, _, gx0, gx1, dz = orc.loss_grad(m, seen, prm.astype(np.float64), s, x0.T, x1.T, hit, t, nr.T, al.T, mt,
                                               want_x=True, want_dz=True)
    model = P.Model(m, max_batch=B)
    model.set_params(tab, prm, s.astype(np.float32))
    dx0, dx1 = torch.empty((3, B), device="cuda"), torch.empty((3, B), device="cuda")
    P.nif_backward(model.h, dev_f32(x0), dev_f32(x1), B, dev_f32(dz), dx0, dx1, False, P.PREC_FP32)
    g_t, g_p, _ = model.get_grads()
    torch.cuda.synchronize()
    _grad_close(g_t.cpu().numpy(), gt, "tables")
    _grad_close(g_p.cpu().numpy(), gp, "mlp")
    _grad_close(dx0.cpu().numpy().T, gx0, "d x0")
    _grad_close(dx1.cpu().numpy().T, gx1, "d x1")
