"""The sign steps that nif_label passes over, against the FP64 oracle, which evaluates every step:
chords from a voxel to across the scene (several surfaces, grazing ones, hits in the last step), narrow
and wide blobs, scenes beyond the kernel-argument size.  Both decide in FP64 by the same steps, so hit
and material must match exactly; t (FP32, up to 2), normal and albedo within 1e-6 as the FP32 outputs'
rounding and the 1e-13 root demand."""
import numpy as np
import pytest

import nif_synth as S
from _helpers import dev_f32, say

pytestmark = pytest.mark.gpu


def _blobs(n, sigma, seed):
    rng = np.random.default_rng(seed)
    rows = np.zeros((n, 8))
    rows[:, :3] = rng.uniform(0.1, 0.9, (n, 3))
    rows[:, 3] = sigma * rng.uniform(0.5, 2.0, n)
    rows[:, 4:7] = rng.uniform(0.0, 1.0, (n, 3))
    rows[:, 7] = np.arange(n) % 4
    return np.concatenate([[float(n)], rows.reshape(-1)])


def _scene(name):
    if name in ("torus16", "spheres64", "blobs128"):
        w = S.workload(name)
        return w.scene_kind, np.asarray(S.scene_params(w.scene_kind, w.seed), dtype=np.float64)
    n, sigma = {"narrow": (20, 0.01), "wide": (3, 0.3), "one": (1, 0.1), "many": (60, 0.04)}[name]
    return S.workload("blobs128").scene_kind, _blobs(n, sigma, 5)


@pytest.mark.parametrize("name", ["torus16", "spheres64", "blobs128", "narrow", "wide", "one", "many"])
@pytest.mark.parametrize("reach", [0.01, 0.3, 2.0])
def test_marched_labels_match_oracle(orc, name, reach):
    import torch
    import paper_2604_24666_amd as P
    kind, sp = _scene(name)
    rng = np.random.default_rng(41)
    n = 3001
    x0 = rng.uniform(-0.2, 1.2, (n, 3))
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x0, x1 = x0.astype(np.float32), (x0 + reach * rng.uniform(0.0, 1.0, (n, 1)) * u).astype(np.float32)
    say(f"marched labels: {name} reach {reach}")
    got = P.label(kind, sp, dev_f32(x0.T), dev_f32(x1.T), force_march=True)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in got.items()}
    hit, t, nr, al, mt = orc.label(kind, sp, x0.astype(np.float64), x1.astype(np.float64), force_march=True)
    h = hit == 1
    say(f"  hits {int(h.sum())}, after the start {int((t > 0).sum())}")
    assert np.array_equal(g["hit"], hit)
    assert np.array_equal(g["material"][h], mt[h])
    assert np.abs(g["t"] - t).max() <= 1e-6
    assert np.abs(g["normal"].T - nr).max() <= 1e-6 and np.abs(g["albedo"].T - al).max() <= 1e-6
