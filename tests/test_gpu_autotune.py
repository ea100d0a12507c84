"""The launch-shape autotuner must compare launches that differ.  Batches that nif_query evaluates in
stages leave the fused kernel a remainder in one fixed form, so timing nif_query there would choose the
rays per wave by noise, process-wide; and where every number of workgroups makes the same launch, the
one that was set must stay."""
import pytest

import nif_synth as S
from _helpers import dev_f32, model_params, offsets, say

pytestmark = pytest.mark.gpu


@pytest.fixture
def setup():
    import torch
    import paper_2604_24666_amd as P
    w = S.workload("torus16")
    occ = torch.zeros(w.N ** 3, dtype=torch.uint8, device="cuda")
    P.nif_voxelize(w.scene_kind, S.scene_params(w.scene_kind, w.seed), w.N, occ)
    tab, prm, _ = model_params(w.model, w.seed + 100, scale_tables=1e3)
    model = P.Model(w.model)
    model.set_params(tab, prm)
    grid = P.Grid(occ, w.N, [S.TWIST], [1.0])

    def tune(n):
        keep = (dev_f32(S.rays_random(n, 3)[0]), dev_f32(S.rays_random(n, 3)[1]), offsets([n]))
        out = P.alloc_hits(n, "cuda")
        return P.nif_autotune_query(model.h, grid.h, P.make_rays(*keep), n, P.hits_struct(out), 0, 5)
    yield P, tune
    P.nif_set_query_blocks_per_cu(12)
    P.nif_set_query_rays_per_wave(0)


def test_rays_per_wave_of_a_staged_batch_is_a_measured_choice(setup):
    """20,001 rays fill a third of the SIMDs in 64-ray waves and all of them in 16-ray waves, which
    are far ahead: every run of the tuner must find them."""
    P, tune = setup
    found = [tune(20001) for _ in range(5)]
    say(f"autotuned, staged batch: {found}")
    assert all(rpw == 16 for _, rpw, _ in found)


@pytest.mark.parametrize("bpc", [6, 20])
def test_workgroups_stay_where_they_make_no_difference(setup, bpc):
    P, tune = setup
    P.nif_set_query_blocks_per_cu(bpc)
    found = [tune(3000) for _ in range(2)]
    say(f"autotuned, small batch: {found}")
    assert all(b == bpc for b, _, _ in found)
