"""lbm_profile_step, lbm_batch_profile_step and the batch tuner on 2-D lattices:
they time the kernel that lbm_step and lbm_batch_step run, and leave the state
of ordinary steps."""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G

from .test_gpu_step2d import lattice

pytestmark = pytest.mark.gpu

CASES = [dict(n=(96 - 7 * k, 70 + 5 * k), solid=dict(center=(45.2, 14.6), radius=11.2, mu_w=0.04),
              drop=((45.0, 35.0), 9.0)) for k in range(3)]


@pytest.mark.parametrize("model", ["chemical", "pseudopotential", "phase"])
def test_lattice_profile_names_the_single_launch(model):
    # the body force of these lattices starts at step 21, inside the profile
    a, b, c = (lattice("floor", model, G.LBM_F32, G.LBM_BGK, G.LBM_BC_HALFWAY, k)
               for k in (G.LBM_STEP_AUTO, G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT))
    for x in (a, b, c):
        x.step(12)
    prof = a.profile(19)
    assert set(prof) == {"k_step2d"} and prof["k_step2d"] > 0.0
    assert "k_step2d" not in c.profile(19)
    b.step(19)
    assert np.array_equal(a.f, b.f) and np.array_equal(c.f, b.f)
    assert a.info()["step"] == b.info()["step"] == 31
    # the device counts those steps too: the measure steps that follow are the same
    sa, sb = (x.step(20, measure_every=10, cap=3) for x in (a, b))
    assert [bytes(r) for r in sa] == [bytes(r) for r in sb] and [r.step for r in sa] == [40, 50]


@pytest.mark.parametrize("model", [0, 2])
def test_batch_profile_names_the_single_launch(model):
    params = {} if model == 0 else dict(model=model, pf_A=0.01, pf_kappa=0.02)
    a, b, c = (G.Batch(CASES, precision=G.LBM_F32, Tr=0.8, g=(2e-6, -3e-6), g_start_step=21, step_kernel=k, **params)
               for k in (G.LBM_STEP_AUTO, G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT))
    for x in (a, b, c):
        x.step(12)
    prof = a.profile(19)
    assert set(prof) == {"k_step2d"} and prof["k_step2d"] > 0.0
    split = {"kb_density", "kb_mu", "kb_collide"} if model == 0 else {"kb_pf_density", "kb_pf_mu", "kb_pf_collide"}
    assert set(c.profile(19)) == split
    b.step(19)
    assert a.info()["step"] == b.info()["step"] == 31
    for i in range(len(CASES)):
        assert np.array_equal(a.read(i, G.FIELD_F), b.read(i, G.FIELD_F))
        assert np.array_equal(c.read(i, G.FIELD_F), b.read(i, G.FIELD_F))


def test_tuning_a_2d_batch_searches_no_shape_and_keeps_the_state(tmp_path):
    cache = str(tmp_path / "tune.json")
    a = G.Batch(CASES, precision=G.LBM_F32, Tr=0.8, tile_w=256, blocks_per_cu=2)
    b = G.Batch(CASES, precision=G.LBM_F32, Tr=0.8)
    for x in (a, b):
        x.step(13)
    a.tune(cache)  # from pull form, in the buffer an odd number of steps leaves
    inf = a.info()
    assert (inf["tile_w"], inf["blocks_per_cu"]) == (64, 4) and inf["tune_ms_per_step"] > 0.0 and inf["step"] == 13
    for x in (a, b):
        x.step(40, measure_every=10)
        x.sync()
    assert [bytes(r) for r in a.angles()] == [bytes(r) for r in b.angles()]
    for i in range(len(CASES)):
        assert np.array_equal(a.read(i, G.FIELD_F), b.read(i, G.FIELD_F))
    c = G.Batch(CASES, precision=G.LBM_F32, Tr=0.8, autotune=True, cache_path=cache)
    assert (c.info()["tile_w"], c.info()["blocks_per_cu"]) == (64, 4)
