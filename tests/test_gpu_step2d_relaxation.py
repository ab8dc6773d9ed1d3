"""The single-launch D2Q9 step at relaxation times other than one (at tau = 1
the BGK collision forgets the populations it came from, and half of its
expressions drop out): against the split step bit for bit, with both collisions
on both walls, and against the FP64 oracle."""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G

from .pairs import gpu_lattice, oracle_lattice, rel_err
from .test_gpu_step2d import LAYOUTS, MODELS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["tiny", "box", "floor", "cavity", "middle", "large"])
@pytest.mark.parametrize("model", list(MODELS))
@pytest.mark.parametrize("precision", [G.LBM_F32, G.LBM_F64, G.LBM_F32_MIXED])
@pytest.mark.parametrize("tau", [0.8, 1.3])
def test_equals_the_split_step(layout, model, precision, tau):
    n, box, solid, drop = LAYOUTS[layout]
    mu_w, width, params = MODELS[model]
    if model == "phase":
        params = dict(params, pf_tau=0.9)
    for collision in (G.LBM_MRT, G.LBM_BGK):
        for wall in (G.LBM_BC_HALFWAY, G.LBM_BC_BOUZIDI_MC):
            lats = []
            for kernel in (G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT):
                lat = G.Lattice(G.LBM_D2Q9, n=n + (1,), precision=precision, axis_bc=box + (0,), collision=collision,
                                bc_mode=wall, tau=tau, Tr=0.8, g=(2e-6, -3e-6), g_start_step=9, step_kernel=kernel,
                                **params)
                if solid:
                    lat.set_solids([dict(solid, mu_w=mu_w)])
                lat.init_drops([drop], W=width)
                series = lat.step(41, measure_every=20, cap=4) if solid else lat.step(41)
                lats.append((lat, series))
            (a, sa), (b, sb) = lats
            assert [bytes(r) for r in sa or ()] == [bytes(r) for r in sb or ()]
            assert np.isfinite(a.f).all()
            assert np.array_equal(a.f, b.f)
            if model == "phase":
                assert np.array_equal(a.g, b.g)


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("tau", [0.8, 1.3])
def test_matches_the_oracle(collision, model, tau):
    wl = dict(dim=2, n=(97, 63), wall=(0, 1), drops=[((47.5, 36.2), 9.5)], W=5.0, model=model,
              solids=[dict(center=(47.7, 12.3), radius=14.4, mu_w=1.2 if model == 1 else 0.04)])
    kw = dict(tau=tau) if model else dict(tau=tau, Tr=0.8)
    gp = gpu_lattice(wl, G.LBM_F64, collision, **kw)
    o = oracle_lattice(wl, collision, **kw)
    gp.step(30)
    o.step(30)
    assert np.isfinite(o.rho[o.cls == 0]).all()
    assert rel_err(gp.f, o.f) <= 1e-12
