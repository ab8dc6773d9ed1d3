"""The single-launch D2Q9 step against the split step (LBM_STEP_SPLIT): both
evaluate the same expressions node by node, so populations, fields and angles
agree bit for bit.  The sizes sit at the edges of the tiles (16 x 16, 32 x 16
and 64 x 16 nodes): smaller than one tile and its halo, one node over or under
a tile, and large enough for the wider shapes."""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G
from paper_2202_06516_amd import workloads as W
from tests.pairs import SC_PARAMS

pytestmark = pytest.mark.gpu

MODELS = {"chemical": (0.04, 10.0, {}), "pseudopotential": (0.8, 5.0, dict(SC_PARAMS, model=1)),
          "phase": (0.3, W.PF_W, dict(W.PF_PARAMS, model=2))}
# nodes, outer walls, solid (None: no solid), drop
LAYOUTS = {
    "tiny": ((5, 5), (0, 0), None, ((2.2, 2.4), 1.5)),
    "box": ((9, 11), (1, 1), None, ((4.0, 5.0), 2.0)),
    "odd": ((65, 41), (0, 0), dict(center=(32.3, 12.4), radius=8.2), ((32.0, 28.0), 7.5)),
    "floor": ((97, 63), (0, 1), dict(center=(47.7, 12.3), radius=14.4), ((47.5, 36.2), 9.5)),
    "cavity": ((64, 64), (0, 0), dict(center=(31.6, 32.2), radius=27.5, cavity=True), ((31.6, 14.0), 9.0)),
    "wrapped": ((70, 52), (0, 0), dict(center=(3.3, 49.6), radius=11.2), ((35.0, 20.0), 9.0)),
    "middle": ((385, 303), (1, 1), dict(center=(190.2, 60.3), radius=50.5), ((190.0, 139.0), 28.0)),
    "large": ((833, 497), (0, 1), dict(center=(410.2, 60.3), radius=70.5), ((410.0, 180.0), 49.0)),
}


def lattice(layout, model, precision, collision, wall, step_kernel):
    n, box, solid, drop = LAYOUTS[layout]
    mu_w, width, params = MODELS[model]
    lat = G.Lattice(G.LBM_D2Q9, n=n + (1,), precision=precision, axis_bc=box + (0,), collision=collision, bc_mode=wall,
                    Tr=0.8, g=(2e-6, -3e-6), g_start_step=21, step_kernel=step_kernel, **params)
    if solid:
        lat.set_solids([dict(solid, mu_w=mu_w)])
    lat.init_drops([drop], W=width)
    return lat


@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("model", list(MODELS))
@pytest.mark.parametrize("precision", [G.LBM_F32, G.LBM_F64, G.LBM_F32_MIXED])
def test_equals_the_split_step(layout, model, precision):
    for collision, wall in ((G.LBM_MRT, G.LBM_BC_HALFWAY), (G.LBM_BGK, G.LBM_BC_BOUZIDI_MC)):
        a, b = (lattice(layout, model, precision, collision, wall, k) for k in (G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT))
        every = 19 if LAYOUTS[layout][2] else 0
        for n in (1, 18, 79):  # the first step from S_t, then windows that are captured, and measure steps between them
            sa, sb = (x.step(n, measure_every=every, cap=10 if every else 0) for x in (a, b))
            assert [r.step for r in sa] == [r.step for r in sb]
            for ra, rb in zip(sa, sb):
                assert bytes(ra) == bytes(rb)
        assert np.array_equal(a.f, b.f)
        assert np.array_equal(a.rho, b.rho)
        if model == "phase":
            assert np.array_equal(a.g, b.g) and np.array_equal(a.phi, b.phi)
        assert a.info()["step"] == b.info()["step"] == 98


def test_large_batch_equals_the_split_step():
    # over 4 million nodes in all, several tiles per compute unit
    cases = [dict(n=(1201 + 64 * k, 1099 - 30 * k), solid=dict(center=(600.3, 200.2), radius=150.0, mu_w=0.04),
                  drop=((600.0, 430.0), 80.0)) for k in range(4)]
    a, b = (G.Batch(cases, Tr=0.8, step_kernel=k) for k in (G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT))
    for x in (a, b):
        x.step(37, measure_every=18)
        x.sync()
    for ra, rb in zip(a.angles(), b.angles()):
        assert bytes(ra) == bytes(rb)
    for i in range(len(cases)):
        assert np.array_equal(a.read(i, G.FIELD_F), b.read(i, G.FIELD_F))
