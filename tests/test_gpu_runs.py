"""The split step on lattices whose rows and planes end inside a workgroup's
run of 256 consecutive nodes, against the FP64 oracle."""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G

from .pairs import gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

# rows shorter and longer than a run, a last run that is not full, planes
# that end inside runs, and a plane smaller than two runs
SHAPES = [(37, 29, 31), (131, 21, 23), (17, 15, 37), (257, 13, 21), (65, 19, 27), (297, 41, 1), (41, 25, 1)]


@pytest.mark.parametrize("n", SHAPES)
@pytest.mark.parametrize("model", [0, 1, 2])
def test_runs_of_nodes_match_oracle(n, model):
    dim = 2 if n[2] == 1 else 3
    m = n[:dim]
    r = 0.2 * min(m)
    c = tuple(0.5 * v for v in m[:-1]) + (0.33 * m[-1],)
    drop = tuple(c[:-1]) + (c[-1] + 2 * r - 1.0,)
    wl = dict(dim=dim, n=m, wall=(1,) * dim, drops=[(drop, r)], W=5.0, model=model,
              solids=[dict(center=c, radius=r, mu_w=1.2 if model == 1 else 0.02)])
    kw = {} if model else dict(Tr=0.8)
    gp = gpu_lattice(wl, G.LBM_F64, "bgk", step_kernel=G.LBM_STEP_SPLIT, **kw)
    o = oracle_lattice(wl, "bgk", **kw)
    gp.step(6)
    o.step(6)
    assert np.isfinite(o.rho[o.cls == 0]).all()
    assert rel_err(gp.f, o.f) <= 1e-12
