"""FP32 BGK rows of 384 and 448 nodes (six and seven waves) take the force
stencil from the LDS ring: whole chunks of 16 and 32 planes, x neighbours across
the periodic row end and at a wall, both wall schemes, against the FP64 oracle."""
import pytest

from paper_2202_06516_amd import lbm as G

from .pairs import gpu_lattice, oracle_lattice, rel_err
from .test_gpu_fused import SMALL, case, is_fused

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [384, 448])
@pytest.mark.parametrize("zc,nz", [("16", 48), ("32", 64)])
@pytest.mark.parametrize("wall,bc", [((0, 0, 0), "halfway"), ((1, 1, 1), "halfway"), ((0, 0, 1), "bouzidi")])
def test_rows_with_the_ring(nx, zc, nz, wall, bc, monkeypatch):
    monkeypatch.setenv("LBM_FUSED_ZC", zc)
    wl = case((nx, 20, nz), wall)
    gp = gpu_lattice(wl, G.LBM_F32, "bgk", bc, **SMALL)
    assert is_fused(gp)
    o = oracle_lattice(wl, "bgk", bc, **SMALL)
    o.step(1)
    gp.step(29)
    o.step(29)
    o.update_derived()
    assert rel_err(gp.rho, o.rho, o.cls <= 2) <= 1e-6
