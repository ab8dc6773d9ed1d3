"""The one-pass step (k_step, D3Q19 lattices of whole-row tiles) against the
FP64 oracle and against the split step, element by element.

k_step collides step t and sums the density of step t + 1 in the same pass;
partial sums that cross its tiles go through ghost arrays.  The cases cover
one, two and three waves per row, every z-chunk depth it picks (32, 16, 8, 4, 2),
walls and periodic axes (ghost rows and planes that wrap), the FP32 force
stencil's LDS ring on every shape, halfway and
interpolated walls, MRT and BGK, gravity switched on mid-run, the pseudopotential model, FP64 /
FP32 / FP32 with FP64 arithmetic, in-step measurement, reads between steps, and
graph-captured against eager stepping.
"""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G

from .pairs import gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

SMALL = dict(Tr=0.8)


def case(n, wall, c=None, r=7.3, drop=6.5):
    nx, ny, nz = n
    c = c or (nx / 2 + 0.2, ny / 2 + 0.1, nz / 3 + 0.4)
    return dict(dim=3, n=n, wall=wall, solids=[dict(center=c, radius=r, mu_w=0.04)],
                drops=[((c[0] - 0.2, c[1] - 0.1, c[2] + r + drop - 1.6), drop)])


def fields(gp, o, tol, vel=False):
    o.update_derived()
    fl = o.cls == 0
    layers = (o.cls == 1) | (o.cls == 2)
    e_rho = rel_err(gp.rho, o.rho, fl | layers)
    e_f = rel_err(gp.f, o.f)
    assert e_rho <= tol, f"rho {e_rho:.3e}"
    assert e_f <= tol, f"f {e_f:.3e}"
    if vel:
        vo = o.velocity()
        assert rel_err(gp.read(G.FIELD_VEL), vo, np.broadcast_to(fl, vo.shape)) <= 100 * tol
    return e_rho


def is_fused(gp):
    # the one-pass step reports k_step in its per-kernel profile
    return "k_step" in gp.profile(1)


CASES = [
    # (lattice, walls): 1, 2 and 3 waves per row; z chunks of 8, 2 and 4 planes
    ((64, 24, 32), (1, 1, 1)),
    ((128, 20, 38), (0, 0, 0)),
    ((192, 20, 36), (1, 0, 1)),
]


@pytest.mark.parametrize("n,wall", CASES)
@pytest.mark.parametrize("collision,bc", [("bgk", "halfway"), ("mrt", "halfway"), ("mrt", "bouzidi")])
def test_one_pass_matches_oracle_f64(n, wall, collision, bc):
    wl = case(n, wall)
    kw = dict(s_q=1.0, s_m=1.0, s_pi=1.0, **SMALL)
    gp = gpu_lattice(wl, G.LBM_F64, collision, bc, **kw)
    assert is_fused(gp)
    o = oracle_lattice(wl, collision, bc, **kw)
    o.step(1)  # the profile call above advanced the GPU lattice one step
    gp.step(9)
    o.step(9)
    fields(gp, o, 1e-12, vel=True)


@pytest.mark.parametrize("zc", ["16", "32"])
def test_one_pass_deep_plane_chunks_match_oracle(zc, monkeypatch):
    # 32 planes per workgroup (the default on large lattices) and 16, set
    # through LBM_FUSED_ZC on a small lattice whose depth they divide
    monkeypatch.setenv("LBM_FUSED_ZC", zc)
    wl = case((64, 24, 64), (1, 0, 0), r=9.1, drop=7.5)
    gp = gpu_lattice(wl, G.LBM_F64, "mrt", "bouzidi", **SMALL)
    assert is_fused(gp)
    o = oracle_lattice(wl, "mrt", "bouzidi", **SMALL)
    o.step(1)
    gp.step(11)
    o.step(11)
    fields(gp, o, 1e-12, vel=True)


def test_one_pass_gravity_and_split_path_agree():
    wl = case((64, 24, 32), (1, 1, 1))
    g = (2e-5, -1e-5, -3e-5)
    a = gpu_lattice(wl, G.LBM_F64, "bgk", g=g, g_start=5, **SMALL)
    b = gpu_lattice(wl, G.LBM_F64, "bgk", g=g, g_start=5, step_kernel=G.LBM_STEP_SPLIT, **SMALL)
    o = oracle_lattice(wl, "bgk", g=g, g_start=5, **SMALL)
    a.step(40)
    b.step(40)
    o.step(40)
    fields(a, o, 1e-12, vel=True)
    assert rel_err(a.f, b.f) <= 1e-13
    assert rel_err(a.read(G.FIELD_MU), b.read(G.FIELD_MU)) <= 1e-12


def test_one_pass_pseudopotential_f64():
    wl = case((64, 24, 32), (1, 1, 1))
    wl.update(model=1, W=5.0)
    wl["solids"][0]["mu_w"] = 1.2   # the wall density
    gp = gpu_lattice(wl, G.LBM_F64, "bgk")
    o = oracle_lattice(wl, "bgk")
    gp.step(20)
    o.step(20)
    fields(gp, o, 1e-12)


@pytest.mark.parametrize("precision,tol", [(G.LBM_F32, 1e-6), (G.LBM_F32_MIXED, 3e-7)])
def test_one_pass_fp32_200_steps(precision, tol):
    wl = case((64, 24, 32), (1, 1, 1))
    gp = gpu_lattice(wl, precision, "bgk", **SMALL)
    o = oracle_lattice(wl, "bgk", **SMALL)
    errs = []
    for _ in range(4):
        gp.step(50)
        o.step(50)
        o.update_derived()
        errs.append(rel_err(gp.rho, o.rho, o.cls <= 2))
    print("density error every 50 steps:", ["%.2e" % e for e in errs])
    assert max(errs) <= tol, errs


@pytest.mark.parametrize("n,wall", CASES + [((512, 16, 32), (0, 1, 1))])
@pytest.mark.parametrize("collision", ["bgk", "mrt"])
def test_one_pass_fp32_stencil_ring_shapes(n, wall, collision):
    # FP32 storage takes the force stencil's centre, z and x neighbours from the
    # LDS ring on rows of up to 256 nodes: one, two and three waves per row (x
    # neighbours across waves and across the periodic row end), every
    # plane-chunk depth of CASES; and a row of 512 (eight waves, no ring)
    wl = case(n, wall)
    kw = dict(s_q=1.0, s_m=1.0, s_pi=1.0, **SMALL)
    gp = gpu_lattice(wl, G.LBM_F32, collision, **kw)
    assert is_fused(gp)
    o = oracle_lattice(wl, collision, **kw)
    o.step(1)
    gp.step(59)
    o.step(59)
    o.update_derived()
    e = rel_err(gp.rho, o.rho, o.cls <= 2)
    print(f"{n} {collision}: density error {e:.2e}")
    assert e <= 1e-6


@pytest.mark.parametrize("nx,zc", [(320, None), (384, "16"), (448, None), (512, "16")])
@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("precision,tol", [(G.LBM_F32, 1e-6), (G.LBM_F32_MIXED, 3e-7), (G.LBM_F64, 1e-12)])
def test_one_pass_rows_of_five_to_eight_waves(nx, zc, collision, precision, tol, monkeypatch):
    # double arithmetic has a kernel each for rows of up to 384 and 512 nodes,
    # FP32 BGK one with the stencil ring for 321 to 384: x neighbours across
    # waves and the periodic row end, planes per workgroup of 8 (small lattice)
    # and 16
    if zc:
        monkeypatch.setenv("LBM_FUSED_ZC", zc)
    wl = case((nx, 16, 32), (0, 1, 1))
    gp = gpu_lattice(wl, precision, collision, **SMALL)
    assert is_fused(gp)
    o = oracle_lattice(wl, collision, **SMALL)
    o.step(1)
    gp.step(29)
    o.step(29)
    o.update_derived()
    assert rel_err(gp.rho, o.rho, o.cls <= 2) <= tol


def test_one_pass_in_step_measurement_matches_oracle():
    wl = case((128, 24, 40), (1, 1, 1), r=9.1, drop=8.0)
    gp = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    gp.set_measure(0, 16)
    o = oracle_lattice(wl, "bgk", **SMALL)
    ga = gp.step(150, measure_every=50, cap=8)
    oa = o.step_measured(150, 50, 0, 16)
    assert len(ga) == len(oa) == 3
    for a, b in zip(ga, oa):
        assert a.step == b.step and a.n_valid == b.n_valid
        for s in range(16):
            x, y = a.sector_deg[s], b.sector_deg[s]
            assert (np.isnan(x) and np.isnan(y)) or abs(x - y) < 1e-6, (a.step, s, x, y)
    # a measurement call that starts at a measure step after steps that did not measure
    gp.step(50)
    o.step(50)
    ga = gp.step(1, measure_every=200, cap=2)
    oa = o.step_measured(1, 200, 0, 16)
    assert len(ga) == len(oa) == 1 and ga[0].n_valid == oa[0].n_valid > 0
    assert abs(ga[0].mean_deg - oa[0].mean_deg) < 1e-6
    # and the standalone measurement after one-pass steps
    m = gp.measure(0, 16)
    mo = o.measure(0, 16)
    assert abs(m.mean_deg - mo.mean_deg) < 1e-6


def test_one_pass_graph_and_eager_agree():
    # 70 steps = eager steps to parity + two captured graphs of 32 + the rest
    wl = case((64, 24, 32), (1, 1, 1))
    a = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    b = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    a.step(70)
    for _ in range(70):
        b.step(1)
    assert np.array_equal(a.f, b.f)
    assert np.array_equal(a.rho, b.rho)


def test_one_pass_quiet_graphs_keep_the_measure_steps():
    # cadence 40 over 200 steps: captured windows of 32 steps with a measure
    # step (full steps) and without one (quiet steps, without k_cross and
    # k_finalize); the angles, their steps and the fields equal those of
    # single eager steps bit for bit, and so does a later measurement
    wl = case((64, 24, 32), (1, 1, 1))
    a = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    b = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    a.set_measure(0, 8)
    b.set_measure(0, 8)
    ga = a.step(200, measure_every=40, cap=8)
    gb = []
    for _ in range(200):
        gb += b.step(1, measure_every=40, cap=1)
    assert [r.step for r in ga] == [r.step for r in gb] == [0, 40, 80, 120, 160]
    for x, y in zip(ga, gb):
        assert x.n_valid == y.n_valid > 0
        assert np.array_equal(np.asarray(x.sector_deg), np.asarray(y.sector_deg), equal_nan=True)
    assert np.array_equal(a.f, b.f)
    assert np.array_equal(a.rho, b.rho)
    # a later call whose windows are all quiet, then one that measures at once
    a.step(96, measure_every=1000)
    for _ in range(96):
        b.step(1, measure_every=1000)
    ra, rb = a.step(40, measure_every=8, cap=8), b.step(40, measure_every=8, cap=8)
    assert [r.step for r in ra] == [r.step for r in rb] == [296, 304, 312, 320, 328]
    assert np.array_equal(np.asarray(ra[-1].sector_deg), np.asarray(rb[-1].sector_deg), equal_nan=True)
    ma, mb = a.measure(0, 8), b.measure(0, 8)
    assert ma.step == mb.step == 336 and ma.n_valid == mb.n_valid
    assert np.array_equal(np.asarray(ma.sector_deg), np.asarray(mb.sector_deg), equal_nan=True)


def test_one_pass_reads_and_writes_between_steps():
    wl = case((64, 24, 32), (1, 1, 1))
    a = gpu_lattice(wl, G.LBM_F64, "bgk", **SMALL)
    o = oracle_lattice(wl, "bgk", **SMALL)
    a.step(15)
    o.step(15)
    m0 = a.mass()
    f = a.f
    rho = a.rho
    a.write(G.FIELD_F, f)          # checkpoint restore: the density is derived again
    a.step(15)
    o.step(15)
    fields(a, o, 1e-12)
    assert abs(a.mass() / m0 - 1.0) < 1e-12
    a.write(G.FIELD_RHO, rho)      # warm start from a density
    o.set_rho(rho)
    a.step(10)
    o.step(10)
    fields(a, o, 1e-12)


def test_split_is_used_where_the_one_pass_step_cannot_tile():
    for n in ((70, 24, 32), (64, 22, 32), (64, 24, 33)):
        gp = gpu_lattice(case(n, (1, 1, 1)), G.LBM_F64, "bgk", **SMALL)
        assert not is_fused(gp), n
    # the interpolated wall takes the one-pass step too; the phase-field model does not
    assert is_fused(gpu_lattice(case((64, 24, 32), (1, 1, 1)), G.LBM_F64, "bgk", "bouzidi", **SMALL))


@pytest.mark.parametrize("precision,tol", [(G.LBM_F32, 1e-6), (G.LBM_F64, 1e-12)])
def test_one_pass_interpolated_wall_matches_split_path(precision, tol):
    # a sphere whose cut links span q in (0, 1) and a drop over it, 60 steps on
    # both paths of the same build: the one-pass step's interpolated wall
    # equals the split path's gather (the density sums differ in order only)
    wl = case((128, 28, 40), (1, 1, 1), r=9.3, drop=7.0)
    a = gpu_lattice(wl, precision, "bgk", "bouzidi", **SMALL)
    b = gpu_lattice(wl, precision, "bgk", "bouzidi", step_kernel=G.LBM_STEP_SPLIT, **SMALL)
    assert is_fused(a) and not is_fused(b)
    a.step(59)
    b.step(59)
    fl = a.read(G.FIELD_CLASS) <= 2
    assert rel_err(a.rho, b.rho, fl) <= tol
    assert rel_err(a.f, b.f) <= tol
    assert abs(a.mass() / b.mass() - 1.0) <= tol
