"""lbm_step and lbm_batch_step issued while their stream is being captured: the
capture records the split step, and what replays and later ordinary calls do
equals the same sequence on a lattice that takes the split step throughout
(whose launches read the step counter on the device)."""
import numpy as np
import pytest

from paper_2202_06516_amd import lbm as G

from .test_gpu_step2d import LAYOUTS, MODELS

pytestmark = pytest.mark.gpu

EVERY, REPLAYS = 7, 5


def captured(stream, step):
    import torch
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        step()
    return graph


@pytest.mark.parametrize("model", list(MODELS))
@pytest.mark.parametrize("precision", [G.LBM_F32, G.LBM_F64])
def test_replays_count_for_the_steps_that_follow(model, precision):
    # 2 steps, a captured call of 4 replayed 5 times (the body force starts at
    # step 21, within a replay), then 42 ordinary steps: graph windows and
    # measurements fall where the device's step counter says
    import torch
    n, box, solid, drop = LAYOUTS["floor"]
    mu_w, width, params = MODELS[model]
    lats, graphs = [], []
    for kernel in (G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT):
        stream = torch.cuda.Stream()
        lat = G.Lattice(G.LBM_D2Q9, n=n + (1,), precision=precision, axis_bc=box + (0,), collision=G.LBM_BGK, Tr=0.8,
                        g=(2e-6, -3e-6), g_start_step=21, step_kernel=kernel, stream=stream.cuda_stream, **params)
        lat.set_solids([dict(solid, mu_w=mu_w)])
        lat.init_drops([drop], W=width)
        lat.step(2)
        lat.sync()
        graphs.append(captured(stream, lambda: lat.step(4, measure_every=EVERY)))
        lats.append((lat, stream))
    eager = G.Lattice(G.LBM_D2Q9, n=n + (1,), precision=precision, axis_bc=box + (0,), collision=G.LBM_BGK, Tr=0.8,
                      g=(2e-6, -3e-6), g_start_step=21, step_kernel=G.LBM_STEP_SPLIT, **params)
    eager.set_solids([dict(solid, mu_w=mu_w)])
    eager.init_drops([drop], W=width)
    eager.step(2)
    for _ in range(REPLAYS):
        eager.step(4, measure_every=EVERY)
        for graph, (lat, stream) in zip(graphs, lats):
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(lat.f, eager.f)
    a, b = (lat for lat, _ in lats)
    for nsteps in (7, 35):
        sa, sb, se = (x.step(nsteps, measure_every=EVERY, cap=10) for x in (a, b, eager))
        assert len(sa) == len(sb) == len(se) > 0
        for ra, rb, re in zip(sa, sb, se):
            assert bytes(ra) == bytes(rb) == bytes(re)
        assert np.array_equal(a.f, b.f) and np.array_equal(a.f, eager.f)
    # a new initial state counts from zero on the host and on the device alike
    for x in (a, b, eager):
        x.init_drops([drop], W=width)
    sa, sb, se = (x.step(44, measure_every=EVERY, cap=10) for x in (a, b, eager))
    assert [r.step for r in sa] == [r.step for r in sb] == [r.step for r in se] == list(range(0, 44, EVERY))
    assert np.array_equal(a.f, b.f) and np.array_equal(a.f, eager.f)


def test_captured_batch_steps_equal_the_split_step():
    # every lbm_batch_step call sets the device's counter from the batch's own,
    # replays included
    import torch
    cases = [dict(n=(96 - 7 * k, 70 + 5 * k), solid=dict(center=(45.2, 14.6), radius=11.2, mu_w=0.04),
                  drop=((45.0, 35.0), 9.0)) for k in range(3)]
    batches = []
    for kernel in (G.LBM_STEP_AUTO, G.LBM_STEP_SPLIT):
        stream = torch.cuda.Stream()
        b = G.Batch(cases, precision=G.LBM_F32, Tr=0.8, g=(2e-6, -3e-6), g_start_step=9, step_kernel=kernel,
                    stream=stream.cuda_stream)
        b.step(2)
        b.sync()
        graph = captured(stream, lambda: b.step(4, measure_every=EVERY))
        for _ in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            b.read(0, G.FIELD_RHO)
        b.step(40, measure_every=EVERY)
        b.sync()
        batches.append(b)
    for ra, rb in zip(*(b.angles() for b in batches)):
        assert bytes(ra) == bytes(rb)
    for i in range(len(cases)):
        assert np.array_equal(batches[0].read(i, G.FIELD_F), batches[1].read(i, G.FIELD_F))
