"""D-phase graph capture and replay (GPU, through the C ABI).

The paper's D path replays captured graphs against the phase's stable
buffers (Section 6.1).  A D layer captured once and replayed must give the
eager layer's bits on every replay, with the other phase's eager work and
host synchronisations between replays.
"""
import numpy as np
import pytest

from synth import BF16, LayerSpec, make_config, make_layer
from tests.gpu_util import GpuLayer
from tests.test_gpu_layer import check_phase

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _d_state(g):
    res = g.fetch(1)
    return {k: res[k].copy() for k in ("topk_idx", "topk_w", "counts", "offsets", "row_of_slot", "token_of_row",
                                       "x_perm_raw", "h_raw", "y", "out")}


@pytest.mark.parametrize("d_priority_us", [0, 300])
def test_d_layer_graph_replays_match_eager(d_priority_us):
    import torch

    inp = make_config(1)
    g = GpuLayer(inp, d_priority_us=d_priority_us)
    try:
        M = g.M
        sg = torch.cuda.Stream()
        # eager D on the capture stream first (the phase last ran there)
        g.run(1, stream=sg)
        torch.cuda.synchronize()
        ref = _d_state(g)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=sg):
            M.layer(g.ctx, 1, g.logits[1], g.T[1], g.x[1], g.out[1], sg)
        torch.cuda.synchronize()
        for rep in range(3):
            g.out[1].zero_()
            g.run(0)  # the P phase, eager, on its own stream
            torch.cuda.synchronize()
            with torch.cuda.stream(sg):
                graph.replay()
            torch.cuda.synchronize()
            got = _d_state(g)
            for key in ref:
                assert np.array_equal(got[key], ref[key]), (rep, key)
        # replay concurrently with eager P, then check once more
        g.out[1].zero_()
        torch.cuda.synchronize()
        g.run(0)
        with torch.cuda.stream(sg):
            graph.replay()
        torch.cuda.synchronize()
        got = _d_state(g)
        for key in ref:
            assert np.array_equal(got[key], ref[key]), ("concurrent", key)
        # the replayed D layer (every stage) and the eager P layer beside it
        # against the oracle
        check_phase(g, inp, 1)
        check_phase(g, inp, 0)
        # the eager API still works on the phase after the replays
        g.run(1, stream=sg)
        torch.cuda.synchronize()
        assert np.array_equal(_d_state(g)["out"], ref["out"])
        del graph
    finally:
        g.close()


@pytest.mark.filterwarnings("ignore:The CUDA Graph is empty")
def test_capture_refuses_a_stream_hand_over():
    """A phase last driven on one stream cannot start a capture on another:
    the hand-over wait could not be part of the graph."""
    import torch

    inp = make_config(1)
    g = GpuLayer(inp)
    try:
        M = g.M
        g.run(1)  # the phase's stream is now g.streams[1]
        torch.cuda.synchronize()
        sg = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        st = None
        with torch.cuda.graph(graph, stream=sg):
            st = M.moe_route(g.ctx, 1, g.logits[1], g.T[1], sg)
        assert st == M.MOE_ERR_STATE
        torch.cuda.synchronize()
        # nothing was enqueued and the phase is still usable from its stream
        g.run(1)
        torch.cuda.synchronize()
        del graph
    finally:
        g.close()


@pytest.mark.parametrize("form", ["staged", "direct"])
def test_captured_ffn_replays_after_eager_dispatch(form):
    """Any of a phase's calls may be captured: here the FFN and the combine,
    replayed after an eager route and dispatch of the same T.  Between the
    capture and the replay the other phase changes its tile regime, so the
    dispatch would choose the other form of the small tiles (LDS-staged or
    register-direct) than the captured one.  Experts of several 32-row blocks
    (up to 201 rows) and more 32-row blocks than a grid of 96-row tiles has
    workgroups for; y is poisoned before each replay, so a row that no tile
    computed would show."""
    import torch

    from tests.test_gpu_layer import _poison_y

    rows = [201, 97, 64, 33, 32, 1, 0, 40]
    E, E_loc, T = 64, len(rows), sum(rows)
    spec = LayerSpec("split-capture", E=E, e0=8, E_loc=E_loc, k=1, H=128, I=192, dtype=BF16, T_P=64 * 512, T_D=T)
    inp = make_layer(spec, seed=51)
    owner = 8 + np.random.default_rng(52).permutation(np.repeat(np.arange(E_loc), rows))
    inp.logits[1] = np.where(np.arange(E)[None, :] == owner[:, None], 1.0, -1.0).astype(np.float32)
    prefill, wide = 64 * 32, 64 * 512  # tokens of the P batches: its prefill tiles, its 256-row tiles
    g = GpuLayer(inp)
    try:
        M = g.M
        sg = torch.cuda.Stream()

        def dispatch():
            M.check(M.moe_route(g.ctx, 1, g.logits[1], T, sg))
            M.check(M.moe_dispatch(g.ctx, 1, g.x[1], sg))

        g.run(0, T=prefill if form == "direct" else wide)
        torch.cuda.synchronize()
        dispatch()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=sg):
            M.check(M.moe_expert_ffn(g.ctx, 1, sg))
            M.check(M.moe_combine(g.ctx, 1, g.out[1], sg))
        torch.cuda.synchronize()
        for rep, p_tokens in enumerate((wide, prefill, wide)):
            g.run(0, T=p_tokens)
            torch.cuda.synchronize()
            dispatch()
            _poison_y(g, 1)
            with torch.cuda.stream(sg):
                graph.replay()
            torch.cuda.synchronize()
            assert np.isfinite(g.fetch(1)["y"]).all(), (form, rep)
            check_phase(g, inp, 1)
            # the captured calls left the host state at the dispatch
            M.check(M.moe_phase_reset(g.ctx, 1))
        del graph
    finally:
        g.close()


def test_eager_d_layer_while_another_thread_captures():
    """D asks whether P has work in flight, on whatever thread drives it: that
    must not break a capture that another thread has open in the global mode."""
    import threading

    import torch

    inp = make_layer(LayerSpec("capture-thread", E=64, e0=0, E_loc=64, k=2, H=256, I=256, dtype=BF16, T_P=300, T_D=20),
                     seed=53)
    g = GpuLayer(inp, d_priority_us=200)
    try:
        g.run(0)  # a small P batch: D's next layer asks about it
        g.run(1)
        torch.cuda.synchronize()
        ref = _d_state(g)
        a = torch.ones(1024, device="cuda")
        b = torch.zeros(1024, device="cuda")
        torch.cuda.synchronize()
        failed = []

        def eager():
            try:
                torch.cuda.set_device(0)
                for _ in range(3):
                    g.run(1)
            except Exception as e:  # noqa: BLE001 (reported below, on the test's thread)
                failed.append(e)

        graph, sg = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=sg, capture_error_mode="global"):
            t = threading.Thread(target=eager)
            t.start()
            t.join()
            torch.add(a, a, out=b)
        assert not failed, failed
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(b, a + a)
        got = _d_state(g)
        for key in ref:
            assert np.array_equal(got[key], ref[key]), key
        del graph
    finally:
        g.close()
