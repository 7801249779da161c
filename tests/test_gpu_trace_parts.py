"""Traces whose scenarios do not all fit the device at once run in several launches, and
pools of up to 1024 sequences per instance keep their queues on chip: choices, TTFTs,
realised TTFTs and final states against the oracle, bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import assert_state_equal, bits, gpu_trace, gpu_trace_realized  # noqa: E402
from oracle import oracle as O  # noqa: E402
from workloads import make_tiny_workload  # noqa: E402


@pytest.mark.parametrize("n_inst,n_scen,mcap,n_q,what", [
    (17, 129, None, 20, "two workgroups of 16 waves each: 258 do not fit, two launches"),
    (17, 300, None, 12, "three launches of 100 scenarios"),
    (33, 171, None, 12, "three workgroups per scenario, three launches of 57"),
    (6, 700, None, 12, "one workgroup per scenario: one launch of any size"),
    (3, 700, None, 12, "one 4-wave workgroup per scenario"),
    (9, 260, 300, 12, "8 slots per lane: two 8-wave workgroups, three launches"),
    (5, 140, 1000, 12, "16 slots per lane: two 4-wave workgroups, two launches"),
    (4, 300, 1000, 12, "16 slots per lane, one workgroup per scenario"),
    (1100, 2, None, 8, "more instances than 64 workgroups hold: the HBM-state kernel"),
])
def test_trace_parts(n_inst, n_scen, mcap, n_q, what):
    wl = make_tiny_workload(40 + n_inst, n_inst=n_inst, max_res=4, n_q=n_q, n_scen=n_scen)
    choice, chosen, util, ctx = gpu_trace(wl, queue_cap=64, max_seqs_cap=mcap)
    for z in sorted({0, n_scen // 2 - 1, n_scen // 2, n_scen - 1} | set(range(0, n_scen, 23))):
        ref = O.trace(wl, scenario=z, queue_cap=64)
        np.testing.assert_array_equal(choice[z], ref.choice, err_msg=f"scenario {z}")
        np.testing.assert_array_equal(bits(chosen[z]), bits(ref.ttft_chosen))
        np.testing.assert_array_equal(bits(util[z]), bits(ref.util_chosen))
        assert_state_equal(ctx, z, ref)
    ctx.close()


@pytest.mark.parametrize("n_inst,n_scen,mcap", [(17, 131, None), (6, 5, 1024)])
def test_trace_parts_realized(n_inst, n_scen, mcap):
    """The same with first tokens tracked, under the constrained objective."""
    wl = make_tiny_workload(90 + n_inst, n_inst=n_inst, max_res=4, n_q=25, n_scen=n_scen)
    tau = O.ttft_targets(wl.q_prefill, wl.tau_u_ms, wl.tau_v) * 0.05
    choice, chosen, real, ctx = gpu_trace_realized(wl, tau=tau, queue_cap=64, max_seqs_cap=mcap)
    for z in sorted({0, n_scen // 2, n_scen - 1}):
        ref = O.trace(wl, scenario=z, queue_cap=64, tau=tau)
        np.testing.assert_array_equal(choice[z], ref.choice, err_msg=f"scenario {z}")
        np.testing.assert_array_equal(bits(chosen[z]), bits(ref.ttft_chosen))
        np.testing.assert_array_equal(bits(real[z]), bits(ref.realized))
        assert_state_equal(ctx, z, ref)
    ctx.close()


@pytest.mark.parametrize("n_inst,n_scen,mcap", [(17, 131, None), (5, 2, 1024)])
def test_trace_parts_captured(n_inst, n_scen, mcap):
    """The launches of such a trace captured in a graph: every replay gives the eager
    run's results, with eager work and a synchronisation between replays."""
    from paper_2607_18253_amd import context_for
    from gpu_util import T
    wl = make_tiny_workload(7 + n_inst, n_inst=n_inst, max_res=4, n_q=20, n_scen=n_scen)
    s = torch.cuda.Stream()
    ctx = context_for(wl, stream=s, queue_cap=64, max_seqs_cap=mcap)
    args = (T(wl.q_prefill, torch.int32), T(wl.q_decode, torch.int32),
            T(wl.q_t_ms, torch.float64), float(wl.q_t_ms[-1]), T(wl.acc, torch.float64),
            T(wl.cost, torch.float64), T(wl.w_cost, torch.float64), T(wl.w_lat_ms, torch.float64))
    choice = torch.zeros((n_scen, wl.n_q), dtype=torch.int32, device="cuda:0")
    chosen = torch.zeros((n_scen, wl.n_q), dtype=torch.float64, device="cuda:0")

    def step():
        ctx.reload_state()
        ctx.advance(float(wl.q_t_ms[0]))
        ctx.route_trace(*args, choice=choice, chosen_ttft=chosen)

    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        step()
    s.synchronize()
    want = choice.clone(), chosen.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        step()
    for _ in range(3):
        choice.zero_()
        chosen.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        s.synchronize()
        assert torch.equal(choice, want[0])
        assert torch.equal(chosen.view(torch.int64), want[1].view(torch.int64))
    ctx.sync()
    ctx.close()


@pytest.mark.parametrize("n_inst,n_scen", [(1, 1), (1, 1300), (2, 2), (2, 600)])
def test_trace_one_or_two_wide_instances(n_inst, n_scen):
    """Up to 1024 sequences on one or two instances: workgroups of as many waves."""
    wl = make_tiny_workload(60 + n_inst, n_inst=n_inst, max_res=40, n_q=70, n_scen=n_scen,
                            max_seqs=(1, 600), budget=(1, 900))
    choice, chosen, util, ctx = gpu_trace(wl, queue_cap=256, max_seqs_cap=1000)
    for z in sorted({0, n_scen - 1} | set(range(0, n_scen, 97))):
        ref = O.trace(wl, scenario=z, queue_cap=256)
        np.testing.assert_array_equal(choice[z], ref.choice, err_msg=f"scenario {z}")
        np.testing.assert_array_equal(bits(chosen[z]), bits(ref.ttft_chosen))
        np.testing.assert_array_equal(bits(util[z]), bits(ref.util_chosen))
        assert_state_equal(ctx, z, O.trace(wl, scenario=z, queue_cap=256, final_state=True))
    ctx.close()


# launches of a trace: the work counters' clear, then per part its exchange's clear and its
# kernel; a refused part leaves its clear
@pytest.mark.parametrize("cus,n_scen,launches", [
    (9, 64, 1 + 2 * 16), (3, 64, 1 + 2 * 64), (1, 62, 1 + 2 * 62), (4096, 131, 1 + 1 + 2 * 2)])
def test_trace_parts_follow_the_device(monkeypatch, cus, n_scen, launches):
    """The parts of a trace are as large as the device holds at once: fewer CUs, smaller
    parts; where it holds less than its CUs say (here: is taken to have more CUs than it
    has), a refused part is halved instead of leaving the chip."""
    import ctypes
    from gpu_util import T
    from paper_2607_18253_amd import context_for
    from paper_2607_18253_amd.lar import LIB_PATH
    monkeypatch.setenv("LAR_TEST_CUS", str(cus))
    wl = make_tiny_workload(90 + cus, n_inst=17, max_res=4, n_q=10, n_scen=n_scen)
    print(f"trace parts: {cus} CUs, {n_scen} scenarios", flush=True)
    choice, chosen, util, ctx = gpu_trace(wl, queue_cap=64)
    for z in sorted({0, n_scen - 1} | set(range(0, n_scen, 13))):
        ref = O.trace(wl, scenario=z, queue_cap=64)
        np.testing.assert_array_equal(choice[z], ref.choice, err_msg=f"scenario {z}")
        np.testing.assert_array_equal(bits(chosen[z]), bits(ref.ttft_chosen))
    ctx.close()
    s = torch.cuda.Stream()
    ctx = context_for(wl, stream=s, queue_cap=64)
    args = (T(wl.q_prefill, torch.int32), T(wl.q_decode, torch.int32),
            T(wl.q_t_ms, torch.float64), float(wl.q_t_ms[-1]), T(wl.acc, torch.float64),
            T(wl.cost, torch.float64), T(wl.w_cost, torch.float64), T(wl.w_lat_ms, torch.float64))
    out = torch.zeros((n_scen, wl.n_q), dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=s):
        ctx.route_trace(*args, choice=out)
    lib, n = ctypes.CDLL(LIB_PATH), ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == launches
    ctx.close()
