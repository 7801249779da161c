"""A routing step (estimate with the trajectory, route in the commit) and the what-if's
estimates over every split of the queries into blocks, against the oracle, bit for bit."""

from __future__ import annotations

import dataclasses
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_util import DEV, T, assert_state_equal, bits  # noqa: E402
from oracle import oracle as O  # noqa: E402
from paper_2607_18253_amd import LarError, context_for  # noqa: E402
from paper_2607_18253_amd.lar import LAR_E_ARG, LAR_E_STATE  # noqa: E402
from workloads import make_tiny_workload  # noqa: E402
from workloads.gen import make_tiny_sched_workload  # noqa: E402


# one lane, a full wave and one more, two passes of 256 instances; the engine beyond the
# trajectory walk's one partly served request comes up in the tiny pools by itself
@pytest.mark.parametrize("n_inst", [1, 5, 64, 65, 257])
@pytest.mark.parametrize("limits,constrained", [(False, False), (False, True), (True, False)])
def test_route_steps(n_inst, limits, constrained):
    make = make_tiny_sched_workload if limits else make_tiny_workload
    wl = make(700 + n_inst, n_inst=n_inst, n_q=24, max_res=5, n_scen=2)
    N, Z = wl.n_q, wl.n_scen
    tau = np.random.default_rng(n_inst).uniform(0.0, 40.0, size=N) if constrained else None
    print(f"route steps: {n_inst} instances, limits {limits}, constrained {constrained}",
          flush=True)
    reading = n_inst % 2
    ctx = context_for(wl, flags=reading, max_iters=200_000)
    ctx.advance(float(wl.q_t_ms[0]))
    f64, i32 = torch.float64, torch.int32
    qp, qd, qt = T(wl.q_prefill, i32), T(wl.q_decode, i32), T(wl.q_t_ms, f64)
    ends = torch.cat([qt[1:], qt[-1:]]).contiguous()
    acc, cost, wc = T(wl.acc, f64), T(wl.cost, f64), T(wl.w_cost, f64)
    wl_ms = T(wl.w_lat_ms, f64)
    tt = T(tau, f64) if constrained else None
    choice = torch.full((N, Z), -2, dtype=i32, device=DEV)
    chosen = torch.full((N, Z), -1.0, dtype=f64, device=DEV)
    util = torch.full((N, Z), -1.0, dtype=f64, device=DEV)
    for i in range(N):
        ctx.route_step(qp[i:i + 1], qd[i:i + 1], qt[i:i + 1], ends[i:i + 1], acc[i], cost[i],
                       wc, None if constrained else wl_ms,
                       tau_ms=tt[i:i + 1] if constrained else None, choice=choice[i],
                       chosen_ttft=chosen[i], utility=util[i])
    ctx.sync()
    for z in range(Z):
        ref = O.trace(wl, scenario=z, reading=reading, tau=tau, max_iters=200_000,
                      final_state=True)
        np.testing.assert_array_equal(choice[:, z].cpu().numpy(), ref.choice)
        np.testing.assert_array_equal(bits(chosen[:, z].cpu().numpy()), bits(ref.ttft_chosen))
        np.testing.assert_array_equal(bits(util[:, z].cpu().numpy()), bits(ref.util_chosen))
        assert_state_equal(ctx, z, ref)
    ctx.close()


# queries per block: 1 (up to 512 blocks' worth), 2 with a remainder, the full 16 with a
# remainder, and two column blocks
@pytest.mark.parametrize("n_inst,n_q", [(3, 1), (3, 512), (3, 513), (3, 1025), (3, 8193),
                                        (257, 257), (257, 261)])
def test_estimate_chunks(n_inst, n_q):
    wl = make_tiny_workload(800 + n_q, n_inst=n_inst, n_q=n_q)
    print(f"estimate chunks: {n_inst} instances x {n_q} queries", flush=True)
    ctx = context_for(wl, max_iters=200_000)
    tt, it = ctx.estimate(T(wl.q_prefill, torch.int32), 0.0)
    ctx.sync()
    # the estimate depends on the prompt alone: the oracle simulates each length once
    lens, at = np.unique(wl.q_prefill, return_index=True)
    ref_t, ref_i = O.estimate_matrix(wl, at.tolist(), range(n_inst), 0.0)[:2]
    row = np.searchsorted(lens, wl.q_prefill)
    np.testing.assert_array_equal(bits(tt.cpu().numpy()[0]), bits(np.asarray(ref_t)[row]))
    np.testing.assert_array_equal(it.cpu().numpy()[0], np.asarray(ref_i)[row])
    ctx.close()


@pytest.mark.parametrize("n_inst", [3, 3000])
def test_step_reports_the_first_kind_of_error(n_inst):
    """One step that finds errors of different kinds reports what separate calls would: an
    instance behind t (the estimate's trajectory) before a prompt out of range (the
    estimate) before an iteration cap (the commit's replay)."""
    wl = make_tiny_workload(900, n_inst=n_inst, n_q=2, max_res=5)
    f64, i32 = torch.float64, torch.int32
    acc, cost = T(wl.acc[0], f64), T(wl.cost[0], f64)
    wc, w_lat = T(wl.w_cost, f64), T(wl.w_lat_ms, f64)

    def step(ctx, p, t, t_next):
        ctx.route_step(T([p], i32), T([4], i32), T([t], f64), T([t_next], f64), acc, cost, wc, w_lat)
        with pytest.raises(LarError) as ei:
            ctx.sync()
        return ei.value.code

    bad = wl.max_prompt + 1
    clocks = np.zeros(n_inst)
    clocks[n_inst - 1] = -5.0   # the last instance alone is behind
    behind = dataclasses.replace(wl, clock_ms=clocks)
    print(f"step errors: {n_inst} instances", flush=True)
    for _ in range(5):
        ctx = context_for(behind)
        assert step(ctx, bad, 0.0, 1.0) == LAR_E_STATE
        ctx.close()
        ctx = context_for(wl, max_iters=3)
        assert step(ctx, bad, 0.0, 1e9) == LAR_E_ARG
        ctx.close()
