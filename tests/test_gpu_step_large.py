"""Routing steps on both sides of the pool size where their launches change: as many
launches as documented, and the oracle's results."""

from __future__ import annotations

import ctypes
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_util import DEV, T, assert_state_equal, bits  # noqa: E402
from oracle import oracle as O  # noqa: E402
from paper_2607_18253_amd import context_for  # noqa: E402
from paper_2607_18253_amd.lar import LIB_PATH  # noqa: E402
from workloads import make_tiny_workload  # noqa: E402
from workloads.gen import make_tiny_sched_workload  # noqa: E402

F64, I32 = torch.float64, torch.int32


def _buffers(wl):
    """The device buffers that a step reads and writes."""
    b = {k: torch.zeros(1, dtype=I32, device=DEV) for k in ("qp", "qd")}
    b.update({k: torch.zeros(1, dtype=F64, device=DEV) for k in ("t", "tn")})
    b.update({k: torch.zeros(wl.n_cols, dtype=F64, device=DEV) for k in ("acc", "cost")})
    b.update(wc=T(wl.w_cost, F64), wl=T(wl.w_lat_ms, F64),
             choice=torch.zeros(wl.n_scen, dtype=I32, device=DEV),
             chosen=torch.zeros(wl.n_scen, dtype=F64, device=DEV))
    return b


def _step(ctx, b):
    ctx.route_step(b["qp"], b["qd"], b["t"], b["tn"], b["acc"], b["cost"], b["wc"], b["wl"],
                   choice=b["choice"], chosen_ttft=b["chosen"])


def _steps_against_oracle(wl, ctx, s):
    """Every query of wl through route_step on stream s; scenario 0 against the oracle."""
    ref = O.trace(wl, scenario=0, max_iters=200_000, final_state=True)
    b = _buffers(wl)
    with torch.cuda.stream(s):
        ctx.advance(float(wl.q_t_ms[0]))
        for i in range(wl.n_q):
            b["qp"].fill_(int(wl.q_prefill[i]))
            b["qd"].fill_(int(wl.q_decode[i]))
            b["t"].fill_(float(wl.q_t_ms[i]))
            b["tn"].fill_(float(wl.q_t_ms[min(i + 1, wl.n_q - 1)]))
            b["acc"].copy_(T(wl.acc[i], F64))
            b["cost"].copy_(T(wl.cost[i], F64))
            _step(ctx, b)
            assert int(b["choice"][0].item()) == int(ref.choice[i]), i
            assert bits(b["chosen"].cpu().numpy())[0] == bits(ref.ttft_chosen[i:i + 1])[0], i
    ctx.sync()
    assert_state_equal(ctx, 0, ref)
    return b


def _launches(ctx, b, s):
    """Nodes of a captured step (not replayed)."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=s):
        _step(ctx, b)
    hip = ctypes.CDLL(LIB_PATH)   # finds the runtime that the library itself is linked with
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# Below 4096 queues the estimate follows the trajectory and the route precedes the commit in
# the same launch; from there on each has its own.  Under limits there is no trajectory, and
# one query per queue shares nothing: no launch for admission points, for any pool.
@pytest.mark.parametrize("limits", [False, True])
@pytest.mark.parametrize("n_inst,n_scen", [(5, 1), (4095, 1), (4096, 1), (4100, 1), (2048, 2)])
def test_step_launches(n_inst, n_scen, limits):
    make = make_tiny_sched_workload if limits else make_tiny_workload
    wl = make(31 + n_inst, n_inst=n_inst, n_q=4, max_res=6, n_scen=n_scen)
    print(f"steps: {n_inst} instances, {n_scen} scenarios, limits {limits}", flush=True)
    s = torch.cuda.Stream()
    ctx = context_for(wl, max_iters=200_000, stream=s)
    b = _steps_against_oracle(wl, ctx, s)
    fused = n_inst * n_scen < 4096
    assert _launches(ctx, b, s) == (2 if fused else (3 if limits else 4))
    ctx.close()
