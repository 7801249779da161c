"""GPU parity of the average-case LPS estimator (Sec. 4.2, Eqs. 10-13), through the
C ABI (lar_estimate_lps), against the oracle: every entry bit for bit, at the size
of the batched what-if workload (4096 queries x 1024 instances), both modes, routed
through lar_route; several scenarios with parameters of their own; parameters
outside the model."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import DEV, T, bits  # noqa: E402
from oracle import oracle as O  # noqa: E402
from paper_2607_18253_amd import LarContext, context_for  # noqa: E402
from paper_2607_18253_amd import lar as L  # noqa: E402
from workloads import make_workload  # noqa: E402
from workloads.gen import lps_params  # noqa: E402


def _dev_params(prms):
    """[Z] dicts of per-instance arrays -> a GPU uint8 tensor of lar_lps_params."""
    recs = [L.lps_params_array(p["alpha"], p["mu"], p["theta"], p["t_dec"], p["k"], p["ca2"],
                               p["cs2"]) for p in prms]
    return torch.as_tensor(np.concatenate(recs).view(np.uint8).copy(), device=DEV)


@pytest.mark.parametrize("mode", [L.LPS_POISSON, L.LPS_VARIABILITY])
def test_lps_whatif_full_size(mode):
    wl = make_workload("c3")
    prm = lps_params(wl)
    ctx = context_for(wl)   # the snapshot gives the instances' columns for the route
    tt = ctx.estimate_lps(_dev_params([prm]), T(wl.q_prefill, torch.int32), mode)
    ch = ctx.route(tt, T(wl.acc, torch.float64), T(wl.cost, torch.float64),
                   T(wl.w_cost, torch.float64), T(wl.w_lat_ms, torch.float64))
    assert ctx.status() == 0
    got = tt.cpu().numpy()[0]
    want = O.lps_matrix(prm, wl.q_prefill, mode)
    assert np.isfinite(want).all()
    np.testing.assert_array_equal(bits(got), bits(want))
    ch = ch.cpu().numpy()[0]
    for i in range(wl.n_q):
        m, _ = O.route_row(want[i], wl.acc[i], wl.cost[i], wl.col, wl.w_cost[0], wl.w_lat_ms[0])
        assert ch[i] == m, i
    ctx.close()


def test_lps_scenarios_and_ragged_sizes():
    """Three scenarios with parameters of their own, 300 instances (a ragged last
    block of 256), 77 queries; no snapshot loaded (the estimate needs none)."""
    wl = make_workload("c3", n_inst=300, n_q=77, resident=8)
    prms = [lps_params(wl, seed=s) for s in (1, 2, 3)]
    ctx = LarContext(3, wl.n_inst, max_seqs_cap=256, queue_cap=16, max_prompt=wl.max_prompt)
    for mode in (L.LPS_POISSON, L.LPS_VARIABILITY):
        tt = ctx.estimate_lps(_dev_params(prms), T(wl.q_prefill, torch.int32), mode)
        assert ctx.status() == 0
        got = tt.cpu().numpy()
        for z in range(3):
            want = O.lps_matrix(prms[z], wl.q_prefill, mode)
            np.testing.assert_array_equal(bits(got[z]), bits(want), err_msg=f"{mode} {z}")
    ctx.close()


def test_lps_outside_the_model():
    """alpha >= mu, k = 0 or above 65536, a zero throughput, a negative variation
    coefficient (Eq. 13) and a prompt of 0 tokens give NaN there and LAR_E_ARG; the
    other entries are the oracle's."""
    wl = make_workload("c3", n_inst=8, n_q=5, resident=8)
    prm = lps_params(wl)
    prm["alpha"][1] = prm["mu"][1]
    prm["k"][2] = 0
    prm["k"][3] = 65537
    prm["theta"][4] = 0.0
    prm["cs2"][5] = -1.0
    q = np.array(wl.q_prefill, np.int32)
    q[3] = 0
    for mode in (L.LPS_POISSON, L.LPS_VARIABILITY):
        ctx = LarContext(1, wl.n_inst, max_seqs_cap=256, queue_cap=16, max_prompt=wl.max_prompt)
        tt = ctx.estimate_lps(_dev_params([prm]), T(q, torch.int32), mode)
        assert ctx.status() == L.LAR_E_ARG
        got = tt.cpu().numpy()[0]
        want = O.lps_matrix(prm, q, mode)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        ok = ~np.isnan(want)
        assert ok.sum() > 0
        np.testing.assert_array_equal(bits(got[ok]), bits(want[ok]))
        ctx.close()


@pytest.mark.parametrize("n_inst,n_q,n_scen", [(1, 1, 1), (257, 3, 2), (3, 4097, 1),
                                               (5, 6143, 1), (2, 32771, 1), (300, 911, 9)])
def test_lps_query_chunks(n_inst, n_q, n_scen):
    """Every length of the queries' chunks: 1, 2 with a remainder, the full 16 with a
    remainder and over two column blocks; chunks never cross a scenario."""
    wl = make_workload("c3", n_inst=n_inst, n_q=min(n_q, 64), resident=8)
    q = np.resize(wl.q_prefill, n_q) + np.arange(n_q, dtype=np.int32) % 37
    prms = [lps_params(wl, seed=s) for s in range(n_scen)]
    print(f"lps chunks {n_inst} x {n_q} x {n_scen}", flush=True)
    ctx = LarContext(n_scen, n_inst, max_seqs_cap=256, queue_cap=16, max_prompt=wl.max_prompt)
    tt = ctx.estimate_lps(_dev_params(prms), T(q, torch.int32), L.LPS_VARIABILITY)
    assert ctx.status() == 0
    got = tt.cpu().numpy()
    for z in range(n_scen):
        np.testing.assert_array_equal(bits(got[z]), bits(O.lps_matrix(prms[z], q,
                                                                      L.LPS_VARIABILITY)))
    ctx.close()
