"""The batch engine under scheduler limits at the edges of its branches, against the
oracle, bit for bit: the requests one stage serves one by one and those it serves by
prefix sums, rows of 64 list entries, victims in several rows, folded batches, admission
points that queries join and that a what-if call shares."""

from __future__ import annotations

import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_util import DEV, T, assert_state_equal, bits  # noqa: E402
from oracle import oracle as O  # noqa: E402
from paper_2607_18253_amd import LarContext, context_for  # noqa: E402
from workloads import make_tiny_workload  # noqa: E402

MAX_ITERS = 200_000


def _pool(seed, *, M, B, res, prompt, decode, H, S, slack, terms, n_q=30, gap=3.0):
    """Pool of 5 instances with `res` residents each; KV blocks: what the residents hold
    plus `slack` (None: no KV cache); terms: with the context and attention terms."""
    wl = make_tiny_workload(seed, n_inst=5, max_res=res, budget=(B, B), max_seqs=(M, M),
                            prompt=prompt, decode=decode, n_q=n_q, mean_gap_ms=gap)
    if not terms:
        wl.d[:], wl.e[:] = 0.0, 0.0
    longest = max([int((rp + cx).max()) for rp, _, cx in
                   (wl.instance_requests(j) for j in range(5)) if len(rp)] + [0])
    X = max(longest, wl.max_prompt) + 1 + decode[1] // 2
    wl.sched = np.zeros((5, 4), np.int32)
    for j in range(5):
        _, _, cx = wl.instance_requests(j)
        K = 0
        if slack is not None:
            K = max(-(-X // S), int(sum(-(-int(c) // S) for c in cx))) + slack
        wl.sched[j] = (H, K, S if K else 0, X)
    return wl


POOLS = {
    # one token a chunk: every partial prefill is served, more than a stage's few
    "many_partials": dict(M=70, B=80, res=70, prompt=(1, 9), decode=(1, 6), H=1, S=2, slack=3),
    "partials_3_4": dict(M=5, B=12, res=5, prompt=(1, 20), decode=(1, 9), H=2, S=2, slack=40),
    # short prompts against a wide budget: long admission prefixes
    "admissions": dict(M=130, B=200, res=200, prompt=(1, 4), decode=(1, 6), H=0, S=1, slack=9),
    "admissions_3_4": dict(M=8, B=8, res=12, prompt=(1, 3), decode=(1, 3), H=2, S=1, slack=2),
    "no_cache": dict(M=65, B=90, res=140, prompt=(1, 6), decode=(1, 12), H=3, S=1, slack=None),
    # full caches: victims in every batch, across rows
    "preempt": dict(M=64, B=70, res=64, prompt=(1, 12), decode=(2, 30), H=4, S=4, slack=0),
    "preempt_rows": dict(M=140, B=150, res=150, prompt=(1, 6), decode=(2, 20), H=2, S=1, slack=1),
    # few requests, long prompts chunk by chunk: folded batches, with and without a cache
    "folds": dict(M=6, B=9, res=3, prompt=(60, 200), decode=(30, 200), H=2, S=8, slack=60,
                  gap=120.0),
    "folds_tight": dict(M=6, B=40, res=4, prompt=(60, 200), decode=(30, 200), H=7, S=16, slack=2,
                        gap=120.0),
    "folds_free": dict(M=4, B=30, res=2, prompt=(100, 300), decode=(50, 300), H=9, S=1,
                       slack=None, gap=300.0),
}


def _against_oracle(wl, reading):
    ctx = context_for(wl, flags=reading, max_iters=MAX_ITERS, queue_cap=1024)
    # what-if estimates from the shared admission points (more than 4096 pairs), from the
    # state, and one query alone
    t = 0.0
    many = T(np.resize(wl.q_prefill, 900), torch.int32)
    tm, im = ctx.estimate(many, t)
    tt, it = ctx.estimate(T(wl.q_prefill, torch.int32), t)
    t1, i1 = ctx.estimate(T(wl.q_prefill[:1], torch.int32), t)
    ctx.sync()
    ref_t, ref_i = O.estimate_matrix(wl, range(wl.n_q), range(wl.n_inst), t, reading=reading)[:2]
    ref_t, ref_i = np.asarray(ref_t), np.asarray(ref_i)
    rows = np.arange(900) % wl.n_q
    np.testing.assert_array_equal(bits(tm.cpu().numpy()[0]), bits(ref_t[rows]))
    np.testing.assert_array_equal(im.cpu().numpy()[0], ref_i[rows])
    np.testing.assert_array_equal(bits(tt.cpu().numpy()[0]), bits(ref_t))
    np.testing.assert_array_equal(it.cpu().numpy()[0], ref_i)
    np.testing.assert_array_equal(bits(t1.cpu().numpy()[0]), bits(ref_t[:1]))
    np.testing.assert_array_equal(i1.cpu().numpy()[0], ref_i[:1])
    # the trace: replays, admission points that queries join, first tokens, final state
    ctx.advance(float(wl.q_t_ms[0]))
    f64 = torch.float64
    chosen = torch.full((1, wl.n_q), -1.0, dtype=f64, device=DEV)
    real = torch.full((1, wl.n_q), -1.0, dtype=f64, device=DEV)
    choice = ctx.route_trace(T(wl.q_prefill, torch.int32), T(wl.q_decode, torch.int32),
                             T(wl.q_t_ms, f64), float(wl.q_t_ms[-1]), T(wl.acc, f64),
                             T(wl.cost, f64), T(wl.w_cost, f64), T(wl.w_lat_ms, f64),
                             chosen_ttft=chosen, realized=real)
    ctx.sync()
    ref = O.trace(wl, scenario=0, reading=reading, max_iters=MAX_ITERS, final_state=True)
    np.testing.assert_array_equal(choice.cpu().numpy()[0], ref.choice)
    np.testing.assert_array_equal(bits(chosen.cpu().numpy()[0]), bits(ref.ttft_chosen))
    np.testing.assert_array_equal(bits(real.cpu().numpy()[0]), bits(ref.realized))
    assert_state_equal(ctx, 0, ref)
    ctx.close()


@pytest.mark.parametrize("terms", [False, True])
@pytest.mark.parametrize("name", sorted(POOLS))
def test_batches(name, terms):
    kw = POOLS[name]
    wl = _pool(900 + len(name), terms=terms, **kw)
    print(f"limits batches {name} terms {terms}", flush=True)
    _against_oracle(wl, int(terms))


# windows of 8 and 16 rows with requests running in the upper ones
DEEP = {
    "preempt_300": dict(M=300, B=330, res=420, prompt=(1, 12), decode=(2, 40), H=4, S=4, slack=0,
                        gap=300.0),
    "admissions_400": dict(M=400, B=900, res=500, prompt=(1, 6), decode=(1, 9), H=0, S=1,
                           slack=30, gap=300.0),
    "folds_330": dict(M=330, B=2000, res=330, prompt=(1, 12), decode=(150, 300), H=5, S=8,
                      slack=9000, gap=2000.0),
    "preempt_700": dict(M=700, B=760, res=900, prompt=(1, 8), decode=(2, 40), H=2, S=1, slack=1,
                        gap=600.0),
    "partials_700": dict(M=700, B=720, res=700, prompt=(1, 9), decode=(1, 6), H=1, S=2, slack=3,
                         gap=600.0),
    "no_cache_650": dict(M=650, B=800, res=1000, prompt=(1, 6), decode=(1, 20), H=3, S=1,
                         slack=None, gap=600.0),
    "admissions_1000": dict(M=1000, B=1500, res=1100, prompt=(1, 5), decode=(1, 12), H=3, S=2,
                            slack=200, gap=600.0),
}


@pytest.mark.parametrize("terms", [False, True])
@pytest.mark.parametrize("name", sorted(DEEP))
def test_deep_windows(name, terms):
    kw = DEEP[name]
    # the first seed whose pool runs requests in the row of M / 2 and, beyond M, lists more
    for seed in range(100):
        wl = _pool(seed, terms=terms, **kw)
        run = max(int((wl.instance_requests(j)[2] > 0).sum()) for j in range(5))
        if 2 * run > kw["M"] and np.diff(wl.offsets).max() > min(kw["M"], 0.9 * kw["res"]):
            break
    assert 2 * run > kw["M"] and run > 128
    print(f"limits deep windows {name} terms {terms} seed {seed}: {run} running", flush=True)
    _against_oracle(wl, int(terms))


def test_set_scheduler_takes_no_device_memory():
    """The context's device state is what its creation and load_state allocate; a what-if
    call's admission points lie in it (2048 queues of 1024 sequences)."""
    limits = np.tile(np.array([0, 0, 0, 4096], np.int32), (2048, 1))
    ctx = LarContext(1, 2048, max_seqs_cap=1024, queue_cap=16, max_prompt=64)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(3):
        ctx.set_scheduler(limits)
    assert torch.cuda.mem_get_info()[0] == free
    ctx.close()
