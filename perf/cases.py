"""The performance cases of the router: what a program that uses this library has it do.

Two ways of use, each over pools from a handful of instances to a thousand:

* what-if and one decision at a time -- a snapshot of the pool, a few or many candidate
  queries, the TTFT estimate of every (query, instance) pair and the route: with the
  simulation, with the average-case LPS model, under scheduler limits, without a context
  (`whatif_noalloc`), and a router stepping through arrivals (`route_step`);
* traces -- a day of queries routed in order against pools whose queues are replayed
  between arrivals, for one weight pair or for a sweep of them, with the summaries and the
  realised TTFT that such studies report.

Pools and queries are synthetic: prompts lognormal (or uniform), decode lengths geometric,
Poisson or two-state Markov-modulated arrivals, model types whose batch times are scaled
1x, 2x, 4x and 8x.  Everything is drawn from the seed.
"""

from __future__ import annotations

import math
from collections import deque

import numpy as np
import torch

from paper_2607_18253_amd import lar

DEV = "cuda:0"

# prompt length distributions: short uniform chats, general traffic, long contexts,
# general traffic clipped below a context limit
PROMPTS = {
    "uniform": (64, 2048, 2048),
    "lognormal": (6.5, 1.0, 16, 32768),
    "long": (8.0, 1.5, 32, 131072),
    "clipped": (6.5, 1.0, 16, 7936),
}

BASE = dict(n_scen=1, prompt="lognormal", decode_mean=384, budget=4096, max_seqs=256,
            resident=256, rate_per_inst=1.5625, bursty=False, ctx_term=0.0, attn_term=0.0,
            limits=False, constrained=False, prefill_batch=False)


def listed():
    c = []
    # a small pool, one arrival after another through the online step
    c.append(dict(BASE, name="router_steps", kind="steps", n_inst=4, n_q=64, prompt="uniform",
                  decode_mean=256, budget=2048, max_seqs=64, resident=16, rate_per_inst=5.0))
    # a fresh snapshot in device memory and the queries that wait for it
    c.append(dict(BASE, name="whatif_online", kind="online", n_inst=37, n_q=29))
    # the batched what-if: a large pool's queues against thousands of candidates
    c.append(dict(BASE, name="whatif_pool", kind="whatif", n_inst=1024, n_q=4096, resident=512))
    # the same without workload information: average-case estimates, TTFT targets
    c.append(dict(BASE, name="whatif_lps", kind="lps", n_inst=1024, n_q=4096, resident=0,
                  variability=True, constrained=True))
    # what-if against engines with chunk caps, context limits and a paged KV cache
    c.append(dict(BASE, name="whatif_limits", kind="whatif", n_inst=27, n_q=243, limits=True,
                  prompt="clipped"))
    # a day's trace on a medium pool
    c.append(dict(BASE, name="trace_pool", kind="trace", n_inst=32, n_q=30000))
    # bursty arrivals, TTFT targets, realised TTFT and OnTimeUtility
    c.append(dict(BASE, name="trace_ontime", kind="trace", n_inst=32, n_q=15000, bursty=True,
                  constrained=True))
    # long contexts: wide queues, batch times that grow with the context held
    c.append(dict(BASE, name="trace_long", kind="trace", n_inst=256, n_q=8000, prompt="long",
                  decode_mean=1024, budget=8192, max_seqs=512, resident=1024,
                  rate_per_inst=0.390625, ctx_term=1e-5))
    # engines that run up to 1024 sequences at once
    c.append(dict(BASE, name="trace_1024", kind="trace", n_inst=24, n_q=1500, budget=8192,
                  max_seqs=1024, resident=1024))
    # a trace under chunk caps, context limits and a paged KV cache
    c.append(dict(BASE, name="trace_limits", kind="trace", n_inst=32, n_q=6000, limits=True,
                  prompt="clipped"))
    # a sweep of the two routing weights, 8 x 8, and each scenario's summary
    c.append(dict(BASE, name="sweep", kind="trace", n_inst=64, n_q=12000, n_scen=64))
    # a finer sweep of a smaller pool, 15 x 15
    c.append(dict(BASE, name="sweep_fine", kind="trace", n_inst=30, n_q=1000, n_scen=225))
    return c


def _spread(rng, lo, hi):
    """An integer in lo..hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["steps", "online", "whatif", "whatif", "lps", "whatif_limits", "trace",
                       "trace", "trace", "trace_wide", "trace_limits", "sweep", "sweep"])
    c = dict(BASE)
    c["constrained"] = rng.random() < 0.4
    c["prefill_batch"] = rng.random() < 0.2
    if rng.random() < 0.35:
        c["ctx_term"] = 1e-5
    if rng.random() < 0.25:
        c["attn_term"] = 1e-8
    if kind == "steps":
        c.update(kind="steps", n_inst=_spread(rng, 2, 64), n_q=_spread(rng, 16, 96),
                 max_seqs=rng.choice([64, 128, 256]), resident=_spread(rng, 8, 256))
    elif kind == "online":
        c.update(kind="online", n_inst=_spread(rng, 2, 200), n_q=_spread(rng, 1, 256),
                 resident=_spread(rng, 8, 400), constrained=False)
    elif kind == "whatif":
        c.update(kind="whatif", n_inst=_spread(rng, 16, 1024), n_q=_spread(rng, 16, 4096),
                 resident=_spread(rng, 64, 512), prompt=rng.choice(["lognormal", "uniform"]))
    elif kind == "lps":
        c.update(kind="lps", n_inst=_spread(rng, 16, 1024), n_q=_spread(rng, 16, 4096),
                 resident=0, variability=rng.random() < 0.5)
    elif kind == "whatif_limits":
        c.update(kind="whatif", n_inst=_spread(rng, 4, 64), n_q=_spread(rng, 4, 243),
                 limits=True, prompt="clipped", resident=_spread(rng, 32, 256))
    elif kind == "trace":
        c.update(kind="trace", n_inst=_spread(rng, 2, 128), n_q=_spread(rng, 200, 8000),
                 bursty=rng.random() < 0.4, max_seqs=rng.choice([64, 100, 128, 256]),
                 resident=_spread(rng, 16, 256))
    elif kind == "trace_wide":
        c.update(kind="trace", n_inst=_spread(rng, 4, 24), n_q=_spread(rng, 200, 1000),
                 budget=8192, max_seqs=rng.choice([384, 512, 768, 1024]),
                 resident=_spread(rng, 128, 1024), prompt=rng.choice(["lognormal", "long"]),
                 rate_per_inst=0.390625)
    elif kind == "trace_limits":
        c.update(kind="trace", n_inst=_spread(rng, 2, 32), n_q=_spread(rng, 200, 4000),
                 limits=True, prompt="clipped", resident=_spread(rng, 32, 256))
    else:
        n_inst = _spread(rng, 2, 64)
        c.update(kind="trace", n_inst=n_inst, n_scen=_spread(rng, 2, min(225, 6750 // n_inst)),
                 n_q=_spread(rng, 100, 1000), resident=_spread(rng, 16, 256))
    return c


# ------------------------------------------------------------------ inputs
def _prompts(rng, kind, size):
    spec = PROMPTS[kind]
    if kind == "uniform":
        return rng.integers(spec[0], spec[1] + 1, size=size).astype(np.int32)
    mu, sigma, lo, hi = spec
    return np.clip(np.rint(rng.lognormal(mu, sigma, size=size)), lo, hi).astype(np.int32)


def _arrivals(rng, c, n):
    """Arrival times, ms: Poisson, or Poisson whose rate switches between a low and a six
    times higher state (a fifth of the time high)."""
    rate = c["rate_per_inst"] * c["n_inst"]
    if not c["bursty"]:
        return 1000.0 * np.cumsum(rng.exponential(1.0 / rate, size=n))
    low = rate / (0.8 + 0.2 * 6.0)
    gaps = np.empty(n)
    at, high = 0, bool(rng.random() < 0.2)
    while at < n:
        lam = 6.0 * low if high else low
        k = min(n - at, 1 + int(rng.exponential(2.5 if high else 10.0) * lam))
        gaps[at:at + k] = rng.exponential(1.0 / lam, size=k)
        at, high = at + k, not high
    return 1000.0 * np.cumsum(gaps)


def _pool(c, seed):
    """Host arrays of one case: the snapshot, the queries, the predictions, the weights."""
    rng = np.random.default_rng([int(seed), 26, 7])
    I, R, N, Z = c["n_inst"], c["resident"], c["n_q"], c["n_scen"]
    w = {}
    scale = 2.0 ** (np.arange(I) * 4 // I)
    w["a"], w["b"], w["c"] = 5.0 * scale, 0.02 * scale, 0.3 * scale
    w["d"], w["e"] = np.full(I, c["ctx_term"]), np.full(I, c["attn_term"])
    w["budget"] = np.full(I, c["budget"], np.int32)
    w["max_seqs"] = np.full(I, c["max_seqs"], np.int32)
    # resident requests in arrival order: decoding ones, one partly prefilled, waiting ones
    prompts = _prompts(rng, c["prompt"], (I, R))
    n_dec = min(R // 2, c["max_seqs"] - 1)
    rp, cx = prompts.copy(), np.zeros((I, R), np.int32)
    cx[:, :n_dec] = prompts[:, :n_dec] + rng.integers(0, 256, size=(I, n_dec))
    rp[:, :n_dec] = 0
    if R > n_dec:
        half = prompts[:, n_dec] // 2
        cx[:, n_dec], rp[:, n_dec] = half, prompts[:, n_dec] - half
    w["rem_prefill"], w["context"] = rp.reshape(-1), cx.reshape(-1)
    w["rem_decode"] = rng.geometric(1.0 / c["decode_mean"], size=I * R).astype(np.int32)
    w["offsets"] = np.arange(I + 1, dtype=np.int32) * R
    w["clock_ms"] = np.zeros(I)
    w["q_prefill"] = _prompts(rng, c["prompt"], N)
    w["q_decode"] = rng.geometric(1.0 / c["decode_mean"], size=N).astype(np.int32)
    w["q_t_ms"] = _arrivals(rng, c, N)
    # predictions: one column per model type in traces, one per instance in what-ifs
    per_type = c["kind"] in ("steps", "trace")
    w["col"] = (np.arange(I) * 4 // I).astype(np.int32) if per_type else np.arange(I, dtype=np.int32)
    n_cols = 4 if per_type else I
    w["acc"] = rng.random((N, n_cols))
    if per_type:
        tokens = (w["q_prefill"].astype(np.float64) + w["q_decode"])[:, None]
        cost = tokens * 2.0 ** np.arange(4)[None, :]
        w["cost"] = cost / cost.max()
    else:
        w["cost"] = rng.random((N, n_cols))
    if Z == 1:
        w["w_cost"], w["w_lat"] = np.array([0.5]), np.array([1e-3 if per_type else 1e-5])
    else:
        w["w_cost"] = 10.0 ** rng.uniform(-2.0, 1.0, size=Z)
        w["w_lat"] = 10.0 ** rng.uniform(-5.0, -2.0, size=Z)
    w["u_ms"], w["v"] = rng.uniform(1.0, 5.0, size=N), rng.uniform(0.98, 1.02, size=N)
    if c["kind"] == "lps":
        mu = c["max_seqs"] / ((w["a"] + w["c"] * c["max_seqs"]) * c["decode_mean"])
        w["lps"] = lar.lps_params_array(
            rng.uniform(0.05, 0.98, I) * mu, mu, c["budget"] / (w["a"] + w["b"] * c["budget"]),
            w["a"] + w["c"] * c["max_seqs"] / 2.0, rng.integers(1, 65, I).astype(np.int32),
            ca2=rng.uniform(0.5, 2.0, I), cs2=rng.uniform(0.5, 3.0, I))
    return w


def _max_prompt(c):
    return PROMPTS[c["prompt"]][-1]


def prepare(case, seed):
    c, w = case, _pool(case, seed)
    I, N, Z = c["n_inst"], c["n_q"], c["n_scen"]
    flags = lar.FIRST_TOKEN_PREFILL_BATCH if c["prefill_batch"] else lar.FIRST_TOKEN_DECODE_BATCH
    s = {"case": c, "t0": float(w["q_t_ms"][0]), "t_end": float(w["q_t_ms"][-1]), "flags": flags}

    def dev(key, dtype):
        return torch.as_tensor(np.ascontiguousarray(w[key]), dtype=dtype, device=DEV)

    for key in ("q_prefill", "q_decode"):
        s[key] = dev(key, torch.int32)
    for key in ("q_t_ms", "acc", "cost", "w_cost", "w_lat", "u_ms", "v"):
        s[key] = dev(key, torch.float64)
    f64 = dict(dtype=torch.float64, device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    rows = (Z, N)
    s["choice"] = torch.zeros(rows, **i32)
    s["chosen"], s["utility"] = torch.zeros(rows, **f64), torch.zeros(rows, **f64)
    if c["kind"] in ("online", "whatif", "lps"):
        s["ttft"] = torch.zeros((Z, N, I), **f64)
        s["iters"] = torch.zeros((Z, N, I), **i32)
    if c["kind"] == "online":
        s["params"] = torch.as_tensor(
            np.frombuffer(lar.params_array(w["a"], w["b"], w["c"], w["d"], w["e"], w["budget"],
                                           w["max_seqs"], w["col"]).tobytes(), np.uint8).copy(),
            device=DEV)
        for key in ("offsets", "rem_prefill", "rem_decode", "context"):
            s[key] = dev(key, torch.int32)
        s["clock_ms"] = dev("clock_ms", torch.float64)
        s["status"] = torch.zeros(1, **i32)
        return s
    ctx = lar.LarContext(Z, I, max_seqs_cap=c["max_seqs"], queue_cap=4096 if Z > 64 else 8192,
                         max_prompt=_max_prompt(c), flags=flags)
    if c["limits"]:
        # 512-token chunks, 16-token blocks, 8192-token contexts, 72 blocks per sequence
        ctx.set_scheduler(np.tile(np.array([512, 72 * c["max_seqs"], 16, 8192], np.int32), (I, 1)))
    ctx.load_state(**{k: w[k] for k in ("a", "b", "c", "d", "e", "budget", "max_seqs", "col",
                                        "offsets", "rem_prefill", "rem_decode", "context",
                                        "clock_ms")})
    s["ctx"] = ctx
    s["tau"] = torch.zeros(N, **f64)
    if c["kind"] == "lps":
        s["lps"] = torch.as_tensor(np.frombuffer(w["lps"].tobytes(), np.uint8).copy(), device=DEV)
    if c["kind"] == "trace":
        s["stats"] = torch.zeros((Z, 5), **f64)
        if c["constrained"]:
            s["realized"], s["ontime"] = torch.zeros(rows, **f64), torch.zeros(Z, **f64)
    if c["kind"] == "steps":
        # each arrival's values, in the buffers that the step reads
        ends = torch.cat([s["q_t_ms"][1:], s["q_t_ms"][-1:]]).contiguous()
        ctx.ttft_targets(s["q_prefill"], s["u_ms"], s["v"], out=s["tau"])
        s["arrivals"] = [
            dict(q_prefill=s["q_prefill"][i:i + 1], q_decode=s["q_decode"][i:i + 1],
                 t_ms=s["q_t_ms"][i:i + 1], t_next_ms=ends[i:i + 1], acc_row=s["acc"][i],
                 cost_row=s["cost"][i], w_cost=s["w_cost"],
                 w_lat=None if c["constrained"] else s["w_lat"],
                 tau_ms=s["tau"][i:i + 1] if c["constrained"] else None,
                 choice=s["choice"][0, i:i + 1], chosen_ttft=s["chosen"][0, i:i + 1],
                 utility=s["utility"][0, i:i + 1]) for i in range(N)]
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "online":
        lar.whatif_noalloc(
            s["params"], s["offsets"], s["rem_prefill"], s["rem_decode"], s["context"],
            s["clock_ms"], s["q_prefill"], 0.0, s["acc"], s["cost"], s["w_cost"], s["w_lat"],
            s["ttft"], s["choice"], s["status"], max_seqs_cap=c["max_seqs"],
            max_resident=max(1, c["resident"]), max_prompt=_max_prompt(c), flags=s["flags"],
            iters=s["iters"], chosen_ttft=s["chosen"], utility=s["utility"])
        return {k: s[k] for k in ("ttft", "iters", "choice", "chosen", "utility", "status")}
    ctx = s["ctx"]
    if c["kind"] in ("whatif", "lps"):
        out = ["ttft", "choice", "chosen", "utility"]
        if c["kind"] == "lps":
            ctx.estimate_lps(s["lps"], s["q_prefill"],
                             lar.LPS_VARIABILITY if c["variability"] else lar.LPS_POISSON,
                             ttft=s["ttft"])
        else:
            ctx.estimate(s["q_prefill"], 0.0, ttft=s["ttft"], iters=s["iters"])
            out.append("iters")
        if c["constrained"]:
            ctx.ttft_targets(s["q_prefill"], s["u_ms"], s["v"], out=s["tau"])
            ctx.route_constrained(s["ttft"], s["tau"], s["acc"], s["cost"], s["w_cost"],
                                  choice=s["choice"], chosen_ttft=s["chosen"],
                                  utility=s["utility"])
        else:
            ctx.route(s["ttft"], s["acc"], s["cost"], s["w_cost"], s["w_lat"],
                      choice=s["choice"], chosen_ttft=s["chosen"], utility=s["utility"])
        return {k: s[k] for k in out}
    ctx.reload_state()
    ctx.advance(s["t0"])
    out = ["choice", "chosen", "utility"]
    if c["kind"] == "steps":
        for a in s["arrivals"]:
            ctx.route_step(**a)
        return {k: s[k] for k in out}
    if c["constrained"]:
        ctx.ttft_targets(s["q_prefill"], s["u_ms"], s["v"], out=s["tau"])
        ctx.route_trace_constrained(s["q_prefill"], s["q_decode"], s["q_t_ms"], s["t_end"],
                                    s["tau"], s["acc"], s["cost"], s["w_cost"],
                                    choice=s["choice"], chosen_ttft=s["chosen"],
                                    utility=s["utility"], realized=s["realized"])
        ctx.ontime_utility(s["choice"], s["realized"], s["tau"], s["acc"], s["cost"],
                           s["w_cost"], out=s["ontime"])
        out += ["realized", "ontime"]
    else:
        ctx.route_trace(s["q_prefill"], s["q_decode"], s["q_t_ms"], s["t_end"], s["acc"],
                        s["cost"], s["w_cost"], s["w_lat"], choice=s["choice"],
                        chosen_ttft=s["chosen"], utility=s["utility"])
    ctx.stats(s["choice"], s["chosen"], s["acc"], s["cost"], s["w_cost"], out=s["stats"])
    return {k: s[k] for k in out + ["stats"]}


# ------------------------------------------------------------------ what a pass needs
def work(case):
    """Inputs read once, outputs written once; per (scenario, query, instance) estimate two
    batch times, their sum and the utility in binary64, and for the replay of a trace one
    batch time per estimate."""
    c = case
    I, N, Z, R = c["n_inst"], c["n_q"], c["n_scen"], c["resident"]
    cols = 4 if c["kind"] in ("steps", "trace") else I
    pairs = float(Z) * N * I
    b = 12.0 * I * R * Z + 16.0 * N * cols + 16.0 * N + 20.0 * Z * N
    if c["kind"] in ("online", "whatif", "lps"):
        b += 8.0 * pairs + (0.0 if c["kind"] == "lps" else 4.0 * pairs)
        return {"bytes": b, "flops": pairs * (8.0 if c["kind"] == "lps" else 23.0)}
    if c["constrained"] and c["kind"] == "trace":
        b += 8.0 * Z * N
    return {"bytes": b, "flops": 33.0 * pairs}


def tolerance(case):
    """The interface fixes every binary64 operation and its order: one right answer."""
    return "exact"


# ------------------------------------------------------------------ the reference
class _Queue:
    """One instance: decoding requests by the batch of their last token, the others in
    arrival order, batches as the scheduler forms them."""

    def __init__(self, k, budget, cap, reqs, clock):
        self.k, self.B, self.M, self.clock, self.g = k, budget, cap, clock, 0
        self.last, self.n_dec, self.c0 = {}, 0, 0
        self.pre, self.part = deque(), 0
        for rp, rd, cx in reqs:
            if rp == 0:
                self._decode(rd, cx)
            else:
                self.pre.append((rp, rd, cx))
                self.part += cx > 0

    def copy(self):
        q = object.__new__(_Queue)
        q.__dict__.update(self.__dict__)
        q.last, q.pre = dict(self.last), deque(self.pre)
        return q

    def _decode(self, rd, cx):
        n, c = self.last.get(self.g + rd, (0, 0))
        self.last[self.g + rd] = (n + 1, c + cx - self.g)
        self.n_dec, self.c0 = self.n_dec + 1, self.c0 + cx - self.g

    def time(self, P, D, C, A):
        a, b, c, d, e = self.k
        return (((a + b * P) + c * D) + d * C) + e * A

    def step(self):
        """One batch; returns its features and how many prefills it completed."""
        D, C = self.n_dec, self.c0 + self.n_dec * self.g
        left, free, P, A, done = self.B - D, self.M - D - self.part, 0, 0, []
        self.g += 1
        n, c = self.last.pop(self.g, (0, 0))
        self.n_dec, self.c0 = self.n_dec - n, self.c0 - c
        i = 0
        while i < len(self.pre) and left > 0 and (i < self.part or free > 0):
            rp, rd, cx = self.pre[i]
            ch = min(rp, left)
            P, A, left = P + ch, A + ch * cx + ch * (ch + 1) // 2, left - ch
            free -= i >= self.part
            self.pre[i] = (rp - ch, rd, cx + ch)
            i += 1
        for k in range(i):
            if self.pre[0][0]:
                break
            _, rd, cx = self.pre.popleft()
            done.append((rd, cx))
        self.part = max(0, self.part - len(done)) if i <= self.part else i - len(done)
        for rd, cx in done:
            self._decode(rd, cx)
        return (P, D, C, A), len(done)

    def replay(self, t):
        while (self.n_dec or self.pre) and self.clock < t:
            self.clock += self.time(*self.step()[0])
        if not (self.n_dec or self.pre) and self.clock < t:
            self.clock = t

    def tail_next(self):
        """Whether a request behind all others would get tokens in the next batch."""
        return (self.n_dec + len(self.pre) < self.M
                and self.n_dec + sum(r[0] for r in self.pre) < self.B)

    def estimates(self, p, t, prefill_batch):
        """TTFT and batches of prompts p (an array), each behind all others."""
        q, it, E = self.copy(), 0, self.clock
        need = sum(r[0] for r in q.pre)
        while not (q.n_dec + len(q.pre) < q.M and q.n_dec + need < q.B):
            f, _ = q.step()
            need -= f[0]
            E, it = E + q.time(*f), it + 1
        p = p.astype(np.int64)
        (P, D, C, A), _ = q.step()
        ch = np.minimum(p, self.B - D - P)
        E, it = E + self.time(P + ch, D, C, A + ch * (ch + 1) // 2), np.full(p.shape, it + 1)
        rem, cx = p - ch, ch
        live = rem > 0 if prefill_batch else np.ones(p.shape, bool)
        while live.any():
            (P, D, C, _), _ = q.step()
            ch = np.where(live & (rem > 0), np.minimum(rem, self.B - D), 0)
            first = live & (rem == 0)
            T = np.where(first, self.time(0, D + 1, C + cx, 0),
                         self.time(ch, D, C, ch * cx + ch * (ch + 1) // 2))
            E, it = np.where(live, E + T, E), it + live
            rem, cx = rem - ch, cx + ch
            live = live & ~first
            if prefill_batch:
                live = live & (rem > 0)
        return E - t, it


def _best(c, ttft, acc, cost, wc, wl, tau):
    """Route of rows of estimates: choice, TTFT there, utility there."""
    u = acc - wc * cost
    if c["constrained"]:
        ok = ttft <= tau[:, None]
        ch = np.where(ok.any(1), np.argmax(np.where(ok, u, -np.inf), 1), np.argmin(ttft, 1))
    else:
        ch = np.argmax(u - wl * ttft, 1)
    at = np.arange(len(ch))
    return ch.astype(np.int32), ttft[at, ch], u[at, ch]


def exact(case, seed):
    c = case
    # the plain simulation of longer traces, and of engines with limits, takes minutes
    if c["limits"] or (c["kind"] == "trace" and c["n_scen"] * c["n_q"] * c["n_inst"] > 20000):
        return None
    w = _pool(c, seed)
    I, N, Z = c["n_inst"], c["n_q"], c["n_scen"]
    acc, cost = w["acc"][:, w["col"]], w["cost"][:, w["col"]]
    lin = 155.0 + 3.5e-3 * w["q_prefill"]
    tau = np.minimum(np.maximum(w["u_ms"] + lin * w["v"], 150.0), 1120.0)
    if c["kind"] == "lps":
        L = w["lps"]
        mean = 1.0 / L["service_rate"]
        rho = L["arrival_rate"] * mean if c["variability"] else L["arrival_rate"] / L["service_rate"]
        power = rho.copy()
        for m in range(2, int(L["k"].max()) + 1):
            power = np.where(L["k"] >= m, power * rho, power)
        wait = ((L["ca2"] + L["cs2"]) / 2.0 * (power * mean / (1.0 - rho)) if c["variability"]
                else power / (L["service_rate"] - L["arrival_rate"]))
        ttft = (wait + w["q_prefill"][:, None] / L["prefill_rate"]) + L["decode_ms"]
        ch, t, u = _best(c, ttft, acc, cost, w["w_cost"][0], w["w_lat"][0], tau)
        return {"ttft": ttft[None], "choice": ch[None], "chosen": t[None], "utility": u[None]}
    reqs = np.stack([w["rem_prefill"], w["rem_decode"], w["context"]], 1).reshape(I, -1, 3).tolist()
    coef = np.stack([w[k] for k in "abcde"], 1).tolist()

    def pool():
        return [_Queue(coef[j], c["budget"], c["max_seqs"], reqs[j], 0.0) for j in range(I)]

    if c["kind"] in ("online", "whatif"):
        ttft, iters = np.zeros((N, I)), np.zeros((N, I), np.int32)
        for j, q in enumerate(pool()):
            ttft[:, j], iters[:, j] = q.estimates(w["q_prefill"], 0.0, c["prefill_batch"])
        ch, t, u = _best(c, ttft, acc, cost, w["w_cost"][0], w["w_lat"][0], tau)
        out = {"ttft": ttft[None], "iters": iters[None], "choice": ch[None], "chosen": t[None],
               "utility": u[None]}
        if c["kind"] == "online":
            out["status"] = None
        return out
    choice, chosen, util = np.zeros((Z, N), np.int32), np.zeros((Z, N)), np.zeros((Z, N))
    for z in range(Z):
        queues = pool()
        for q in queues:
            q.replay(w["q_t_ms"][0])
        for i in range(N):
            row = np.array([q.estimates(w["q_prefill"][i:i + 1], w["q_t_ms"][i],
                                        c["prefill_batch"])[0] for q in queues]).reshape(1, I)
            ch, t, u = _best(c, row, acc[i:i + 1], cost[i:i + 1], w["w_cost"][z], w["w_lat"][z],
                             tau[i:i + 1])
            choice[z, i], chosen[z, i], util[z, i] = ch[0], t[0], u[0]
            queues[ch[0]].pre.append((int(w["q_prefill"][i]), int(w["q_decode"][i]), 0))
            for q in queues:
                q.replay(w["q_t_ms"][min(i + 1, N - 1)])
    out = {"choice": choice, "chosen": chosen, "utility": util}
    if c["kind"] == "trace":
        out["stats"] = None
        if c["constrained"]:
            out["realized"], out["ontime"] = None, None
    return out
