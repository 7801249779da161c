// sfs_limits.h -- the wave batch engine under scheduler limits: a per-request
// prefill chunk cap H, a context limit X and a KV cache of K blocks of 2^sh tokens
// with recompute preemption (the system appendix lists context limits, KV-cache
// allocation and preemption among what the simulation follows; Sec. 2 describes
// paged KV caches and chunked prefill).
//
// The batch, per instance:
//   * running requests in list order: one decode token to each decoding one, then
//     min(rp, H, budget left) to each partial prefill;
//   * when a request's new blocks (ceil((cx + n) / S) - ceil(cx / S)) do not fit, the
//     last running request is preempted until they do or the request itself is
//     out: it returns its blocks (with those taken in this batch) and its tokens of
//     this batch, and becomes the first waiting request with rp = cx + rp, cx = 0;
//   * only in a batch without preemption: admissions in FCFS order while budget is
//     left, fewer than M run and the first chunk's blocks fit.
// The predicted decode is cut to X - (cx + rp) when a request enters, which ends it
// at the context limit.
//
// One wavefront owns one (scenario, instance) queue.  Because a preempted request
// becomes the first waiting one in place, the resident list never reorders: it is
// kept in arrival order, running requests first.  Its first KS*64 entries (KS*64 >= M,
// so every entry a batch can touch) sit in registers, list position s*64 + lane in
// slot s; the rest stay in the queue's HBM ring at index (head + position) mod rcap.
// (Every member function is inlined by force: past some size the compiler calls it
// instead, and the queue then lives in scratch memory.)
//
// A batch's decode tokens and new blocks are counted by ballots; the blocks held and
// the context of the decoding requests are carried from batch to batch, and in QScal
// from one kernel to the next.  Chunks and admissions are saturating DPP prefix sums
// over the rows that hold any; a batch that must preempt pops its victims one by one.
// Batches that repeat the one before are folded (LQueue::fold).  One wave per SIMD runs at
// the latency of its dependent instructions, so their number is the engine's time.  Against
// wave sums for every count and one lane walking lists in LDS to preempt (and without the
// shared and carried admission points of sfs_limits.hip), of 256 sequences each: 27
// instances x 243 queries 534 -> 339 us; 32 instances, 2500 queries 132 -> 91 ms; of 1024
// each, 32 x 100 1.59 -> 1.21 ms.
#pragma once

#include "sfs_device.h"

namespace lar {

// Limits on device, [I] each: chunk cap (0: none), KV blocks (0: unlimited),
// log2 of the block size, context limit (0: none).
struct DevLimits {
  const int32_t *H, *K, *sh, *X;
};

// LDS words per wave of the limits engine: five rows of KS*64 (compaction staging).
template <int KS>
constexpr int lim_lds_words() { return 5 * KS * kWave; }

struct LEnv {
  Coef k;
  int H;      // chunk cap, INT_MAX when none
  int K;      // KV blocks, 0 when unlimited
  int sh;     // log2 of the block size
  int X;      // context limit, 0 when none
  bool need_C, need_A;
  int32_t *r_rp, *r_rd, *r_cx, *r_seq;
  int rcap;
  int* lds;   // lim_lds_words<KS>() ints, 16-byte aligned
};

__device__ __forceinline__ LEnv make_lenv(const DevState& S, const DevParams& pr,
                                          const DevLimits& lm, int qid, int j, int* lds) {
  LEnv e;
  e.k = load_coef(pr, j);
  e.need_C = e.k.d != 0.0;
  e.need_A = e.k.e != 0.0;
  const int h = lm.H[j];
  e.H = h > 0 ? h : 0x7fffffff;
  e.K = lm.K[j];
  e.sh = lm.sh[j];
  e.X = lm.X[j];
  e.rcap = S.rcap;
  const int64_t rb = (int64_t)qid * S.rcap;
  e.r_rp = S.r_rp + rb; e.r_rd = S.r_rd + rb; e.r_cx = S.r_cx + rb; e.r_seq = S.r_seq + rb;
  e.lds = lds;
  return e;
}

// Blocks that hold x cached tokens.
// (x < 2^31 and a block is at most 65536 tokens, so the sum fits 32 unsigned bits.)
__device__ __forceinline__ int kv_blocks(int x, int sh) {
  return (int)(((uint32_t)x + (1u << sh) - 1u) >> sh);
}

// Predicted decode of a request entering with p prompt tokens: >= 1, cut to what the
// context limit leaves (0 when p does not fit it).
__device__ __forceinline__ int entry_decode(const LEnv& e, int p, int d) {
  d = d < 1 ? 1 : d;
  if (e.X > 0) {
    if (p >= e.X) return 0;
    if (d > e.X - p) d = e.X - p;
  }
  return d;
}

// First-token outputs of a replay that tracks routed queries (see the trace kernels).
struct LTrack {
  double* out;   // [N] first-token time per query of the running trace
  int tag0, N, reading;
};

struct LStep {
  double T;        // batch time
  bool last_dec;   // the last list entry received a decode token
  bool last_fill;  // the last list entry's prefill completed
  bool tail_ok;    // (TAIL steps) a new request at the tail could have been admitted
  bool same;       // the next batch serves the same requests the same tokens, unless one
                   // finishes or completes its prefill in it or the KV cache runs short
  int P, D;        // prefill and decode tokens
  int64_t C, A;    // context and attention features
};

// A set of window entries.  Up to four rows: the lanes of each row, wave-uniform (SGPRs,
// counted and scanned by the scalar unit).  More rows: one word per lane, bit s for row
// s.  Sixteen rows of wave-uniform masks, several sets at once, are more SGPRs than there
// are: spilled, they doubled the instructions of an estimate.  set() and rest() together
// give the number of entries.
template <int KS>
struct RowSet {
  static constexpr bool kWide = KS > 4;
  uint64_t m[kWide ? 1 : KS];
  uint32_t b;

  __device__ __forceinline__ RowSet() : b(0) {
#pragma unroll
    for (int s = 0; s < (kWide ? 1 : KS); ++s) m[s] = 0;
  }
  // Puts row s's entry of each lane with p in (once per row); its number, if counted here.
  __device__ __forceinline__ int set(int s, bool p) {
    if constexpr (kWide) {
      b |= p ? 1u << s : 0u;
      return 0;
    } else {
      m[s] = ballot(p);
      return popc(m[s]);
    }
  }
  // What set() left uncounted.
  __device__ __forceinline__ int rest() const {
    if constexpr (kWide) return ballot(b != 0) ? wave_sum32(__builtin_popcount(b)) : 0;
    else return 0;
  }
  // The number of entries.
  __device__ __forceinline__ int count() const {
    if constexpr (kWide) {
      return wave_sum32(__builtin_popcount(b));
    } else {
      int n = 0;
#pragma unroll
      for (int s = 0; s < KS; ++s) n += popc(m[s]);
      return n;
    }
  }
  // The lanes of row s (s wave-uniform).
  __device__ __forceinline__ uint64_t row(int s) const {
    if constexpr (kWide) {
      return ballot((b >> s) & 1u);
    } else {
      uint64_t x = 0;
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (k == s) x = m[k];
      return x;
    }
  }
  // Whether this lane's entry of row s is in the set.
  __device__ __forceinline__ int lane(int s) const {
    if constexpr (kWide) return (int)((b >> s) & 1u);
    else return (int)((m[s] >> lane_id()) & 1);
  }
  // Only the entries before list position n stay.
  __device__ __forceinline__ void clip(int n) {
    const int ln = lane_id();
    if constexpr (kWide) {
      const int rows = n > ln ? (n - ln + kWave - 1) >> 6 : 0;
      b &= (1u << rows) - 1u;
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s) m[s] &= ballot(s * kWave + ln < n);
    }
  }
};

template <int KS>
struct LQueue {
  int rp[KS], rd[KS], cx[KS], sq[KS], tg[KS];
  int nwin;      // window entries (positions 0 .. nwin-1)
  int n_list;    // list length
  int n_run;     // running prefix
  int head;      // ring index of list position 0
  int next_seq;
  int ntrk;      // tracked queries without a first token (tracking replays)
  int held;      // KV blocks of the running requests (K > 0; kept in QScal::pre_sum)
  int64_t csum;  // context of the decoding requests (d != 0; kept in QScal::c0sum)
  int nfin;      // batches to the first finish of a decoding request; 0: not known
  double clock;
  int64_t iters;
  // a query appended by an estimate to its private copy is written nowhere: while it
  // lies beyond the window it lives here, at list position n_list - 1
  bool vq;
  int vq_p, vq_d;

  template <bool TRK>
  __device__ __forceinline__ void fetch(const LEnv& e, const int32_t* tags, int s, int pos) {
    if (vq && pos == n_list - 1) {
      rp[s] = vq_p; rd[s] = vq_d; cx[s] = 0; sq[s] = next_seq - 1;
      if constexpr (TRK) tg[s] = -1;
      return;
    }
    int r = head + pos;
    if (r >= e.rcap) r -= e.rcap;
    rp[s] = e.r_rp[r]; rd[s] = e.r_rd[r]; cx[s] = e.r_cx[r]; sq[s] = e.r_seq[r];
    if constexpr (TRK) tg[s] = tags[r];
  }

  // Bring list positions nwin .. min(n_list, KS*64) - 1 into the window.
  template <bool TRK>
  __device__ __forceinline__ void refill(const LEnv& e, const int32_t* tags) {
    const int want = min(n_list, KS * kWave);
    if (nwin >= want) return;
    const int ln = lane_id();
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int pos = s * kWave + ln;
      if (pos >= nwin && pos < want) fetch<TRK>(e, tags, s, pos);
    }
    nwin = want;
  }

  template <bool TRK>
  __device__ __forceinline__ void load(const DevState& S, const LEnv& e, int qid,
                                       const int32_t* tags) {
    const QScal* q = S.sc + qid;
    n_list = uni(q->n_pre); n_run = uni(q->n_part); head = uni(q->head);
    next_seq = uni(q->next_seq);
    ntrk = TRK ? uni(q->ntrk) : 0;
    held = (int)uni64(q->pre_sum);
    csum = uni64(q->c0sum);
    nfin = 0;
    clock = q->clock;
    iters = uni64(q->iters);
    vq = false; vq_p = 0; vq_d = 0;
    nwin = 0;
#pragma unroll
    for (int s = 0; s < KS; ++s) { rp[s] = 0; rd[s] = 0; cx[s] = 0; sq[s] = 0; tg[s] = -1; }
    refill<TRK>(e, tags);
  }

  template <bool TRK>
  __device__ __forceinline__ void store(const DevState& S, const LEnv& e, int qid, int32_t* tags) const {
    const int ln = lane_id();
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int pos = s * kWave + ln;
      if (pos < nwin) {
        int r = head + pos;
        if (r >= e.rcap) r -= e.rcap;
        e.r_rp[r] = rp[s]; e.r_rd[r] = rd[s]; e.r_cx[r] = cx[s]; e.r_seq[r] = sq[s];
        if constexpr (TRK) tags[r] = tg[s];
      }
    }
    if (ln == 0) {
      QScal* q = S.sc + qid;
      q->g = 0; q->n_dec = 0; q->n_part = n_run; q->n_pre = n_list; q->head = head;
      q->next_seq = next_seq; q->c0sum = csum; q->pre_sum = held; q->clock = clock;
      q->iters = iters;
      if constexpr (TRK) { q->ntrk = ntrk; q->pend = 0; }
    }
    // the same wave loads this queue again later in the same kernel
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }

  __device__ __forceinline__ int waiting() const { return n_list - n_run; }

  // Append a waiting request at the tail (the caller checked p and the capacity).
  // real == false: an estimate's private copy; nothing is written to HBM.
  template <bool TRK>
  __device__ __forceinline__ void append(const LEnv& e, int p, int d, bool real, int32_t* tags, int tag) {
    const int ln = lane_id();
    const int pos = n_list;
    if (nwin == n_list && pos < KS * kWave) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (s * kWave + ln == pos) {
          rp[s] = p; rd[s] = d; cx[s] = 0; sq[s] = next_seq;
          if constexpr (TRK) tg[s] = tag;
        }
      nwin = pos + 1;
    } else if (real) {
      if (ln == 0) {
        int r = head + pos;
        if (r >= e.rcap) r -= e.rcap;
        e.r_rp[r] = p; e.r_rd[r] = d; e.r_cx[r] = 0; e.r_seq[r] = next_seq;
        if constexpr (TRK) tags[r] = tag;
      }
      // other lanes of this wave read the entry back on refill
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      vq = true; vq_p = p; vq_d = d;
    }
    n_list += 1;
    next_seq += 1;
  }

  // Copy to / from a what-if's admission point (a private copy: no arrival numbers).  It
  // is kept where the default engine keeps what this one has no use for: the first mcap
  // entries in the queue's decode slots, the scalars in its trajectory.  Entries from
  // position mcap on have never run (at most M <= mcap do, and positions only fall), so
  // the ring still holds them as they are.  pre: batches folded into the clock.
  __device__ __forceinline__ void to_front(const DevState& S, const DevTraj& f, int qid,
                                           int64_t pre) const {
    const int ln = lane_id();
    const int64_t o = (int64_t)qid * S.mcap;
    const int n = min(nwin, S.mcap);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int x = s * kWave + ln;
      if (x < n) { S.d_last[o + x] = rp[s]; S.d_cx0[o + x] = rd[s]; S.d_seq[o + x] = cx[s]; }
    }
    if (ln == 0) {
      f.P[qid] = n_list; f.left[qid] = n_run; f.pre[qid] = head;
      f.D[qid] = held; f.C[qid] = csum; f.A[qid] = pre; f.E[qid] = clock;
    }
  }
  __device__ __forceinline__ void from_front(const DevState& S, const LEnv& e, const DevTraj& f,
                                             int qid, int64_t* pre) {
    const int ln = lane_id();
    const int64_t o = (int64_t)qid * S.mcap;
    n_list = (int)uni64(f.P[qid]); n_run = uni(f.left[qid]); head = uni(f.pre[qid]);
    held = (int)uni64(f.D[qid]); csum = uni64(f.C[qid]); clock = f.E[qid];
    *pre = uni64(f.A[qid]);
    nfin = 0; next_seq = 0; ntrk = 0; iters = 0;
    vq = false; vq_p = 0; vq_d = 0;
    nwin = min(n_list, S.mcap);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int x = s * kWave + ln;
      const bool v = x < nwin;
      rp[s] = v ? S.d_last[o + x] : 0;
      rd[s] = v ? S.d_cx0[o + x] : 0;
      cx[s] = v ? S.d_seq[o + x] : 0;
      sq[s] = 0; tg[s] = -1;
    }
    refill<false>(e, nullptr);
  }

  // A private copy takes the request that the live queue has just appended: into the
  // window when it is that long; else the ring slot already holds it (a copy ahead of
  // its queue has as many requests fewer as its head is further).
  __device__ __forceinline__ void join(int p, int d) {
    const int ln = lane_id();
    const int pos = n_list;
    if (nwin == n_list && pos < KS * kWave) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (s * kWave + ln == pos) { rp[s] = p; rd[s] = d; cx[s] = 0; }
      nwin = pos + 1;
    }
    n_list += 1;
    next_seq += 1;
  }

  // The batch when it must preempt.  dm: the D decoding requests, nm: those of them that
  // need a new block; free0: free blocks.
  //
  // Decode tokens go in list order, and the victim is always the last running request,
  // so no request that has its token is a victim of this stage: the victims are the
  // fewest last ones whose blocks, with the free ones, give every remaining request
  // that needs a block one.  Then the partial prefills in list order, each popping
  // victims until its blocks fit or it is out itself; a victim that holds a decode
  // token of this batch returns it and the block it took.  On return chk holds the
  // chunks, n_run the new running count, D and P the tokens; the victims are waiting again
  // (rp, cx updated).
  // Admissions do not happen in such a batch.  Returns the free blocks.
  __device__ __forceinline__ int compose_preempt(const LEnv& e, const RowSet<KS>& dm,
                                                 const RowSet<KS>& nm, int free0,
                                                 int (&chk)[KS], int& D, int& P) {
    const int ln = lane_id();
    const int sh = e.sh;
    const int run0 = n_run;
    int run = n_run, freeb = free0, nn = nm.count();
    int hb[KS];   // blocks held
#pragma unroll
    for (int s = 0; s < KS; ++s) hb[s] = kv_blocks(cx[s], sh);
    // the row of the last running request, kept while victims are popped from it
    int v_row = -1, v_hb = 0;
    uint64_t v_dm = 0, v_nm = 0;
    auto pop = [&]() {
      run -= 1;
      if ((run >> 6) != v_row) {
        v_row = run >> 6;
#pragma unroll
        for (int k = 0; k < KS; ++k)
          if (k == v_row) v_hb = hb[k];
        v_dm = dm.row(v_row);
        v_nm = nm.row(v_row);
      }
      return run & (kWave - 1);
    };
    while (freeb < nn) {   // (a pass pops one request; with none left nn is 0)
      const int vl = pop();
      freeb += lane_read(v_hb, vl);
      nn -= (int)((v_nm >> vl) & 1);
      D -= (int)((v_dm >> vl) & 1);
    }
    freeb -= nn;
    int left = e.k.B - D;
    P = 0;
#pragma unroll 1
    for (int s = 0; s * kWave < run && left > 0; ++s) {
      uint64_t m = ballot(s * kWave + ln < run) & ~dm.row(s);   // partial prefills of this row
      if (m == 0) continue;
      int r_rp = 0, r_cx = 0, r_hb = 0;
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (k == s) { r_rp = rp[k]; r_cx = cx[k]; r_hb = hb[k]; }
      const int r_w = min(r_rp, e.H);
      const int r_nb = kv_blocks(r_cx + r_w, sh) - r_hb;
      int r_ch = 0;
      while (m) {
        const int l = __builtin_ctzll(m);
        m &= m - 1;
        const int r = s * kWave + l;
        int g = lane_read(r_w, l);
        int need = lane_read(r_nb, l);
        if (g > left) {
          g = left;
          need = kv_blocks(lane_read(r_cx, l) + g, sh) - lane_read(r_hb, l);
        }
        while (freeb < need && r < run) {
          const int vl = pop();
          const int tok = (int)((v_dm >> vl) & 1);
          freeb += lane_read(v_hb, vl) + (int)((v_nm >> vl) & 1);
          left += tok;
          D -= tok;
        }
        if (r >= run) break;
        r_ch = ln == l ? g : r_ch;
        freeb -= need;
        left -= g;
        P += g;
        if (left == 0) break;
      }
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (k == s) chk[k] = r_ch;
    }
    n_run = run;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int i = s * kWave + ln;
      if (i >= run && i < run0) { rp[s] += cx[s]; cx[s] = 0; }
    }
    return freeb;
  }

  // Remove the finished window entries fm keeping the order, and refill the window from
  // the ring.  LIVE: with the arrival numbers.
  template <bool TRK, bool LIVE>
  __device__ __forceinline__ void compact(const LEnv& e, const int32_t* tags, const RowSet<KS>& fm, int nf) {
    const int ln = lane_id();
    int* Srp = e.lds;
    int* Srd = Srp + KS * kWave;
    int* Scx = Srd + KS * kWave;
    int* Ssq = Scx + KS * kWave;
    int* Stg = Ssq + KS * kWave;
    // (rows before the first finished request stay as they are)
    int first = KS - 1;
#pragma unroll
    for (int s = KS - 2; s >= 0; --s)
      if (fm.row(s) != 0) first = s;
    int base = first * kWave;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s < first) continue;
      const bool keep = s * kWave + ln < nwin && !fm.lane(s);
      const uint64_t m = ballot(keep);
      if (keep) {
        const int dst = base + mbcnt(m);
        Srp[dst] = rp[s]; Srd[dst] = rd[s]; Scx[dst] = cx[s];
        if constexpr (LIVE) Ssq[dst] = sq[s];
        if constexpr (TRK) Stg[dst] = tg[s];
      }
      base += popc(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int nw = nwin - nf;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int pos = s * kWave + ln;
      if (s >= first && pos < nw) {
        rp[s] = Srp[pos]; rd[s] = Srd[pos]; cx[s] = Scx[pos];
        if constexpr (LIVE) sq[s] = Ssq[pos];
        if constexpr (TRK) tg[s] = Stg[pos];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    nwin = nw;
    n_list -= nf;
    n_run -= nf;
    head += nf;
    if (head >= e.rcap) head -= e.rcap;
    refill<TRK>(e, tags);
  }

  // One batch: compose, time, (TRK) first tokens at the batch end clk0 + T, apply.
  // Only the window rows that hold entries are visited (wave-uniform row count).
  // LIVE: a live queue, not a private copy (of those, only an estimate's reports on the
  // last list entry).  TAIL: also report whether a request
  // appended at the tail before this batch could have been admitted in it -- no
  // preemption, every waiting request admitted, a sequence slot, budget and a KV block
  // left -- which every admission needs, whatever the request's prompt; if it could,
  // the batch is not applied.  chk receives each entry's chunk.
  template <bool TRK, bool LIVE, bool TAIL>
  __device__ __forceinline__ LStep step(const LEnv& e, const int32_t* tags, double clk0,
                                        const LTrack* tk, int (&chk)[KS]) {
    constexpr bool EST = !LIVE && !TAIL;   // an estimate: reports on the last list entry
    const int ln = lane_id();
    const int sh = e.sh;
    const bool kv = e.K > 0;
    const int B = e.k.B, M = e.k.M;
    const int nrows = (nwin + kWave - 1) >> 6;
    const int lp = n_list - 1;
    // decoding requests and those of them that need a new block: the ones whose blocks
    // are full
    RowSet<KS> dm, nm;
    int D = 0, need = 0;
    const int smask = (1 << sh) - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      chk[s] = 0;
      if (s < nrows) {
        const bool dec = s * kWave + ln < n_run && rp[s] == 0;
        D += dm.set(s, dec);
        if (kv) need += nm.set(s, dec && (cx[s] & smask) == 0);
      }
    }
    D += dm.rest();
    need += nm.rest();
    const int L1 = B - D;
    int left = L1;
    // chunks of the partial prefills, in list order: min(rp, H, budget left).  When the
    // decode tokens alone run out of blocks the preempting pass gives them.
    const int room0 = kv ? e.K - held : 0;   // free blocks
    int preempted = kv && need > room0 ? 1 : 0;
    int P = 0;
    int64_t A = 0;
    if (n_run > D && left > 0 && !preempted) {
      // exclusive saturating prefix sums, row by row where there are any
      unsigned carry = 0;
      int nd = 0;
      int64_t a = 0;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s < nrows && carry < (unsigned)L1) {
          const uint64_t pm = ballot(s * kWave + ln < n_run) & ~dm.row(s);
          if (pm == 0) continue;
          const int want = (pm >> ln) & 1 ? min(min(rp[s], e.H), L1) : 0;
          const unsigned excl =
              min((unsigned)scan_sat(prev_lane(want), L1) + carry, (unsigned)L1);
          const int g = min(want, L1 - (int)excl);
          chk[s] = g;
          carry = (unsigned)uni(lane_last((int)min(excl + (unsigned)want, (unsigned)L1)));
          if (kv) nd += kv_blocks(cx[s] + g, sh) - kv_blocks(cx[s], sh);
          if (e.need_A) a += (int64_t)g * cx[s] + (int64_t)g * (g + 1) / 2;
        }
      }
      P = (int)carry;
      left = L1 - P;
      const int needp = kv ? wave_sum32(nd) : 0;
      if (e.need_A) A = wave_sum64(a);
      if (kv && need + needp > room0) preempted = 1;
      need += needp;
    }
    int room = room0 - need;   // blocks free after the running requests' (K > 0)
    int adm = 0;
    if (preempted) {
#pragma unroll
      for (int s = 0; s < KS; ++s) chk[s] = 0;
      room = compose_preempt(e, dm, nm, room0, chk, D, P);
      int64_t a = 0;
      dm.clip(n_run);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (e.need_A) a += (int64_t)chk[s] * cx[s] + (int64_t)chk[s] * (chk[s] + 1) / 2;
      }
      A = e.need_A ? wave_sum64(a) : 0;
      csum = e.need_C ? dec_context(dm) : 0;
    }
    if (!preempted && n_list > n_run && n_run < M && left > 0) {
      // admissions: a prefix of the waiting requests, cut where the budget, the
      // sequence cap or the blocks of a first chunk run out
      const int lim = min(nwin, M);
      const int left0 = left;
      int bcarry = 0, nblk = 0, pw = 0;
      unsigned carry = 0;
      int64_t a = 0;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s < nrows && (s + 1) * kWave > n_run) {
          const int i = s * kWave + ln;
          const bool wait = i >= n_run && i < lim;
          const int want = wait ? min(min(rp[s], e.H), left0) : 0;
          const unsigned excl =
              min((unsigned)scan_sat(prev_lane(want), left0) + carry, (unsigned)left0);
          const int g = min(want, left0 - (int)excl);
          carry = (unsigned)uni(lane_last((int)min(excl + (unsigned)want, (unsigned)left0)));
          const int need3 = (kv && g > 0) ? kv_blocks(g, sh) : 0;
          int cum = bcarry;
          if (kv) {
            cum += scan_add32(need3);
            bcarry = uni(lane_last(cum));
          }
          const bool ok = wait && g > 0 && (!kv || cum <= room);
          if (wait) chk[s] = ok ? g : 0;
          adm += popc(ballot(ok));
          nblk += ok ? need3 : 0;
          pw += ok ? g : 0;
          if (e.need_A && ok) a += (int64_t)g * (g + 1) / 2;
        }
      }
      const int pws = wave_sum32(pw);
      P += pws;
      left -= pws;
      if (kv) room -= wave_sum32(nblk);
      if (e.need_A) A += wave_sum64(a);
    }
    // features and time
    const int64_t C = csum;
    LStep o;
    o.T = batch_time(e.k, P, D, C, A);
    o.P = P; o.D = D; o.C = C; o.A = A;
    o.tail_ok = false;
    o.same = false;
    o.last_dec = false;
    o.last_fill = false;
    if constexpr (TAIL) {
      o.tail_ok = !preempted && adm == n_list - n_run && n_run + adm < M && left > 0 &&
                  (!kv || room >= 1);
      if (o.tail_ok) return o;
    }
    if constexpr (EST) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (s == (lp >> 6)) {
          const uint64_t fill = ballot(chk[s] > 0 && chk[s] == rp[s]);
          o.last_dec = ((dm.row(s) >> (lp & (kWave - 1))) & 1) != 0;
          o.last_fill = ((fill >> (lp & (kWave - 1))) & 1) != 0;
        }
    }
    if constexpr (TRK) {
      const double end = __dadd_rn(clk0, o.T);
      int hit = 0;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s < nrows) {
          const bool first = tk->reading == 1 ? (chk[s] > 0 && chk[s] == rp[s])
                                              : dm.lane(s) != 0;
          const int q = tg[s] - tk->tag0;
          if (first && tg[s] >= 0 && q >= 0 && q < tk->N) {
            tk->out[q] = end;
            tg[s] = -1;
            ++hit;
          }
        }
      }
      ntrk -= wave_sum32(hit);
    }
    // apply; decoding requests whose predicted decode is used up leave
    RowSet<KS> fm;
    int nf = 0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s < nrows) {
        const int d = dm.lane(s);
        cx[s] += d + chk[s];
        rd[s] -= d;
        rp[s] -= chk[s];
        nf += fm.set(s, d != 0 && rd[s] == 0);
      }
    }
    nf += fm.rest();
    int fillc = 0;       // requests whose prefill this batch completes: they decode next
    int64_t cfill = 0;   // their context
    if (P > 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s < nrows) {
          const uint64_t mf = ballot(chk[s] > 0 && rp[s] == 0);
          fillc += popc(mf);
          if (e.need_C) cfill += sum_lanes64(cx[s], mf);
        }
      }
    }
    n_run += adm;
    if (kv) held = e.K - room;
    csum += D + cfill;
    nfin = preempted || fillc > 0 || nfin <= 1 ? 0 : nfin - 1;
    if (nf > 0) {
      if constexpr (RowSet<KS>::kWide) {
        int h = 0;
        int64_t c = 0;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          h += fm.lane(s) ? kv_blocks(cx[s], sh) : 0;
          c += fm.lane(s) ? cx[s] : 0;
        }
        held -= kv ? wave_sum32(h) : 0;
        csum -= e.need_C ? wave_sum64(c) : 0;
      } else {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          uint64_t m = fm.row(s);
          while (m) {
            const int l = __builtin_ctzll(m);
            m &= m - 1;
            const int c = lane_read(cx[s], l);
            held -= kv ? kv_blocks(c, sh) : 0;
            csum -= c;
          }
        }
      }
      nfin = 0;
      compact<TRK, LIVE>(e, tags, fm, nf);
    } else {
      o.same = !preempted && adm == 0 && fillc == 0 && D + P > 0;
    }
    return o;
  }

  // Context of the decoding requests in dm.
  __device__ __forceinline__ int64_t dec_context(const RowSet<KS>& dm) const {
    int64_t c = 0;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      if (dm.lane(s)) c += cx[s];
    return wave_sum64(c);
  }

  // Runs the batches after a batch o (with o.same) that serve the same requests the same
  // tokens: no request is admitted, finishes, completes its prefill or is preempted in
  // them.  What held back the waiting requests in o still does (no slot or budget comes
  // free, the free blocks only get fewer).  They differ in C, which grows by D, and A,
  // which grows by the squared chunks.  Stops before a batch that starts at t_stop or
  // later; at most `most` batches.  Returns their number; E is the running clock.
  // Stretches are long where few requests run and a long prompt goes chunk by chunk;
  // their blocks are bounded from above, so near a full cache the batches are stepped.
  __device__ __forceinline__ int fold(const LEnv& e, const LStep& o, const int (&chk)[KS],
                                      double& E, double t_stop, int64_t most) {
    const int ln = lane_id();
    const int big = 0x7fffffff;
    const int64_t room = e.K - held;
    // (the blocks of one more batch, bounded as below: near a full cache nothing folds)
    if (e.K > 0 && (int64_t)o.D * (e.sh == 0 ? 2 : 1) + (o.P >> e.sh) > room) return 0;
    int np = 0;   // requests with a chunk
    if (o.P > 0) {
      uint64_t end = 0;   // those that complete their prefill in the next batch
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        np += popc(ballot(chk[s] > 0));
        end |= ballot(rp[s] <= chk[s] && chk[s] > 0);
      }
      if (end) return 0;
    }
    if (nfin == 0) {
      int x = big;
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (s * kWave + ln < n_run && rp[s] == 0) x = min(x, rd[s]);
      nfin = wave_min(x);
    }
    if (nfin < 3) return 0;
    int n = nfin == big ? big : nfin - 1;
    if (np > 0) {
      int x = big;
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (chk[s] > 0) x = min(x, (int)((unsigned)(rp[s] - 1) / (unsigned)chk[s]));
      n = min(n, wave_min(x));
    }
    if ((int64_t)n > most) n = (int)most;
    if (e.K > 0) {
      // each decoding request takes at most n / S + 1 blocks, each chunk sum at most one
      // more than its tokens fill
      const int64_t grow = (int64_t)o.D * ((n >> e.sh) + 1) + (((int64_t)o.P * n) >> e.sh) +
                           2 * (int64_t)np;
      if (grow > room) return 0;
    }
    if (n <= 0) return 0;
    int k = 0;
    if (!e.need_C && !e.need_A) {
      for (; k < n && E < t_stop; ++k) E = __dadd_rn(E, o.T);
    } else {
      int64_t C = o.C, A = o.A, gg = 0;   // gg: sum of the squared chunks
      if (e.need_A && np > 0) {
        int64_t x = 0;
#pragma unroll
        for (int s = 0; s < KS; ++s) x += (int64_t)chk[s] * chk[s];
        gg = wave_sum64(x);
      }
      for (; k < n && E < t_stop; ++k) {
        C += o.D;
        A += gg;
        E = __dadd_rn(E, batch_time(e.k, o.P, o.D, C, A));
      }
    }
    n = k;
    if (n == 0) return 0;
    int grew = 0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bool dec = s * kWave + ln < n_run && rp[s] == 0;
      const int c0 = cx[s];
      cx[s] += dec ? n : chk[s] * n;
      rd[s] -= dec ? n : 0;
      rp[s] -= dec ? 0 : chk[s] * n;
      if (dec || chk[s] > 0) grew += kv_blocks(cx[s], e.sh) - kv_blocks(c0, e.sh);
    }
    if (e.K > 0) held += wave_sum32(grew);
    csum += (int64_t)o.D * n;
    if (nfin != big) nfin -= n;
    return n;
  }
};

}  // namespace lar
