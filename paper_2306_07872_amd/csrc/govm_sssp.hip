// govm_sssp.hip -- single-source GOVM (Section 3.4, Algorithm 2) on gfx950.
//
// One step expands every row in the frontier delta (the rows whose distance
// changed in the previous step, Algorithm 2's `delta[j] = true and start != end`
// test): for each out-edge (u, v, w) it forms cand = alpha[u] (+) w and lowers
// alpha[v] to cand if cand is strictly smaller (with the `index != source`
// guard).  Every v lowered this step is recorded in beta; beta becomes the next
// delta and the loop stops after a step that lowers nothing (`ptr` false) or
// after n steps.
//
// Mapping to the device:
// - delta is the beta bitmap of the step, split by out-degree:
//     lane tier (deg <= t_lane): found by scanning the bitmap a block of words
//       at a time, 64 rows per wavefront; the wavefront's rows are concatenated
//       through an LDS prefix sum so each lane takes one edge;
//     wave tier (deg <= t_wave): also queued; one wavefront per row, lanes
//       stride the row;
//     workgroup tier: also queued, the row cut into t_chunk-edge chunks, one
//       workgroup each.
// - the lane whose atomicOr first sets a long row's bit appends it to the
//   right next-step queue (wavefront ballot + mbcnt prefix, gathered per
//   workgroup in LDS, one atomicAdd per tier and workgroup).  The scan clears
//   the bitmap of the current step, n/32 words per step.
// - Short rows far above the frontier's smallest distance may be left in the frontier
//   for a later step (see "deferral of far rows").
// - The relaxation reads alpha[v] with a plain load first (a stale value can
//   only be higher, so skipping on it is safe) and uses atomicMin only when
//   the candidate is smaller.  Order of updates inside a step does not matter:
//   the fixed point is unique (Section 3.5: the method does not care in which
//   order paths appear).
// - Step loop: one workgroup with the run's state in LDS (small graphs; several
//   sources, one workgroup each), one persistent launch with a grid barrier per
//   step, or a fixed number of launches of one step each (last-block bookkeeping)
//   followed by the persistent launch for the remaining steps.  The host never
//   waits.
#include <stdio.h>

#include <algorithm>

#include "govm_host.hpp"

namespace dawn {

// ---------------------------------------------------------------------------
// deferral of far rows
//
// A frontier row whose distance lies far above the smallest one is likely to be
// lowered again before its turn comes; expanding it now is work done twice.  On
// a 2048 x 2048 grid with fp32 weights every vertex used to be expanded 72
// times, on an ER graph 2.8 times.  So a step expands the frontier rows up to
// thr = M + delta (M: the smallest distance in the frontier) and leaves the
// others in the frontier: their bits go to a bitmap of their own, read and written
// by the lane that scans the word alone, so that the next step's bitmap holds the
// vertices that the step lowered and nothing else, and is counted as such.  A
// persistent launch keeps the words of a wavefront's first block in a register, on
// copies those of its next blocks in LDS, and the others in df (2048 x 2048 grid 38.1
// ms, 38.2 with the bits in the next step's bitmap, where they could not be told
// apart; 8 sources 106 ms, 117 with all but the first blocks in df).
// (Rows of the queued tiers are never left: a queue entry lasts one step.)  The
// fixed point does not depend on the order
// (distances are unique), and a row at M is always expanded.  With weights >= 0
// no later path can lower it, so every step settles a vertex and at most n
// steps are taken, as without deferral.  At unit weights all frontier rows have
// one distance and nothing is ever deferred.
//
// delta starts at nf_delta mean weights.  A step of more than nf_work edges
// keeps the chip busy: delta is halved, down to where it started.  A step of
// less than half as many costs little beyond its barrier: delta grows by a
// tenth, and doubles once there has been a busy step (the tail of a run).
// Rows are deferred only where degrees are even (grids, ER): on skewed graphs
// (R-MAT) the rows that matter are reached in few steps whose distances lie
// close together, and deferral only adds steps (a CPU model of R-MAT scale 18
// with lognormal weights: 15 steps instead of 12 for 1 % less work).  Measured:
// 2048 x 2048 grid 73.8 -> 38 ms (1187M -> 66M edges expanded), 64 ER graphs in
// one launch 11.8 -> 6.0 ms, together with the scan's order and kFresh below.
// ---------------------------------------------------------------------------
// SsCtl::converged of a run on copies that is not needed: the tile's is done.
constexpr int32_t kNoRun = 2;

constexpr uint32_t kNoKey = 0xFFFFFFFFu;  // above every distance that a row can have
constexpr float kNfDelta = 1.2f;
constexpr float kNfWork = 30000.f;
constexpr int kNfSamples = 4096;

// Copies (several sources in one run): a step holds the work of all.  (Three
// times as much: grid 1000 x 1021, k = 2 24.6 -> 30.8 ms, k = 8 37.4 -> 36.8.)
constexpr float copies_work(int k) { return k < 4 ? 1.f : (float)k / 4.f; }

template <int WT>
__device__ __forceinline__ constexpr bool nf_weights() {
  return WT == kWU32 || WT == kWF32;
}

// M + delta as a key, at least M (and not 0, which says "no frontier").
template <int WT>
__device__ __forceinline__ uint32_t nf_threshold(uint32_t M, float delta) {
  if constexpr (WT == kWF32) {
    const uint32_t t = __float_as_uint(__uint_as_float(M) + delta);
    return t > M ? t : M + 1u;
  } else {
    const uint32_t d = delta >= 4.0e9f ? kNoKey : delta < 1.f ? 1u : (uint32_t)delta;
    const uint32_t t = M + d;
    return t < M ? kNoKey : t;
  }
}

// The next step's threshold, from the frontier's smallest key and the edges of
// the step that ended.
template <int WT>
__device__ __forceinline__ void nf_advance(NfState& s, uint32_t M, float work, float busy) {
  if (!nf_weights<WT>() || s.floor == 0.f) return;
  if (work > busy) {
    s.delta = fmaxf(0.5f * s.delta, s.floor);
    s.big = 1u;
  } else if (work < 0.5f * busy && s.delta < 1e30f) {
    s.delta *= s.big ? 2.f : 1.1f;
  }
  s.thr = nf_threshold<WT>(M, s.delta);
}

// The run's smallest delta, or 0 for no deferral: from samples of the weights
// (their mean) and of the row lengths (deferral only where the mean length of an
// edge's row is at most four times the mean length of a row).  batch: and only
// where the weights are of one scale throughout, by the mean of their logarithms
// over runs of 64 samples (within a factor of 8): with one threshold for all, the
// graphs of larger weights would wait for the others to end, and the steps add up.
// 16 ER graphs of 240,000 edges, one with weights 100 times the others': 35 steps,
// 1077 us with deferral, 19 and 870 without.  even: whether those rules hold (also
// for weights that are never deferred).  Every thread of the workgroup (whole
// wavefronts) calls it and gets the results.
template <int WT>
__device__ float nf_floor(int64_t n, int64_t m, const int32_t* rowptr, const uint32_t* w,
                          int samples, bool batch, bool& even) {
  even = false;
  if (!rowptr || m < 1 || (nf_weights<WT>() && !w)) return 0.f;
  __shared__ float part[5][kMaxWavesPerBlock];
  __shared__ float s_floor;
  __shared__ bool s_even;
  float sw = 0.f, sd = 0.f, sd2 = 0.f, lo = 1e9f, hi = -1e9f;
  const int64_t ew = m > samples ? m / samples : 1, rw = n > samples ? n / samples : 1;
  const int ne = (int)(m < samples ? m : samples), nr = (int)(n < samples ? n : samples);
#pragma unroll 4
  for (int i = threadIdx.x; i < (nf_weights<WT>() ? ne : 0); i += blockDim.x)
    sw += WT == kWF32 ? __uint_as_float(w[i * ew]) : (float)w[i * ew];
  if (nf_weights<WT>() && batch) {
    const int ne64 = ne & ~63;
    for (int i = threadIdx.x; i < ne64; i += blockDim.x) {
      const uint32_t x = w[i * ew];
      float lg = x == 0u ? 0.f : WT == kWF32 ? (float)(x >> 23) : (float)(31 - __clz((int)x));
      const int cnt = __popcll(__ballot(x != 0u));
      for (int off = kWave / 2; off > 0; off >>= 1) lg += __shfl_xor(lg, off, kWave);
      if (cnt >= 16) {
        lo = fminf(lo, lg / (float)cnt);
        hi = fmaxf(hi, lg / (float)cnt);
      }
    }
  }
#pragma unroll 4
  for (int i = threadIdx.x; i < nr; i += blockDim.x) {
    const float d = (float)(rowptr[i * rw + 1] - rowptr[i * rw]);
    sd += d;
    sd2 += d * d;
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    sw += __shfl_xor(sw, off, kWave);
    sd += __shfl_xor(sd, off, kWave);
    sd2 += __shfl_xor(sd2, off, kWave);
  }
  const int wv = threadIdx.x / kWave;
  if (lane_id() == 0) {
    part[0][wv] = sw;
    part[1][wv] = sd;
    part[2][wv] = sd2;
    part[3][wv] = lo;
    part[4][wv] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sw = sd = sd2 = 0.f;
    for (int i = 0; i < (int)(blockDim.x / kWave); i++) {
      sw += part[0][i];
      sd += part[1][i];
      sd2 += part[2][i];
      lo = fminf(lo, part[3][i]);
      hi = fmaxf(hi, part[4][i]);
    }
    // sd2 / sd <= 4 * sd / nr
    s_even = sd2 * nr <= 4.f * sd * sd && hi - lo <= 3.f;
    s_floor = nf_weights<WT>() && s_even ? fmaxf(kNfDelta * (sw / ne), 1e-30f) : 0.f;
  }
  __syncthreads();
  even = s_even;
  return s_floor;
}

// ---------------------------------------------------------------------------
// init
// ---------------------------------------------------------------------------
// Step 0's counts and long rows: a seed's row in the queue of its tier.  (A
// short row is found by its bit.)  ALONE: the only seed, right after the same
// workgroup has cleared the control words with plain stores: no atomics.
template <bool ALONE>
__device__ __forceinline__ void ss_queue_seed(const SsArgs& A, int64_t s) {
  SsCtl* C = A.ctl;
  const int32_t start = A.rowptr[s], deg = A.rowptr[s + 1] - start;
  if (deg == 0) return;
  const bool wave = deg > A.t_lane && deg <= A.t_wave, wg = deg > A.t_lane && !wave;
  const uint32_t nch = wg ? (uint32_t)((deg + A.t_chunk - 1) / A.t_chunk) : 0u;
  uint32_t p = 0u;
  if (ALONE) {
    C->ctr.fedges[0] = (unsigned long long)deg;
    C->ctr.frows[0] = 1ull;
    if (wave) C->cnt[0][1].v = 1u;
    if (wg) C->cnt[0][2].v = nch;
  } else {
    atomicAdd(&C->ctr.fedges[0], (unsigned long long)deg);
    atomicAdd(&C->ctr.frows[0], 1ull);
    if (wave) p = atomicAdd(&C->cnt[0][1].v, 1u);
    if (wg) p = atomicAdd(&C->cnt[0][2].v, nch);
  }
  if (wave) A.qwave[0][p] = (int32_t)s;
  for (uint32_t c = 0; c < nch; c++) {
    const int32_t off = (int32_t)c * A.t_chunk;
    if (p + c < A.cap_wg)
      A.qwg[0][p + c] = make_int4((int32_t)s, start + off, min(A.t_chunk, deg - off), c == 0);
  }
}

// hv (may be null): bit v set when row v has more than t_lane edges, the rows
// that steps take from the wave and workgroup queues rather than from the bitmap.
// seed (or -1): the run's only source, placed here, which saves the launch that
// places several (with the run's report in its last launch: ER n = 40,000 272 ->
// 254 us, R-MAT scale 16 376 -> 366, scale 20 802 -> 789).
// batch: the run is a batch's.  dist: null when the distances are there already.
// over (or null): a word that says whether nothing is left to run.
template <int WT>
__global__ void ss_fill_kernel(uint32_t* dist, int64_t n, uint32_t* bm0, uint32_t* bm1,
                               int64_t nwords, SsCtl* ctl, const int32_t* rowptr, uint32_t* hv,
                               int32_t t_lane, const uint32_t* w, int64_t m, int32_t n1,
                               int64_t seed, bool batch, const uint32_t* over, SsArgs A) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (over && *over) {  // (written by an earlier launch)
    if (tid == 0) {
      ctl->converged = kNoRun;
      ctl->done = 1u;
    }
    return;
  }
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  if (dist)
    for (int64_t i = tid; i < n; i += stride) dist[i] = i == seed ? zero_key<WT>() : inf_key<WT>();
  for (int64_t i = tid; i < nwords; i += stride) {
    bm0[i] = seed >= 0 && i == seed >> 5 ? 1u << (seed & 31) : 0u;
    bm1[i] = 0;
    A.df[i] = 0;
  }
  if (hv) {
    // a wavefront per 64 vertices: the ballot's halves are two bitmap words
    // (blockDim and the grid's thread count are multiples of 64)
    const int lane = lane_id();
    for (int64_t v0 = tid - lane; v0 < n; v0 += stride) {
      const int64_t v = v0 + lane;
      const uint32_t u = (uint32_t)v % (uint32_t)n1;  // (the row of a copy's vertex)
      const bool heavy = v < n && rowptr[u + 1] - rowptr[u] > t_lane;
      const unsigned long long b = __ballot(heavy);
      const int64_t wi = v0 / 32 + (lane >> 5);
      if ((lane & 31) == 0 && wi < nwords) hv[wi] = (uint32_t)(b >> (lane & 32));
    }
  }
  // the barrier's slots, then the other control words (one workgroup, which
  // also takes the run's samples)
  for (int64_t i = tid; i < kMaxGrid; i += stride) ctl->bar.slot[i] = 0ull;
  if (blockIdx.x == 0) {
    uint32_t* c = reinterpret_cast<uint32_t*>(ctl);
    for (int i = threadIdx.x; i < (int)(offsetof(SsCtl, bar.slot) / 4); i += blockDim.x) c[i] = 0;
    __syncthreads();
    if (threadIdx.x < kRot) ctl->minp[threadIdx.x].v = kNoKey;
    bool even;
    const float floor = nf_floor<WT>(n1, m, rowptr, w, kNfSamples, batch, even);
    if (threadIdx.x == 0) {
      ctl->even = even;
      ctl->nf = NfState{kNoKey, floor, floor, 0u};
      if (seed >= 0) ss_queue_seed<true>(A, seed);
    }
  }
}

// CSR checks (tuning field `validate`): rowptr[0] == 0, rowptr[n] == m,
// non-decreasing rows, column ids in range, fp32 weights finite with the sign
// bit clear.  A failure marks the run done with converged = -1.
__global__ void ss_validate_kernel(const int32_t* rowptr, const int32_t* colidx,
                                   const uint32_t* w, int32_t n, int32_t m, int32_t is_f32,
                                   uint32_t* done, int32_t* converged) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  if (tid == 0) bad = rowptr[0] != 0 || rowptr[n] != m;
  for (int64_t i = tid; i < n; i += stride) bad |= rowptr[i + 1] < rowptr[i];
  for (int64_t e = tid; e < m; e += stride) {
    const int32_t v = colidx[e];
    bad |= v < 0 || v >= n;
    if (is_f32) bad |= (w[e] & 0x80000000u) != 0 || (w[e] & 0x7F800000u) == 0x7F800000u;
  }
  if (bad) {
    st_agent_i(converged, -1);
    st_agent(done, 1u);
  }
}

// Put the seeds in step 0's delta: alpha[s] = 0, beta bit set, row queued.
template <int WT>
__global__ void ss_seed_kernel(SsArgs A, const int32_t* sources, const int64_t* voff,
                               int32_t count, int32_t single) {
  SsCtl* C = A.ctl;
  if (ld_agent(&C->done)) return;
  for (int j = threadIdx.x; j < count; j += blockDim.x) {
    int64_t s = sources ? (int64_t)sources[j] : (int64_t)single;
    if (voff) s += voff[j];
    A.dist[s] = zero_key<WT>();
    const uint32_t bit = 1u << (s & 31);
    const uint32_t old = atomicOr(&A.bm[0][s >> 5], bit);
    if (old & bit) continue;  // duplicate seed
    ss_queue_seed<false>(A, s);
  }
}

// int32 weights: keys back to int32 values (INF -> INT32_MAX).
__global__ void ss_decode_i32_kernel(uint32_t* dist, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    dist[i] ^= 0x80000000u;
}

// The end of a run's bookkeeping (one thread): the run's status (see
// run_status; with int32 weights a path sum that left the int32 range also
// makes the run count as not converged) and counters go to `info`, or, when
// the caller gave none, a status other than 1 goes to the run-status latch.
template <int WT>
__device__ void ss_report(SsCtl* C, dawn_run_info* info, uint32_t* latch) {
  int32_t conv = run_status(ld_agent_i(&C->converged), ld_agent(&C->abort), ld_agent(&C->overflow));
  if (WT == kWI32 && conv == 1 && ld_agent(&C->negfloor)) conv = 0;
  if (!info) {
    latch_status(latch, conv);
    return;
  }
  const unsigned long long fe = ld_agent64(&C->ctr.fe);
  const unsigned long long es = ld_agent64(&C->ctr.es);
  const unsigned long long im = ld_agent64(&C->ctr.im);
  info->steps = (int32_t)ld_agent(&C->step);
  info->converged = conv;
  info->frontier_entries = (int64_t)fe;
  info->edges_scanned = (int64_t)es;
  info->improvements = (int64_t)im;
  info->union_rows = (int64_t)(fe + C->u_rows);  // (written by an earlier launch)
  info->union_edges = (int64_t)(es + C->u_edges);
}

// ---------------------------------------------------------------------------
// one step
// ---------------------------------------------------------------------------

// Next-frontier entries found by a workgroup are gathered in LDS and written
// to the global queues once at the end of the step with one atomicAdd per
// tier per workgroup (a queue that fills up spills straight to global memory).
constexpr int kLdsQWave = 512;
constexpr int kUnroll = 4;      // edges in flight per lane (wave and workgroup tiers)
constexpr int kUnrollLane = 4;  // edges in flight per lane (lane tier)

// Position of the set bit of x that has r set bits below it (x has more than
// r set bits): a binary search on the population counts of its low halves.
__device__ __forceinline__ int nth_set_bit(uint32_t x, int r) {
  int pos = 0;
#pragma unroll
  for (int s = 16; s >= 1; s >>= 1) {
    const int lo = __popc(x & ((1u << s) - 1u));
    if (r >= lo) {
      r -= lo;
      x >>= s;
      pos += s;
    }
  }
  return pos;
}

// Rows of a block of bitmap words, 64 at a time: lane l holds a word; the set
// bits of the words, in order, are dealt to the lanes as the rows' edges are.
struct ScanRows {
  uint2 word[kWave];  // by rank among the non-empty words: {bits, bits before | lane << 16}
  DealMarks<kWave * 32> mk;
};

// f(has, o, bit): this lane's row is bit `bit` of the word lane o holds.
// Reached by the whole wavefront; f is called once per 64 rows.
template <typename F>
__device__ __forceinline__ void scan_rows(ScanRows& st, uint32_t bits, F&& f) {
  const int lane = lane_id();
  const int cnt = __popc(bits);
  const int incl = wave_incl_scan(cnt);
  const int nrows = __builtin_amdgcn_readlane(incl, kWave - 1);
  if (nrows == 0) return;
  const int excl = incl - cnt;
  const unsigned long long nz = __ballot(cnt > 0);
  if (cnt > 0)
    st.word[lanes_below(nz)] = make_uint2(bits, (uint32_t)excl | ((uint32_t)lane << 16));
  deal_mark(st.mk, excl, cnt, 0);
  int before = 0;
  for (int r0 = 0; r0 < nrows; r0 += kWave) {
    const uint2 w = st.word[deal_rank(st.mk, r0, before)];
    const bool has = r0 + lane < nrows;
    const int bit = has ? nth_set_bit(w.x, r0 + lane - (int)(w.y & 0xFFFFu)) : 0;
    f(has, (int)(w.y >> 16), bit);
  }
  wave_lds_sync();
}

struct SsShared {
  DealRows<4096, true> rows[kMaxWavesPerBlock];  // lane-tier batch
  ScanRows scan[kMaxWavesPerBlock];        // bitmap block
  uint32_t def[kMaxWavesPerBlock][kWave];  // rows left for later, by word of the block
  int32_t qw[kLdsQWave];
  uint32_t nqw, upd, gbase_w;
  uint32_t minp, work, heavy;  // smallest key left in the frontier, edges expanded, rows queued
};

// How a step treats its frontier: kAll, every row is expanded; kNear, rows above
// the threshold are left in the frontier; kFresh, as kNear, for steps of few
// edges whose launch has not dropped stale cache lines (the targets' distances
// are read at agent scope).
constexpr int kAll = 0, kNear = 1, kFresh = 2;

// What a lane has seen of a step: the smallest key that it put or left in the
// next frontier, and the edges of the rows that it held.
struct StepSeen {
  uint32_t minp = kNoKey, work = 0u;
};

// Push `v` for lanes with `pred` into the workgroup's LDS queue; lanes past
// its capacity go to the global queue.  Reached by the whole wavefront.
__device__ __forceinline__ void block_push(bool pred, int32_t v, int32_t* sq, uint32_t* sn,
                                           uint32_t lcap, int32_t* gq, uint32_t* gcnt,
                                           uint32_t gcap, uint32_t* overflow) {
  const unsigned long long b = __ballot(pred);
  if (b == 0) return;
  const int leader = __ffsll((long long)b) - 1;
  uint32_t base = 0;
  if (lane_id() == leader) base = atomicAdd(sn, (uint32_t)__popcll(b));
  base = __shfl(base, leader, kWave);
  const uint32_t pos = base + lanes_below(b);
  const bool spill = pred && pos >= lcap;
  if (pred && !spill) sq[pos] = v;
  wave_push(spill, v, gq, gcnt, gcap, overflow);
}

// Lanes with `pred` append row v (edges [start, start + deg), deg > t_lane) to
// the next step's queue of its tier.  Reached by the whole wavefront.
__device__ __forceinline__ void ss_queue_row(const SsArgs& A, bool pred, int32_t v, int32_t start,
                                             int32_t deg, int nxt, int rn, SsShared& sh) {
  SsCtl* C = A.ctl;
  if (__ballot(pred) == 0ull) return;
  block_push(pred && deg <= A.t_wave, v, sh.qw, &sh.nqw, kLdsQWave, A.qwave[nxt],
             &C->cnt[rn][1].v, A.cap_v, &C->overflow);
  if (pred) sh.heavy = 1u;
  if (pred && deg > A.t_wave) {
    const uint32_t nch = (uint32_t)((deg + A.t_chunk - 1) / A.t_chunk);
    const uint32_t base = atomicAdd(&C->cnt[rn][2].v, nch);
    for (uint32_t c = 0; c < nch; c++) {
      const int32_t off = (int32_t)c * A.t_chunk;
      if (base + c < A.cap_wg)
        st_queue4(&A.qwg[nxt][base + c], v, start + off, min(A.t_chunk, deg - off), c == 0);
      else
        atomicOr(&C->overflow, 1u);
    }
  }
}

// Record improvements of alpha[v[i]] (lanes with imp[i]): the ptr flag, the
// beta bitmap, and for the first setter of a bit whose row has more than
// t_lane edges, the next-step queue of its degree tier (shorter rows are found
// by the next step's bitmap scan).  kFresh: hvw holds the targets' long-row words.
// Reached by the whole wavefront.  CNT: also count the vertices lowered (else
// the next step's scan does) and the next frontier's rows and out-edges (the
// pull decision of the next step).
// off: what the copy adds to vertex ids (v has it added).
template <int WT, int U, bool CNT, int MODE>
__device__ __forceinline__ void ss_enqueue(const SsArgs& A, const bool (&imp)[U],
                                           const int32_t (&v)[U], const int32_t (&off)[U],
                                           const uint32_t (&cand)[U],
                                           const uint32_t (&hvw)[U], int nxt, int rn, Acc& acc,
                                           SsShared& sh, StepSeen& seen) {
  bool any = false;
#pragma unroll
  for (int i = 0; i < U; i++) {
    any |= imp[i];
    if (MODE != kAll && imp[i]) seen.minp = min(seen.minp, cand[i]);
  }
  if (__ballot(any) == 0) return;
  SsCtl* C = A.ctl;
  if (any) sh.upd = 1u;
  bool newv[U];  // first setters that have to queue the row (CNT: all first setters)
#pragma unroll
  for (int i = 0; i < U; i++) newv[i] = false;
  if constexpr (MODE == kFresh) {
    // the long-row words are there: a short row needs no answer, and the
    // atomic is not waited for
#pragma unroll
    for (int i = 0; i < U; i++) {
      if (imp[i]) {
        uint32_t* word = &A.bm[nxt][v[i] >> 5];
        const uint32_t bit = 1u << (v[i] & 31);
        if (hvw[i] & bit) newv[i] = (atomicOr(word, bit) & bit) == 0u;
        else atomicOr(word, bit);
      }
    }
  } else {
    // the long-row words of the few improved targets, loaded beside the test-and-set
    uint32_t hw[U];
#pragma unroll
    for (int i = 0; i < U; i++) hw[i] = imp[i] && !CNT ? A.hv[v[i] >> 5] : ~0u;
#pragma unroll
    for (int i = 0; i < U; i++) {
      if (imp[i]) {
        const uint32_t bit = 1u << (v[i] & 31);
        newv[i] = (atomicOr(&A.bm[nxt][v[i] >> 5], bit) & bit) == 0u;
      }
    }
#pragma unroll
    for (int i = 0; i < U; i++) newv[i] = newv[i] && ((hw[i] >> (v[i] & 31)) & 1u);
  }
#pragma unroll
  for (int i = 0; i < U; i++) {
    if (imp[i]) {
      // unit weights: every candidate of a step is the same level (the
      // frontier holds exactly the vertices of the previous level), so the
      // writers agree and a plain store will do
      if constexpr (WT == kWUNIT) st_agent(&A.dist[v[i]], cand[i]);
      else atomicMin(&A.dist[v[i]], cand[i]);  // result unused: not waited for
    }
  }
  if (CNT) {
#pragma unroll
    for (int i = 0; i < U; i++)
      if (newv[i]) acc.im += 1;  // a vertex lowered in this step counts once
  }
  int32_t start[U], deg[U];
#pragma unroll
  for (int i = 0; i < U; i++) {
    start[i] = 0;
    deg[i] = 0;
    if (newv[i]) {
      start[i] = A.rowptr[v[i] - off[i]];
      deg[i] = A.rowptr[v[i] - off[i] + 1] - start[i];
      if (CNT && deg[i] > 0) {
        acc.sa += (unsigned long long)deg[i];  // the next frontier's out-edges
        acc.se += 1;                           // and rows
      }
    }
  }
#pragma unroll
  for (int i = 0; i < U; i++)
    ss_queue_row(A, newv[i] && deg[i] > A.t_lane, v[i], start[i], deg[i], nxt, rn, sh);
}

// Candidates and the plain-load pre-check only, for ss_enqueue: it issues the
// next-frontier test-and-set first and the non-returning atomicMin after it,
// so waiting for the test-and-set does not wait for the atomicMin too (gfx9's
// vector-memory counter retires in order).  A candidate that passes the
// pre-check but loses to a lower value written in the same step only sets a
// bit that the writer of that value sets as well.  kFresh: read the targets'
// distances at agent scope (no cache line from before the step may serve them).
template <int WT, int U, int MODE>
__device__ __forceinline__ void ss_relax_pre(const SsArgs& A, const int32_t (&e)[U],
                                             const bool (&valid)[U], const uint32_t (&du)[U],
                                             const int32_t (&off)[U], bool (&imp)[U],
                                             int32_t (&v)[U], uint32_t (&cand)[U],
                                             uint32_t (&hvw)[U]) {
#pragma unroll
  for (int i = 0; i < U; i++) {
    v[i] = 0;
    cand[i] = 0u;
    if (valid[i]) {
      v[i] = A.colidx[e[i]] + off[i];
      cand[i] = relax_key<WT>(du[i], WT == kWUNIT ? 1u : A.w[e[i]]);
      if constexpr (WT == kWI32)
        if (cand[i] == 0u) atomicOr(&A.ctl->negfloor, 1u);  // sum left the int32 range
    }
  }
  uint32_t cur[U];
  if constexpr (MODE == kFresh) {
    // the long-row words are loaded beside the distances
#pragma unroll
    for (int i = 0; i < U; i++) hvw[i] = valid[i] ? A.hv[v[i] >> 5] : 0u;
#pragma unroll
    for (int i = 0; i < U; i++) cur[i] = valid[i] ? ld_agent(&A.dist[v[i]]) : 0u;
  } else {
#pragma unroll
    for (int i = 0; i < U; i++) cur[i] = valid[i] ? A.dist[v[i]] : 0u;
  }
#pragma unroll
  for (int i = 0; i < U; i++) imp[i] = valid[i] && cand[i] < cur[i] && v[i] != A.src;
}

// Minimum over the 16 lanes of this lane's row (DPP row rotations).
__device__ __forceinline__ uint32_t row16_min(uint32_t x) {
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, false));
  return x;
}

// A pull step (step launches on a dense frontier): each 16-lane group takes
// one in-edge chunk of a target v from the reverse graph and relaxes the
// in-edges whose source is in the step's frontier (its bit in the current
// bitmap), 16 at a time; the best candidate goes through the same enqueue as
// a push step's.  The (edge) relaxations are exactly the push step's; no
// atomicMin per edge, one per improved target (a target whose in-edges span
// several chunks may be improved from each).  The current bitmap is read
// throughout and not cleared here (the step's last workgroup clears it).
template <int WT, int MODE>
__device__ __forceinline__ void ss_pull(const SsArgs& A, int cur, int nxt, int rn, uint32_t gw,
                                        uint32_t nwv, Acc& acc, SsShared& sh,
                                        StepSeen& seen) {
  const int lane = lane_id(), g = lane >> 4, j16 = lane & 15;
  const uint32_t nch = (uint32_t)min((long long)A.T.hdr->nchunks, (long long)A.T.cap_chunks);
  const uint32_t* fb = A.bm[cur];
  for (uint32_t c0 = gw * 4; c0 < nch; c0 += nwv * 4) {
    const uint32_t c = c0 + (uint32_t)g;
    const bool cok = c < nch;
    const int4 ch = cok ? A.T.chunks[c] : make_int4(0, 0, 0, 0);
    const int32_t v = ch.x, start = ch.y, len = ch.z;
    uint32_t best = inf_key<WT>();
    for (int32_t b = 0; __ballot(cok && b < len) != 0ull; b += 16) {
      if (cok && b + j16 < len) {
        const int32_t u = A.T.colidx[start + b + j16];
        if ((fb[u >> 5] >> (u & 31)) & 1u) {
          const uint32_t w = WT == kWUNIT ? 1u : A.T.w[start + b + j16];
          const uint32_t cand = relax_key<WT>(A.dist[u], w);
          if constexpr (WT == kWI32)
            if (cand == 0u) atomicOr(&A.ctl->negfloor, 1u);  // sum left the int32 range
          best = min(best, cand);
          acc.es += 1;
        }
      }
    }
    best = row16_min(best);
    bool imp[1] = {cok && j16 == 0 && v != A.src && best < A.dist[v]};
    const int32_t vv[1] = {v}, off[1] = {0};
    const uint32_t cc[1] = {best}, hvw[1] = {0u};
    ss_enqueue<WT, 1, true, MODE>(A, imp, vv, off, cc, hvw, nxt, rn, acc, sh, seen);
  }
}

// With skipping (tuning ss_skip): a frontier row whose distance another row
// lowered again during this step is already marked for the next step, where
// it is expanded with a value at least as low; expanding it now as well would
// only repeat that work.  Its current-bitmap word is still cleared.
__device__ __forceinline__ bool ss_skip_row(const SsArgs& A, int nxt, int32_t u) {
  return A.skip && ((ld_agent(&A.bm[nxt][u >> 5]) >> (u & 31)) & 1u);
}

// What the copy of vertex u adds to vertex ids (0 without copies).
template <bool COPIES>
__device__ __forceinline__ int32_t copy_off(const SsArgs& A, int32_t u) {
  if constexpr (!COPIES) return 0;
  // floor(2^32 / n1) gives the quotient or one less
  int32_t off = (int32_t)(__umulhi((uint32_t)u, A.inv1) * (uint32_t)A.n1);
  if (u - off >= A.n1) off += A.n1;
  return off;
}

// Returns true when the step was a pull step.
// thr: short rows above it are left in the frontier (not kAll).  count: the scan
// counts the vertices that the previous step lowered.
// PULL: pull steps may run (step launches with a reverse graph); the push-only
// instance keeps none of their code.
// The step's queue counts (lane, wave, workgroup-chunk tiers); read at the
// start of a step launch, or by the persistent kernel together with the
// previous step's update flag, right after the barrier that ends that step.
struct SsCounts {
  uint32_t w, g;  // wave-tier rows, workgroup-tier chunks
};

__device__ __forceinline__ SsCounts ss_counts(const SsArgs& A, uint32_t step) {
  const SsCtl* C = A.ctl;
  const int rc = step % kRot;
  // Entries past a queue's capacity were never written (the pushes that
  // counted them set the overflow flag, and the run reports -3), so the
  // counts are read up to the capacities only.
  return SsCounts{min(ld_agent(&C->cnt[rc][1].v), A.cap_v), min(ld_agent(&C->cnt[rc][2].v), A.cap_wg)};
}

// How the scan's blocks fall on the wavefronts.  Groups of 1 << gs neighbouring
// words go to the wavefronts in turn (four words, 128 vertices, or fewer when that
// leaves wavefronts without a group; up to 64 words a wavefront at a time), so a
// run of frontier rows is shared by many of them.  With blocks of 32 words per
// wavefront the slowest workgroup took 13 us of a 15 us step on a 2048 x 2048
// grid, against 5 on average.
struct ScanSplit {
  int64_t nwords, span, first;  // words; between a lane's neighbours' groups; of the wavefront's first group
  int gs;
  __device__ __forceinline__ ScanSplit(int32_t n, uint32_t gw, uint32_t nwv)
      : nwords(((int64_t)n + 31) / 32), gs(2) {
    while (gs > 0 && (nwords >> gs) < (int64_t)nwv) gs--;
    span = (int64_t)nwv << gs;
    first = (int64_t)gw << gs;
  }
  // the word of lane l in the block that starts at w0
  __device__ __forceinline__ int64_t word(int64_t w0, int l) const {
    return w0 + first + (l & ((1 << gs) - 1)) + (l >> gs) * span;
  }
  __device__ __forceinline__ int64_t block() const { return span << (6 - gs); }
};

// left0: the rows left for later of this lane's word in the wavefront's first block;
// those of the other blocks are in df, with COPIES of the first nheld of them in
// `held` (LDS).
template <int WT, bool PULL, int MODE, bool COPIES>
__device__ __forceinline__ bool ss_step(const SsArgs& A, uint32_t step, uint32_t gb, uint32_t nb, Acc& acc,
                        SsShared& sh, SsCounts counts, uint32_t thr, bool count, uint32_t& left0,
                        uint32_t* held = nullptr, int nheld = 0) {
  constexpr bool NF = MODE != kAll;
  StepSeen seen;
  const int cur = step & 1, nxt = cur ^ 1;
  const int rc = step % kRot, rn = (step + 1) % kRot;
  SsCtl* C = A.ctl;
  const int lane = lane_id(), wave = threadIdx.x >> 6, W = blockDim.x >> 6;
  // wave-major: consecutive work items go to different workgroups, so a
  // frontier smaller than the grid's waves is spread over every compute unit
  const uint32_t gw = (uint32_t)wave * nb + gb, nwv = nb * W;
  if (threadIdx.x == 0) {
    sh.nqw = 0u;
    sh.upd = 0u;
    sh.minp = kNoKey;
    sh.work = 0u;
    sh.heavy = 0u;
  }
  __syncthreads();
  const uint32_t nw = counts.w, ng = counts.g;
  const bool pull = PULL && A.T.hdr != nullptr && A.pull_min >= 0 &&
                    ld_agent64(&C->ctr.fedges[rc]) >= (unsigned long long)A.pull_min;
  if (pull) {
    if (gb == 0 && threadIdx.x == 0) acc.fe += ld_agent64(&C->ctr.frows[rc]);
    ss_pull<WT, MODE>(A, cur, nxt, rn, gw, nwv, acc, sh, seen);
  } else {

    // workgroup tier: one chunk of one row per workgroup
    for (uint32_t i = gb; i < ng; i += nb) {
      const int4 r = ld_queue4(&A.qwg[cur][i]);
      const int32_t u = r.x, start = r.y, uoff = copy_off<COPIES>(A, u);
      const uint32_t dul = ld_agent(&A.dist[u]);
      const bool skipped = ss_skip_row(A, nxt, u);  // (loaded beside the distance)
      // one value per wavefront (another wavefront may read a lower one; then
      // the row has been lowered in this step and is queued for the next)
      const uint32_t du = (uint32_t)__builtin_amdgcn_readfirstlane((int)dul);
      const int32_t len = skipped ? 0 : r.z;
      if (threadIdx.x == 0) {
        acc.es += (unsigned long long)len;
        if (NF) seen.work += (uint32_t)len;
        if (r.w) acc.fe += 1;
      }
      const int32_t stride = (int32_t)blockDim.x;
      for (int32_t base = 0; base < len; base += stride * kUnroll) {
        int32_t e[kUnroll], v[kUnroll], off[kUnroll];
        bool ok[kUnroll], imp[kUnroll];
        uint32_t d[kUnroll], cand[kUnroll], hvw[kUnroll];
  #pragma unroll
        for (int j = 0; j < kUnroll; j++) {
          const int32_t k = base + j * stride + (int32_t)threadIdx.x;
          ok[j] = k < len;
          e[j] = start + k;
          d[j] = du;
          off[j] = uoff;
        }
        ss_relax_pre<WT, kUnroll, MODE>(A, e, ok, d, off, imp, v, cand, hvw);
        ss_enqueue<WT, kUnroll, PULL, MODE>(A, imp, v, off, cand, hvw, nxt, rn, acc, sh, seen);
      }
    }

    // wave tier: one wavefront per row
    for (uint32_t i = gw; i < nw; i += nwv) {
      const int32_t u = ld_queue(&A.qwave[cur][i]), uoff = copy_off<COPIES>(A, u);
      const uint32_t dul = ld_agent(&A.dist[u]);
      const int32_t start = A.rowptr[u - uoff], last = A.rowptr[u - uoff + 1];
      const bool skipped = ss_skip_row(A, nxt, u);
      const uint32_t du = (uint32_t)__builtin_amdgcn_readfirstlane((int)dul);
      const int32_t end = skipped ? start : last;
      if (lane == 0) {
        acc.fe += 1;
        acc.es += (unsigned long long)(end - start);
        if (NF) seen.work += (uint32_t)(end - start);
      }
      for (int32_t base = start; base < end; base += kWave * kUnroll) {
        int32_t e[kUnroll], v[kUnroll], off[kUnroll];
        bool ok[kUnroll], imp[kUnroll];
        uint32_t d[kUnroll], cand[kUnroll], hvw[kUnroll];
  #pragma unroll
        for (int j = 0; j < kUnroll; j++) {
          e[j] = base + j * kWave + lane;
          ok[j] = e[j] < end;
          d[j] = du;
          off[j] = uoff;
        }
        ss_relax_pre<WT, kUnroll, MODE>(A, e, ok, d, off, imp, v, cand, hvw);
        ss_enqueue<WT, kUnroll, PULL, MODE>(A, imp, v, off, cand, hvw, nxt, rn, acc, sh, seen);
      }
    }

    // lane tier: rows of at most t_lane edges are not queued.  The wavefronts
    // scan the step's bitmap, clear it and take its short rows 64 at a time; the
    // rows' edges are dealt out to the lanes.  The scan clears every word,
    // heavy rows' bits included: nothing else reads this bitmap during a push
    // step.
    const ScanSplit split(A.n, gw, nwv);
    int block = 0;  // of this wavefront's
    for (int64_t w0 = 0; w0 + split.first < split.nwords; w0 += split.block(), block++) {
      const int64_t wi = split.word(w0, lane);
      uint32_t* def = sh.def[wave];
      uint32_t bits = 0u, left = 0u, word = 0u;
      if (wi < split.nwords) {
        word = ld_agent(&A.bm[cur][wi]);
        if (NF)
          left = w0 == 0 ? left0
                 : COPIES && block <= nheld ? held[((block - 1) * W + wave) * kWave + lane]
                                            : ld_agent(&A.df[wi]);
        bits = left;
        if (word) {
          // (read only here: 8 sources on that grid, 1M words a step, most of them zero:
          // 123 ms with the long-row words of all read, 106 so)
          bits |= word & ~A.hv[wi];
          if (!NF) st_agent(&A.bm[cur][wi], 0u);
          if (count) acc.im += (unsigned long long)__popc(word);
        }
      }
      if (NF) def[lane] = 0u;
      scan_rows(sh.scan[wave], bits, [&](bool has, int o, int bit) {
        int32_t start = 0, deg = 0, uoff = 0;
        uint32_t du = 0;
        if (has) {
          const int32_t u = (int32_t)(split.word(w0, o) * 32 + bit);
          uoff = copy_off<COPIES>(A, u);
          start = A.rowptr[u - uoff];
          deg = A.rowptr[u - uoff + 1] - start;
          du = ld_agent(&A.dist[u]);
          const bool skipped = ss_skip_row(A, nxt, u);
          if (NF && du > thr) {
            atomicOr(&def[o], 1u << bit);
            seen.minp = min(seen.minp, du);
            deg = 0;
          }
          if (deg > 0) acc.fe += 1;  // a frontier row (rows without edges are not counted)
          if (skipped) deg = 0;
          acc.es += (unsigned long long)deg;
          if (NF) seen.work += (uint32_t)deg;
        }
        deal_rows<kUnrollLane>(sh.rows[wave], start, deg, du, uoff, [&](const int32_t (&e)[kUnrollLane],
                                                                        const bool (&ok)[kUnrollLane],
                                                                        const uint32_t (&d)[kUnrollLane],
                                                                        const int32_t (&offs)[kUnrollLane]) {
          int32_t v[kUnrollLane], off[kUnrollLane];
#pragma unroll
          for (int j = 0; j < kUnrollLane; j++) off[j] = COPIES ? offs[j] : 0;
          bool imp[kUnrollLane];
          uint32_t cand[kUnrollLane], hvw[kUnrollLane];
          ss_relax_pre<WT, kUnrollLane, MODE>(A, e, ok, d, off, imp, v, cand, hvw);
          ss_enqueue<WT, kUnrollLane, PULL, MODE>(A, imp, v, off, cand, hvw, nxt, rn, acc, sh, seen);
        });
      });
      if (NF) {
        // (cleared only now: what waits for a load waits for an earlier store too, a
        // round trip per block: 2048 x 2048 grid 40.3 ms with the store first, 38.2 here)
        if (word) st_agent(&A.bm[cur][wi], 0u);
        wave_lds_sync();
        const uint32_t x = def[lane];
        if (w0 == 0) left0 = x;
        else if (COPIES && block <= nheld) held[((block - 1) * W + wave) * kWave + lane] = x;
        else if (x != left) st_agent(&A.df[wi], x);
        if (x) sh.upd = 1u;
      }
    }

  }

  // publish the workgroup's next-frontier entries and ptr flag
  if constexpr (NF) {
    const uint32_t mp = wave_min(seen.minp), wk = (uint32_t)wave_incl_scan((int)seen.work);
    if (lane == kWave - 1) {
      if (mp != kNoKey) atomicMin(&sh.minp, mp);
      if (wk) atomicAdd(&sh.work, wk);
    }
  }
  __syncthreads();
  const uint32_t n_w = min(sh.nqw, (uint32_t)kLdsQWave);
  if (threadIdx.x == 0) {
    if (n_w) sh.gbase_w = atomicAdd(&C->cnt[rn][1].v, n_w);
    if (sh.upd) st_agent(&C->upd[rn], 1u);
    if (!NF && sh.upd) sh.minp = 0u;  // some row; its key does not matter
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < n_w; j += blockDim.x) {
    const uint32_t p = sh.gbase_w + j;
    if (p < A.cap_v) st_agent_i(&A.qwave[nxt][p], sh.qw[j]);
    else atomicOr(&C->overflow, 1u);
  }
  return pull;
}

__device__ __forceinline__ void ss_zero_rotation(SsCtl* C, uint32_t step) {
  const int rz = (step + 2) % kRot;
  for (int t = 0; t < 4; t++) st_agent(&C->cnt[rz][t].v, 0u);
  st_agent(&C->upd[rz], 0u);
  st_agent(&C->minp[rz].v, kNoKey);
  st_agent64(&C->ctr.fedges[rz], 0ull);
  st_agent64(&C->ctr.frows[rz], 0ull);
}

// Grid barrier of the single-source steps (grid_sync): an arrival carries the
// workgroup's smallest next-frontier key, whether it queued rows and the edges
// it expanded (to an eighth, as an 8-bit float), and the release word brings
// back the next step's threshold (0: the frontier is empty) and whether the
// queues hold rows, so neither costs an atomic or a load of its own.
//   slot:    key (32) | epoch (23) | queued (1) | edges (8)
//   release: threshold (32) | epoch (30) | fresh (1) | queued (1)
// After a step of few edges (at most twice nf_work) the next one is bound by its chain of dependent
// loads, and the barrier does without the invalidation: distances are then read
// at agent scope (fresh), and the CSR's lines, which neighbouring frontiers
// share, stay in the caches.  (Only where rows are deferred: elsewhere, R-MAT
// above all, one step can be thousands of times larger than the last.)
struct SsNext {
  uint32_t thr;
  bool queued, fresh;
};

template <int WT>
__device__ __forceinline__ bool ss_grid_sync(SsCtl* C, uint32_t nblocks, uint32_t base,
                                             uint32_t& epoch, unsigned long long ticks,
                                             const SsShared& sh, NfState& nf, float busy, SsNext& next) {
  __shared__ int s_ok;
  __shared__ uint32_t s_min, s_queued, s_thr, s_fresh;
  __shared__ float s_work;
  GridBar* bar = &C->bar;
  wait_own_stores();
  if (threadIdx.x == 0) {
    s_ok = 1;
    s_min = sh.minp;
    s_queued = sh.heavy;
    s_work = (float)sh.work;
  }
  __syncthreads();
  epoch += 1;
  const uint32_t target = base + epoch;
  const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
  unsigned long long word;
  if (blockIdx.x == 0) {
    for (uint32_t b = 1 + threadIdx.x; b < nblocks; b += blockDim.x) {
      if (!grid_wait<9>(&bar->slot[b], target, &C->abort, t0, ticks, word)) {
        s_ok = 0;
        break;
      }
      const uint32_t lo = (uint32_t)word;
      atomicMin(&s_min, (uint32_t)(word >> 32));
      if (lo & 0x100u) s_queued = 1u;
      if (lo & 0xFFu)
        atomicAdd(&s_work, __uint_as_float(((lo & 0xFFu) << 20) + 0x3F800000u) - 1.f);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t t = 0u;  // empty frontier
      if (s_min != kNoKey) {
        nf_advance<WT>(nf, s_min, s_work, busy);
        t = nf.thr;
      }
      s_thr = t;
      s_fresh = nf.floor != 0.f && s_work <= 2.f * busy;
      if (s_ok)
        st_agent64(&bar->release.v, ((unsigned long long)t << 32) | (target << 2) |
                                        (s_fresh ? 2u : 0u) | (s_queued ? 1u : 0u));
      if (!s_fresh) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
  } else if (threadIdx.x == 0) {
    const uint32_t wk = (__float_as_uint((float)(sh.work + 1u)) - 0x3F800000u) >> 20;
    st_agent64(&bar->slot[blockIdx.x], ((unsigned long long)sh.minp << 32) | (target << 9) |
                                           (sh.heavy ? 0x100u : 0u) | wk);
    if (!grid_wait<2>(&bar->release.v, target, &C->abort, t0, ticks, word)) s_ok = 0;
    s_thr = (uint32_t)(word >> 32);
    s_queued = (uint32_t)word & 1u;
    s_fresh = (uint32_t)word & 2u;
    if (!s_fresh) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  next.thr = s_thr;
  next.queued = s_queued != 0u;
  next.fresh = s_fresh != 0u;
  return s_ok != 0;
}

// All steps in one launch; a grid barrier separates the steps.  The grid must
// be co-resident: its size is what the compute units hold at once by the
// kernel's compiled resources (residency_of); should a barrier wait still give
// up, the run ends with status -2, reported to the caller.
template <int WT, bool COPIES>
__global__ void __launch_bounds__(1024) ss_persistent_kernel(SsArgs A, dawn_run_info* info,
                                                             int32_t nheld, uint32_t even_wgs,
                                                             uint32_t wide_wgs) {
  __shared__ SsShared sh;
  extern __shared__ uint32_t held[];  // copies: rows left for later, see ss_step
  SsCtl* C = A.ctl;
  // the workgroups that take part (`even` is of an earlier launch)
  const uint32_t gb = blockIdx.x, nb = C->even ? even_wgs : wide_wgs;
  if (gb >= nb) return;
  // Ended by an earlier launch, or given up by workgroup 0, which may happen while
  // this workgroup starts: one read for all of its threads, which would else part
  // here and miss each other at the barriers of the steps.
  if (ld_agent_block(&C->done)) {
    if (COPIES && ld_agent_i(&C->converged) == kNoRun) return;  // (an earlier launch's word)
    if (last_block_arrive(&C->arrive, nb) && threadIdx.x == 0) ss_report<WT>(C, info, A.latch);
    return;
  }
  Acc acc;
  uint32_t epoch = 0;
  const uint32_t bar_base = ld_agent(&C->bar_base);
  uint32_t step = ld_agent(&C->step);
  SsCounts counts = ss_counts(A, step);
  NfState nf = C->nf;  // (workgroup 0 keeps it; written by an earlier launch)
  SsNext next{nf.thr, false, false};
  // the frontier of the first step here: seeds, or counted already when step
  // launches that count as they enqueue came before
  bool count = step > 0 && !A.counted;
  int32_t status = 1;
  const uint32_t wave = threadIdx.x >> 6, W = blockDim.x >> 6;
  uint32_t left0 = 0u;
  if (nf_weights<WT>()) {
    const ScanSplit split(A.n, wave * nb + gb, nb * W);  // (as in ss_step)
    const int64_t wi = split.word(0, lane_id());
    if (wi < split.nwords) left0 = A.df[wi];  // (written by an earlier launch)
  }
  if (COPIES)  // (no step launches came before: nothing is left yet)
    for (int i = lane_id(); i < nheld * kWave; i += kWave)
      held[((i / kWave) * W + wave) * kWave + i % kWave] = 0u;
  for (;;) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ss_zero_rotation(C, step);
    if (nf_weights<WT>() && nf.floor != 0.f) {
      if (next.fresh)
        ss_step<WT, false, kFresh, COPIES>(A, step, gb, nb, acc, sh, counts, next.thr, count, left0, held, nheld);
      else
        ss_step<WT, false, kNear, COPIES>(A, step, gb, nb, acc, sh, counts, next.thr, count, left0, held, nheld);
    } else {
      ss_step<WT, false, kAll, COPIES>(A, step, gb, nb, acc, sh, counts, kNoKey, count, left0, held, nheld);
    }
    count = true;
    if (!ss_grid_sync<WT>(C, nb, bar_base, epoch, A.bar_ticks, sh, nf, A.nf_work, next)) {
      status = -2;
      break;
    }
    step++;
    if (next.thr == 0u) { status = 1; break; }
    if (step >= (uint32_t)A.n) { status = 0; break; }
    counts = next.queued ? ss_counts(A, step) : SsCounts{0u, 0u};
  }
  if (WT == kWI32 && status == 0) {  // no scan follows that would count what the last step lowered
    const int64_t nwords = ((int64_t)A.n + 31) / 32;
    for (int64_t i = (int64_t)gb * blockDim.x + threadIdx.x; i < nwords; i += (int64_t)nb * blockDim.x)
      acc.im += (unsigned long long)__popc(ld_agent(&A.bm[step & 1][i]));
  }
  SsCounters& S = C->ctr;
  flush_acc(acc, &S.fe, &S.es, &S.im, nullptr, nullptr);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st_agent(&C->step, step);
    st_agent_i(&C->converged, status);
    st_agent(&C->done, 1u);
    st_agent(&C->bar_base, bar_base + epoch);
  }
  // the last workgroup to leave has every counter: it reports the run
  if (last_block_arrive(&C->arrive, nb) && threadIdx.x == 0) ss_report<WT>(C, info, A.latch);
}

// One step per launch; the last block to finish advances the step.
template <int WT, bool PULL>
__global__ void __launch_bounds__(1024) ss_step_kernel(SsArgs A) {
  __shared__ SsShared sh;
  SsCtl* C = A.ctl;
  if (ld_agent(&C->done)) return;
  const uint32_t step = ld_agent(&C->step);
  if (blockIdx.x == 0 && threadIdx.x == 0) ss_zero_rotation(C, step);
  Acc acc;
  const uint32_t gb = blockIdx.x, nb = gridDim.x;
  // (written by an earlier launch; with pull steps no row waits: they take the
  // frontier from one bitmap, and their rule needs all of its out-edges counted)
  const bool near = !PULL && nf_weights<WT>() && C->nf.floor != 0.f;
  bool pulled = false;
  uint32_t left0 = 0u;
  if constexpr (!PULL) {
    if (near) {
      const uint32_t wave = threadIdx.x >> 6, W = blockDim.x >> 6;
      const ScanSplit split(A.n, wave * nb + gb, nb * W);  // (as in ss_step)
      const int64_t wi = split.word(0, lane_id());
      if (wi < split.nwords) left0 = A.df[wi];
      const uint32_t was = left0;
      ss_step<WT, false, kNear, false>(A, step, gb, nb, acc, sh, ss_counts(A, step), C->nf.thr,
                                       step > 0, left0);
      if (left0 != was) A.df[wi] = left0;
    }
  }
  if (!near)
    pulled = ss_step<WT, PULL, kAll, false>(A, step, gb, nb, acc, sh, ss_counts(A, step), kNoKey,
                                            !PULL && step > 0, left0);
  if (near && threadIdx.x == 0 && sh.minp != kNoKey)
    atomicMin(&C->minp[(step + 1) % kRot].v, sh.minp);
  // counters, and the next frontier's out-edges and rows (its pull decision)
  SsCounters& S = C->ctr;
  flush_acc(acc, &S.fe, &S.es, &S.im, &S.fedges[(step + 1) % kRot], &S.frows[(step + 1) % kRot]);
  if (last_block_arrive(&C->arrive, gridDim.x)) {
    // a pull step read the current bitmap throughout: clear it now, before it
    // serves as the next step's next-frontier bitmap
    if (pulled)
      for (int64_t i = threadIdx.x; i < ((int64_t)A.n + 31) / 32; i += blockDim.x)
        A.bm[step & 1][i] = 0u;
    const uint32_t upd = ld_agent(&C->upd[(step + 1) % kRot]);
    const uint32_t ns = step + 1;
    if (WT == kWI32 && !PULL && upd && ns >= (uint32_t)A.n) {  // as in the persistent launch
      unsigned long long im = 0;
      for (int64_t i = threadIdx.x; i < ((int64_t)A.n + 31) / 32; i += blockDim.x)
        im += (unsigned long long)__popc(ld_agent(&A.bm[ns & 1][i]));
      if (im) atomicAdd(&S.im, im);
    }
    if (threadIdx.x != 0) return;
    st_agent(&C->step, ns);
    if (near && upd) {
      NfState nf = C->nf;  // (only a launch's last workgroup writes it)
      const unsigned long long es = ld_agent64(&S.es);
      nf_advance<WT>(nf, ld_agent(&C->minp[ns % kRot].v), (float)(es - C->es_seen), A.nf_work);
      C->es_seen = es;
      C->nf = nf;
    }
    if (!upd) {
      st_agent_i(&C->converged, 1);
      st_agent(&C->done, 1u);
    } else if (ns >= (uint32_t)A.n) {
      st_agent_i(&C->converged, 0);
      st_agent(&C->done, 1u);
    }
  }
}

// ---------------------------------------------------------------------------
// one workgroup per source: the run's state in LDS
//
// With n <= kCuMaxN the distances and both beta bitmaps of a run fit in one
// workgroup's LDS, so every step runs on LDS atomics and a workgroup barrier;
// only the CSR is read from global memory (it stays in the L2), and the final
// distances are copied out once.  A step is bound by one compute unit's
// instruction rate and a chain of about ten dependent loads.  Measured, fp32
// ER graphs, call times: n = 15,013, m = 120,104: 1165 us with the frontier
// queue, distances and bitmaps in global memory, 214 us here (347 us with the
// persistent grid); n = 10,000 grid: 387 us against 2046 us.
// MULTI: workgroup j runs source j of a multi-source call, so k sources keep k
// compute units busy with no grid barrier and no tile (all pairs of an ER
// graph with 1531 vertices and 12,248 edges: 5.5 ms with tiles of 256
// columns, 0.39 ms here).
// ---------------------------------------------------------------------------
constexpr int kTinyN = 6144;

// End of a one-workgroup run, reached by every thread: the counters are summed
// over the workgroup (`part`: LDS scratch).  A single run stores them and its
// state in the control words and reports as ss_report does; a run of a
// multi-source call adds them to `info` (zeroed by an earlier launch).  tile: the
// sources of a tile (multi-source calls).
template <int WT, bool MULTI>
__device__ void ss_wg_report(const SsArgs& A, dawn_run_info* info, int32_t status, uint32_t step,
                             const Acc& acc, unsigned long long (*part)[3], uint32_t tile) {
  SsCtl* C = A.ctl;
  const unsigned long long v0 = wave_sum64(acc.fe), v1 = wave_sum64(acc.es),
                           v2 = wave_sum64(acc.im);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) {
    part[w][0] = v0;
    part[w][1] = v1;
    part[w][2] = v2;
  }
  // the int32 range flag is set by any thread's atomic
  if (!MULTI && (WT == kWI32 || status == -1)) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long fe = 0, es = 0, im = 0;
  for (int i = 0; i < (int)(blockDim.x / kWave); i++) {
    fe += part[i][0];
    es += part[i][1];
    im += part[i][2];
  }
  if constexpr (MULTI) {
    if (!info) {
      // a bad source counts as one run that failed, as its tile's would
      if (status != -1 || blockIdx.x % tile == 0) latch_status(A.latch, status);
      return;
    }
    atomicMax(&info->steps, (int32_t)step);
    atomicMin(&info->converged, status);
    auto add = [](int64_t* p, unsigned long long x) {
      atomicAdd(reinterpret_cast<unsigned long long*>(p), x);
    };
    add(&info->frontier_entries, fe);
    add(&info->edges_scanned, es);
    add(&info->improvements, im);
    add(&info->union_rows, fe);
    add(&info->union_edges, es);
    return;
  }
  SsCounters& S = C->ctr;
  st_agent64(&S.fe, fe);
  st_agent64(&S.es, es);
  st_agent64(&S.im, im);
  if (status == -1) {
    // failed validation: report what the control words record
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    ss_report<WT>(C, info, A.latch);
    return;
  }
  if (WT == kWI32) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const uint32_t ab = ld_agent(&C->abort), ov = ld_agent(&C->overflow);
  const uint32_t nf = WT == kWI32 ? ld_agent(&C->negfloor) : 0u;
  st_agent(&C->step, step);
  st_agent_i(&C->converged, status);
  st_agent(&C->done, 1u);
  int32_t conv = run_status(status, ab, ov);
  if (WT == kWI32 && conv == 1 && nf) conv = 0;
  if (!info) {
    latch_status(A.latch, conv);
  } else {
    info->steps = (int32_t)step;
    info->converged = conv;
    info->frontier_entries = (int64_t)fe;
    info->edges_scanned = (int64_t)es;
    info->improvements = (int64_t)im;
    info->union_rows = (int64_t)fe;
    info->union_edges = (int64_t)es;
  }
}

// Whether the tile that source blockIdx.x would be in (of `tile` sources) holds a
// source outside [0, n): such a tile's run ends before its first step.  Every
// thread calls it and gets the result.
__device__ __forceinline__ bool ss_multi_bad(const int32_t* sources, int32_t k, int32_t tile,
                                             int32_t n) {
  const int32_t j0 = (int32_t)blockIdx.x / tile * tile;
  bool bad = false;
  for (int32_t j = j0 + (int32_t)threadIdx.x; j < min(k - j0, tile) + j0; j += blockDim.x)
    bad |= sources[j] < 0 || sources[j] >= n;
  return __syncthreads_or(bad) != 0;
}

// A distance key as the caller sees it (int32: the sign bit flipped back).
template <int WT>
__device__ __forceinline__ uint32_t key_value(uint32_t key) {
  return WT == kWI32 ? key ^ 0x80000000u : key;
}

// Sizes of the kernel's instances: the state of a smaller graph leaves room
// for a copy of the row pointers (one L2 round trip less per step), and for a
// second workgroup per compute unit.
constexpr int kCuMidN = 16384, kCuMaxN = 32768;
constexpr int kUnrollCu = 4;  // edges in flight per lane
// Deferral here: edges per step that keep one compute unit busy, and the fewest
// edges with which a run has such steps.  Below, tracking the smallest key only
// costs (grid of 10,000 vertices, 39,212 edges: 365 -> 404 us).  Measured without
// / with: ER n = 15,013, m = 120,104 195 / 170 us; n = 32,768, m = 262,144 366 /
// 297 us, m = 131,072 275 / 277; grid of 32,761 vertices 1014 / 837 us.
constexpr float kNfWorkCu = 1000.f;
constexpr int kNfMinCu = 65536;
constexpr int kCuWin = 1024;  // edges marked at a time (sized so that kCuMaxN fits)

template <int N>
struct SsCuShared {
  static constexpr bool kRows = N <= kCuMidN;  // row pointers in LDS
  uint32_t dist[N];
  uint32_t bm[2][N / 32];
  int32_t rp[kRows ? N + 1 : 1];
  union {
    struct {
      DealRows<kCuWin> rows;
      ScanRows scan;
    } st[kMaxWavesPerBlock];
    unsigned long long part[kMaxWavesPerBlock][3];  // the report's sums, after the last step
  };
  uint32_t upd[3];
  uint32_t minp[3], work[3];  // deferral: smallest key left in the frontier, edges expanded
};
static_assert(sizeof(SsCuShared<kCuMaxN>) <= 160 * 1024, "LDS of a compute unit");
static_assert(sizeof(SsCuShared<kCuMidN>) <= 160 * 1024, "LDS of a compute unit");

template <int WT, int N, bool MULTI>
__global__ void __launch_bounds__(1024) ss_cu_kernel(SsArgs A, const int32_t* sources,
                                                     const int64_t* voff, int32_t count,
                                                     int32_t single, int32_t check_valid,
                                                     dawn_run_info* info) {
  __shared__ SsCuShared<N> sh;
  constexpr bool kRows = SsCuShared<N>::kRows;
  SsCtl* C = A.ctl;
  const int lane = lane_id(), wave = threadIdx.x >> 6, W = blockDim.x >> 6;
  const int n = A.n, nwords = (n + 31) / 32;
  uint32_t* out = A.dist;
  int32_t src = A.src;
  uint32_t step = 0;
  int32_t status = 1;
  Acc acc;
  if constexpr (MULTI) {
    out += (size_t)blockIdx.x * n;
    src = sources[blockIdx.x];
    if (ss_multi_bad(sources, count, single, n)) status = -1;
  } else {
    if (check_valid && ld_agent(&C->done)) status = -1;
  }
  if (status == -1) {
    // nothing is run: every distance INF (but a source's own, as a tile leaves it)
    for (int i = threadIdx.x; i < n; i += blockDim.x)
      out[i] = key_value<WT>(MULTI && WT != kWUNIT && i == src ? zero_key<WT>() : inf_key<WT>());
  } else {
    for (int i = threadIdx.x; i < n; i += blockDim.x) sh.dist[i] = inf_key<WT>();
    for (int i = threadIdx.x; i < nwords; i += blockDim.x) {
      sh.bm[0][i] = 0u;
      sh.bm[1][i] = 0u;
    }
    if constexpr (kRows)
      for (int i = threadIdx.x; i <= n; i += blockDim.x) sh.rp[i] = A.rowptr[i];
    if (threadIdx.x < 3) {
      sh.upd[threadIdx.x] = 0u;
      sh.minp[threadIdx.x] = kNoKey;
      sh.work[threadIdx.x] = 0u;
    }
    if (!MULTI && threadIdx.x == 0) {
      // the status words the report reads: the workspace may hold an earlier
      // run's (atomics, as the later reports are)
      atomicExch(&C->negfloor, 0u);
      atomicExch(&C->abort, 0u);
      atomicExch(&C->overflow, 0u);
    }
    // far rows wait, as in the multi-workgroup runs
    bool even;
    const float floor =
        nf_weights<WT>() && A.m >= kNfMinCu
            ? nf_floor<WT>(n, A.m, A.rowptr, A.w, 1024, !MULTI && voff, even) : 0.f;
    NfState nf{kNoKey, floor, floor, 0u};
    // (the words of the rows left for later stay in a register of the lane that scans
    // them, one word a lane, as all do at 1024 threads)
    const bool near = nf_weights<WT>() && floor != 0.f && nwords <= kWave * W;
    uint32_t left = 0u;
    __syncthreads();
    if constexpr (MULTI) {
      if (threadIdx.x == 0) {
        sh.dist[src] = zero_key<WT>();
        sh.bm[0][src >> 5] = 1u << (src & 31);
      }
    } else {
      for (int j = threadIdx.x; j < count; j += blockDim.x) {
        int64_t s = sources ? (int64_t)sources[j] : (int64_t)single;
        if (voff) s += voff[j];
        sh.dist[s] = zero_key<WT>();
        atomicOr(&sh.bm[0][s >> 5], 1u << (s & 31));
      }
    }
    __syncthreads();
    auto& st = sh.st[wave];
    for (;;) {
      uint32_t* bc = sh.bm[step & 1];
      uint32_t* bn = sh.bm[(step & 1) ^ 1];
      bool upd = false;
      StepSeen seen;
      // wavefront w scans words w, w + W, ..., up to 64 of them at a time (one
      // pass at 1024 threads): a frontier band is shared by all wavefronts, and
      // a wavefront's rows wait for one chain of loads per 64 of them
      for (int w0 = wave; w0 < nwords; w0 += kWave * W) {
        const int wi = w0 + lane * W;
        uint32_t bits = 0u;
        if (wi < nwords) {
          bits = bc[wi];
          if (bits) {
            bc[wi] = 0u;
            if (step > 0) acc.im += (unsigned long long)__popc(bits);  // lowered by the last step
          }
          bits |= left;
        }
        scan_rows(st.scan, bits, [&](bool has, int o, int bit) {
          int32_t start = 0, deg = 0;
          uint32_t du = 0;
          if (has) {
            const int u = (w0 + o * W) * 32 + bit;
            if constexpr (kRows) {
              start = sh.rp[u];
              deg = sh.rp[u + 1] - start;
            } else {
              start = A.rowptr[u];
              deg = A.rowptr[u + 1] - start;
            }
            du = sh.dist[u];
            if (near && du > nf.thr) {
              atomicOr(&bc[u >> 5], 1u << (u & 31));  // (the wavefront's own word, just cleared)
              seen.minp = min(seen.minp, du);
              deg = 0;
            }
            if (deg > 0) acc.fe += 1;  // a frontier row (rows without edges are not counted)
            // lowered again in this step: expanded in the next, with the lower value
            if (A.skip && ((bn[u >> 5] >> (u & 31)) & 1u)) deg = 0;
            acc.es += (unsigned long long)deg;
            seen.work += (uint32_t)deg;
          }
          deal_rows<kUnrollCu>(st.rows, start, deg, du, 0, [&](const int32_t (&e)[kUnrollCu],
                                                               const bool (&ok)[kUnrollCu],
                                                               const uint32_t (&d)[kUnrollCu],
                                                               const int32_t (&)[kUnrollCu]) {
            int32_t v[kUnrollCu];
            uint32_t cand[kUnrollCu], dv[kUnrollCu];
#pragma unroll
            for (int j = 0; j < kUnrollCu; j++) {
              v[j] = 0;
              cand[j] = 0u;
              if (ok[j]) {
                v[j] = A.colidx[e[j]];
                cand[j] = relax_key<WT>(d[j], WT == kWUNIT ? 1u : A.w[e[j]]);
                if constexpr (WT == kWI32)
                  if (cand[j] == 0u) atomicOr(&C->negfloor, 1u);  // sum left the int32 range
              }
            }
#pragma unroll
            for (int j = 0; j < kUnrollCu; j++) dv[j] = sh.dist[v[j]];
#pragma unroll
            for (int j = 0; j < kUnrollCu; j++) {
              if (ok[j] && cand[j] < dv[j] && v[j] != src &&
                  cand[j] < atomicMin(&sh.dist[v[j]], cand[j])) {
                upd = true;
                seen.minp = min(seen.minp, cand[j]);
                __hip_atomic_fetch_or(&bn[v[j] >> 5], 1u << (v[j] & 31), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
              }
            }
          });
        });
        if (near) {
          wave_lds_sync();
          left = wi < nwords ? bc[wi] : 0u;
          if (left) bc[wi] = 0u;
        }
      }
      // three flags rotate: step t sets (t+1) mod 3, read after the barrier,
      // and clears (t+2) mod 3, which nothing else touches before step t+1 ends
      if (threadIdx.x == 0) {
        sh.upd[(step + 2) % 3] = 0u;
        sh.minp[(step + 2) % 3] = kNoKey;
        sh.work[(step + 2) % 3] = 0u;
      }
      if (near) {
        const uint32_t mp = wave_min(seen.minp), wk = (uint32_t)wave_incl_scan((int)seen.work);
        if (lane == kWave - 1) {
          if (mp != kNoKey) atomicMin(&sh.minp[(step + 1) % 3], mp);
          if (wk) atomicAdd(&sh.work[(step + 1) % 3], wk);
        }
      } else if (upd) {
        sh.upd[(step + 1) % 3] = 1u;
      }
      __syncthreads();
      uint32_t more = sh.upd[(step + 1) % 3];
      if (near) {
        const uint32_t mp = sh.minp[(step + 1) % 3];
        more = mp != kNoKey;
        nf_advance<WT>(nf, mp, (float)sh.work[(step + 1) % 3], kNfWorkCu);
      }
      step++;
      if (!more) { status = 1; break; }
      if (step >= (uint32_t)n) { status = 0; break; }
    }
    if (status == 0)  // lowered by the last step
      for (int i = threadIdx.x; i < nwords; i += blockDim.x)
        acc.im += (unsigned long long)__popc(sh.bm[step & 1][i]);
    for (int i = threadIdx.x; i < n; i += blockDim.x) out[i] = key_value<WT>(sh.dist[i]);
  }
  ss_wg_report<WT, MULTI>(A, info, status, step, acc, sh.part, (uint32_t)single);  // (after the last step's barrier)
}

// ---------------------------------------------------------------------------
// graphs that fit whole in LDS: edge-parallel steps
//
// With n <= kTinyN and m <= kLdsM a workgroup of kLdsThreads threads holds the
// whole run: the distances, the frontier bitmaps and the weights in LDS, and
// each thread's edges t, t + kLdsThreads, ... (at most E, the instance's edges
// per thread) in registers, as packed (source, target) ids.  A step then needs no queue: a thread
// relaxes each of its edges whose source's bit is set in the step's frontier
// bitmap.  Those are exactly the out-edges of the frontier, the relaxations
// Algorithm 2 makes, and every thread gets the same number of edges whatever
// the degrees.  A target lowered in the step gets its bit in the next bitmap.
// Three bitmaps and three update flags rotate, so one barrier per step
// suffices: step t reads bitmap t mod 3, sets bits in (t+1) mod 3 and clears
// (t+2) mod 3, which step t-1 read and step t+1 fills.
// ---------------------------------------------------------------------------
constexpr int kLdsThreads = 1024;
constexpr int kLdsM = kLdsThreads * 16;  // the largest instance: 16 edges per thread
constexpr int kLdsRows = kTinyN / kLdsThreads;  // vertices per thread

template <int E>
struct SsLdsShared {
  uint32_t dist[kTinyN];
  uint32_t bm[3][kTinyN / 32];
  uint32_t upd[3];
  uint16_t src[kLdsThreads * E];  // each edge's source, read once to fill the registers
  uint32_t w[kLdsThreads * E];
  unsigned long long part[kLdsThreads / kWave][3];
};

template <int WT, int E, bool MULTI>
__global__ void __launch_bounds__(kLdsThreads) ss_lds_kernel(SsArgs A, const int32_t* sources,
                                                             const int64_t* voff, int32_t count,
                                                             int32_t single, int32_t check_valid,
                                                             dawn_run_info* info) {
  constexpr int kLdsEdges = E, kLdsHalf = E < 8 ? E : 8;
  __shared__ SsLdsShared<E> sh;
  SsCtl* C = A.ctl;
  const int n = A.n, m = A.m, nwords = (n + 31) / 32, t = threadIdx.x;
  uint32_t* out = A.dist;
  int32_t src = A.src;
  uint32_t step = 0;
  int32_t status = 1;
  Acc acc;
  if constexpr (MULTI) {
    out += (size_t)blockIdx.x * n;
    src = sources[blockIdx.x];
    if (ss_multi_bad(sources, count, single, n)) status = -1;
  } else {
    if (check_valid && ld_agent(&C->done)) status = -1;
  }
  if (status == -1) {
    // nothing is run: every distance INF (but a source's own, as a tile leaves it)
    for (int i = t; i < n; i += kLdsThreads)
      out[i] = key_value<WT>(MULTI && WT != kWUNIT && i == src ? zero_key<WT>() : inf_key<WT>());
  } else {
    if (!MULTI && t == 0) {
      // the status words the report reads: the workspace may hold an earlier
      // run's
      atomicExch(&C->negfloor, 0u);
      atomicExch(&C->abort, 0u);
      atomicExch(&C->overflow, 0u);
    }
    // this thread's edges and rows: every global load issued before any use
    uint32_t tv[kLdsEdges], we[kLdsEdges];
#pragma unroll
    for (int j = 0; j < kLdsEdges; j++) {
      const int e = t + j * kLdsThreads;
      tv[j] = e < m ? (uint32_t)A.colidx[e] : 0u;
      we[j] = (WT != kWUNIT && e < m) ? A.w[e] : 1u;
    }
#pragma unroll
    for (int j = 0; j < kLdsEdges; j++)
      if (t + j * kLdsThreads < m) sh.w[t + j * kLdsThreads] = we[j];
    int32_t ra[kLdsRows], rb[kLdsRows];
#pragma unroll
    for (int i = 0; i < kLdsRows; i++) {
      const int u = t + i * kLdsThreads;
      ra[i] = u < n ? A.rowptr[u] : 0;
      rb[i] = u < n ? A.rowptr[u + 1] : 0;
    }
#pragma unroll
    for (int i = 0; i < kLdsRows; i++) {
      const int u = t + i * kLdsThreads;
      if (u < n) {
        for (int32_t e = ra[i]; e < rb[i]; e++) sh.src[e] = (uint16_t)u;
        sh.dist[u] = inf_key<WT>();
      }
    }
    for (int i = t; i < nwords; i += kLdsThreads) {
      sh.bm[0][i] = 0u;
      sh.bm[1][i] = 0u;
      sh.bm[2][i] = 0u;
    }
    if (t < 3) sh.upd[t] = 0u;
    __syncthreads();
    // (source, target) of each edge packed in one register; bit j of `first`:
    // edge j is its row's first edge (counts the row once per step)
    uint32_t uv[kLdsEdges];
    uint32_t first = 0u;
#pragma unroll
    for (int j = 0; j < kLdsEdges; j++) {
      const int e = t + j * kLdsThreads;
      uv[j] = 0u;
      if (e < m) {
        const uint32_t u = sh.src[e];
        uv[j] = u | (tv[j] << 16);
        if (e == 0 || sh.src[e - 1] != u) first |= 1u << j;
      }
    }
    if constexpr (MULTI) {
      if (t == 0) {
        sh.dist[src] = zero_key<WT>();
        sh.bm[0][src >> 5] = 1u << (src & 31);
      }
    } else {
      for (int j = t; j < count; j += kLdsThreads) {
        int64_t s = sources ? (int64_t)sources[j] : (int64_t)single;
        if (voff) s += voff[j];
        sh.dist[s] = zero_key<WT>();
        atomicOr(&sh.bm[0][s >> 5], 1u << (s & 31));
      }
    }
    __syncthreads();
    for (;;) {
      const uint32_t* bc = sh.bm[step % 3];
      uint32_t* bn = sh.bm[(step + 1) % 3];
      bool upd = false;
      // Values derived from the edge ids (word indices, bit masks, LDS
      // addresses) are recomputed each step rather than kept in registers
      // across steps, which would not fit: the empty asm marks the ids as
      // changed here.
#pragma unroll
      for (int j = 0; j < kLdsEdges; j++) asm volatile("" : "+v"(uv[j]));
      // Frontier test of every edge, then the distances of the active ones,
      // then the atomics.  Every LDS read is unconditional (edges past m read
      // edge 0's slots, vertex 0), so a round's reads go out back to back and
      // are waited for once; a read under a branch would be waited for alone.
      uint32_t act = 0u;
      {
        uint32_t wd[kLdsEdges];
#pragma unroll
        for (int j = 0; j < kLdsEdges; j++) wd[j] = bc[(uv[j] & 0xFFFFu) >> 5];
#pragma unroll
        for (int j = 0; j < kLdsEdges; j++)
          act |= ((wd[j] >> (uv[j] & 31u)) & (t + j * kLdsThreads < m ? 1u : 0u)) << j;
      }
      // the active edges in halves of kLdsHalf (registers for their candidates)
#pragma unroll
      for (int h = 0; h < kLdsEdges; h += kLdsHalf) {
        if (!((act >> h) & ((1u << kLdsHalf) - 1u))) continue;
        uint32_t cand[kLdsHalf], dv[kLdsHalf];
#pragma unroll
        for (int i = 0; i < kLdsHalf; i++) {
          const int j = h + i, e = t + j * kLdsThreads;
          cand[i] = relax_key<WT>(sh.dist[uv[j] & 0xFFFFu], sh.w[e < m ? e : 0]);
          dv[i] = sh.dist[uv[j] >> 16];
        }
        uint32_t need = 0u;
#pragma unroll
        for (int i = 0; i < kLdsHalf; i++) {
          const int j = h + i;
          const uint32_t v = uv[j] >> 16;
          if ((act >> j) & 1u) {
            acc.es += 1;
            acc.fe += (first >> j) & 1u;
            if constexpr (WT == kWI32)
              if (cand[i] == 0u) atomicOr(&A.ctl->negfloor, 1u);  // sum left the int32 range
            if ((int32_t)v != src && cand[i] < dv[i]) need |= 1u << i;
          }
        }
        // returning atomics, all issued before any result is used
        uint32_t old[kLdsHalf];
#pragma unroll
        for (int i = 0; i < kLdsHalf; i++) {
          old[i] = 0u;
          if ((need >> i) & 1u) old[i] = atomicMin(&sh.dist[uv[h + i] >> 16], cand[i]);
        }
#pragma unroll
        for (int i = 0; i < kLdsHalf; i++) {
          const uint32_t v = uv[h + i] >> 16;
          if (((need >> i) & 1u) && cand[i] < old[i]) {
            upd = true;
            __hip_atomic_fetch_or(&bn[v >> 5], 1u << (v & 31), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      for (int i = t; i < nwords; i += kLdsThreads) {
        if (step > 0) acc.im += (unsigned long long)__popc(bc[i]);  // lowered by the last step
        sh.bm[(step + 2) % 3][i] = 0u;
      }
      if (t == 0) sh.upd[(step + 2) % 3] = 0u;
      if (upd) sh.upd[(step + 1) % 3] = 1u;
      __syncthreads();
      const uint32_t more = sh.upd[(step + 1) % 3];
      step++;
      if (!more) { status = 1; break; }
      if (step >= (uint32_t)n) { status = 0; break; }
    }
    if (status == 0)  // lowered by the last step
      for (int i = t; i < nwords; i += kLdsThreads)
        acc.im += (unsigned long long)__popc(sh.bm[step % 3][i]);
    for (int i = t; i < n; i += kLdsThreads) out[i] = key_value<WT>(sh.dist[i]);
  }
  ss_wg_report<WT, MULTI>(A, info, status, step, acc, sh.part, (uint32_t)single);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
SsLayout ss_layout(int64_t n, int64_t m) {
  SsLayout L{};
  Carver c;
  L.cap_v = (uint32_t)n;
  // at most m/65 rows exceed the smallest allowed t_wave (64), each cut into at
  // most deg/256 + 1 chunks (smallest allowed t_chunk 256)
  L.cap_wg = (uint32_t)(m / 65 + m / 256 + 2);
  L.nwords = (n + 31) / 32;
  L.ctl = c.take(sizeof(SsCtl));
  for (int i = 0; i < 2; i++) L.qwave[i] = c.take((size_t)n * 4);
  for (int i = 0; i < 2; i++) L.qwg[i] = c.take((size_t)L.cap_wg * 16);
  for (int i = 0; i < 2; i++) L.bm[i] = c.take((size_t)L.nwords * 4);
  L.hv = c.take((size_t)L.nwords * 4);
  L.df = c.take((size_t)L.nwords * 4);
  L.total = c.off;
  return L;
}

// Whether a graph takes the edge-parallel kernel, which holds it whole.
static bool ss_wg_whole(int64_t n, int64_t m) { return n <= kTinyN && m <= kLdsM; }

// The one-workgroup kernel whose LDS state fits the graph (n <= kCuMaxN).
using SsWgKernel = void (*)(SsArgs, const int32_t*, const int64_t*, int32_t, int32_t, int32_t,
                            dawn_run_info*);
template <int WT, bool MULTI>
static SsWgKernel ss_wg_kernel(int64_t n, int64_t m) {
  if (ss_wg_whole(n, m))
    return m <= 4 * kLdsThreads   ? ss_lds_kernel<WT, 4, MULTI>
           : m <= 8 * kLdsThreads ? ss_lds_kernel<WT, 8, MULTI>
                                  : ss_lds_kernel<WT, 16, MULTI>;
  return n <= kTinyN    ? ss_cu_kernel<WT, kTinyN, MULTI>
         : n <= kCuMidN ? ss_cu_kernel<WT, kCuMidN, MULTI>
                        : ss_cu_kernel<WT, kCuMaxN, MULTI>;
}

// Multi-source calls on small graphs: one workgroup per source, which costs
// the same for 1 to 256 sources (one per compute unit) and grows with m; a
// tile costs less per edge the fewer its columns.  Measured (us, tile against
// workgroups), ER n = 32,768: m = 131,072, k = 2 656 / 284, k = 256 2279 /
// 354; m = 262,144, k = 2 528 / 371; m = 524,288, k = 2 542 / 656, k = 64 1296
// / 744; m = 1,048,576, k = 64 1284 / 1314, k = 256 4044 / 1260.  R-MAT scale
// 15: m = 524,288, k = 16 628 / 657, k = 64 741 / 679; m = 1,048,576, k = 256
// 2305 / 1561.
bool ss_multi_fits(int64_t n, int64_t m, int32_t k) {
  const Tuning& T = tuning();
  const int64_t most = (int64_t)T.small_m * (k >= 128 ? 8 : k >= 32 ? 4 : k >= 2 ? 2 : 1);
  return T.mode == 0 && T.tile_step_launches > 0 && T.validate == 0 && n <= kCuMaxN && m <= most;
}

__global__ void ss_multi_info_kernel(dawn_run_info* info) {
  if (threadIdx.x == 0) {
    *info = dawn_run_info{};
    info->converged = 1;
  }
}

dawn_status ss_multi_run(const int32_t* rowptr, const int32_t* colidx, const void* w, int wt,
                         int32_t n, int32_t m, const int32_t* sources, int32_t k, void* dist,
                         dawn_run_info* info, hipStream_t stream) {
  SsArgs A{};
  A.rowptr = rowptr;
  A.colidx = colidx;
  A.w = static_cast<const uint32_t*>(w);
  A.dist = static_cast<uint32_t*>(dist);
  A.n = n;
  A.m = m;
  A.skip = tuning().ss_skip;
  A.latch = dev_info().latch;
  const SsWgKernel kern = wt == kWF32    ? ss_wg_kernel<kWF32, true>(n, m)
                          : wt == kWUNIT ? ss_wg_kernel<kWUNIT, true>(n, m)
                                         : ss_wg_kernel<kWU32, true>(n, m);
  if (info) hipLaunchKernelGGL(ss_multi_info_kernel, dim3(1), dim3(64), 0, stream, info);
  // A launch holds fewer than 2^32 threads: whole tiles of sources, 2^21 workgroups
  // at most.
  const int32_t tile = std::min(k, tuning().tile_k), most = (1 << 21) / tile * tile;
  void* tk = ktimer_begin(stream);
  int32_t launches = 0;
  for (int32_t j0 = 0; j0 < k; j0 += std::min(most, k - j0)) {
    const int32_t cnt = std::min(most, k - j0);
    hipLaunchKernelGGL(kern, dim3((unsigned)cnt), dim3(1024), 0, stream, A, sources + j0, nullptr,
                       cnt, tile, 0, info);
    A.dist += (size_t)cnt * (size_t)n;
    launches++;
  }
  ktimer_end(tk, stream, launches);
  return hip_check(hipGetLastError(), "one workgroup per source");
}

Residency ss_persistent_residency(int threads) {
  if (threads <= 0) threads = 1024;
  return residency_of(ss_persistent_kernel<kWU32, false>, threads);
}

// Workgroups of a persistent launch on a graph of even degrees.  A barrier costs 1.9
// us with 64 and 3.3 us with 256, and the steps of sparse or small graphs are bound
// by it and by one chain of loads; steps with many edges need the whole chip.  m *
// (m / n) tells the two apart.  Measured at 256 / 128 / 64 / 32 workgroups: grid 2048 x 2048
// 43.5 / 37.9 / 41.2 / 50.1 ms, grid 512 x 512 12.9 / 11.3 / 10.4 / 9.2 ms, ER
// n = 100,000 420 / 359 / 352 / 366 us, ER n = 1,000,000 910 / 863 / 1053 /
// 1519 us, R-MAT scale 16 447 / 439 / 444 / 460 us, scale 20 820 / 952 / 1320 /
// 2129 us.  Powers of two: workgroup b runs on XCD b mod 8, and with 125 or 112
// workgroups the 2048 x 2048 grid took 43.4 and 40.4 ms, against 37.9 with 128
// (the rows below each other of a grid then stay on one XCD).  With 2 to 5 edges per
// vertex, at 32 / 64 / 128 / 256: ER n = 300,000 with 2 543 / 572 / 625 / 751 us, n =
// 1,000,000 with 2 1074 / 937 / 933 / 1088, with 3 1168 / 927 / 835 / 946, grid 1024 x
// 1024 17.3 / 17.7 / 18.4 / 21.3 ms.
static int ss_even_wgs(int64_t n, int64_t m, int resident) {
  const double grow = (double)m * ((double)m / (double)n) / (double)(1 << 26);
  int wgs = m < 6 * n && n < 1 << 19 ? 32 : 64;
  while (wgs < resident && grow * 128 > wgs * 1.42) wgs *= 2;
  return std::min(wgs, resident);
}

// And on others, whose frontiers are wide after a few steps however few edges a
// vertex has.  At 32 / 64 / 128 / 256: R-MAT scale 18 with 2 edges per vertex 238 /
// 216 / 212 / 229 us, scale 20 with 4 1005 / 706 / 570 / 564, scale 21 with 4 1504 /
// 930 / 679 / 588, scale 22 with 4 2319 / 1348 / 902 / 762; a star of 50,000 leaves
// 128 / 129 / 129 / 132, of 2,000,000 882 / 553 / 374 / 240.
static int ss_wide_wgs(int64_t m, int resident) {
  return std::min(m < 3 << 17 ? 64 : m < 1 << 20 ? 128 : resident, resident);
}

// Tier bounds of persistent launches, relative to the tuning's (which are those of
// step launches, with twice the wavefronts per compute unit): a step waits for
// its slowest wavefront, so long rows are cut finer.  Measured at 2048 / 8192
// (wave-tier rows, chunk) against 768 / 2048: R-MAT scale 16 432 / 310 us, 17
// 690 / 508, 18 (int32) 643 / 542, 19 662 / 512, 20 809 / 797, 21 1396 / 1335,
// 22 2233 / 2035, 22 hop counts 1074 / 953; 2048 / 2048 gives 409 us and 657 us
// at scales 16 and 19, 512 / 1024 2271 us at 22.
static void ss_persistent_tiers(SsArgs& A) {
  const Tuning& T = tuning();
  A.t_wave = std::max(std::max(64, T.t_lane), T.t_wave * 3 / 8);
  A.t_chunk = std::max(256, T.t_chunk / 4);
}

// The workgroups of a persistent launch, which the kernel chooses from by the rows'
// lengths: tuning field `grid` where it is set, else the rules', and what the device
// holds at once.
struct SsWgs {
  uint32_t even, wide;
  void limit(int most) {
    even = std::min(even, (uint32_t)most);
    wide = std::min(wide, (uint32_t)most);
  }
};
template <int WT, bool COPIES>
static SsWgs ss_persistent_wgs(int64_t n, int64_t m, int threads) {
  const int most = std::min(residency_of(ss_persistent_kernel<WT, COPIES>, threads).grid, kMaxGrid);
  if (tuning().grid > 0) {
    const uint32_t g = (uint32_t)std::min(tuning().grid, most);
    return SsWgs{g, g};
  }
  return SsWgs{(uint32_t)ss_even_wgs(n, m, most), (uint32_t)ss_wide_wgs(m, most)};
}

template <int WT, bool COPIES>
static dawn_status ss_launch_persistent(const SsArgs& a, SsWgs wgs, int threads, dawn_run_info* info,
                                        hipStream_t stream, bool capture) {
  const int grid = (int)std::max(wgs.even, wgs.wide);
  SsArgs args = a;
  // Copies: LDS for the rows left for later in the blocks after each wavefront's
  // first (1000 x 1021 grid, 32 sources: 58.9 ms; 62.7 with them in memory), as far as
  // the resident workgroups' LDS (with 2 KiB of each for its allocation's rounding)
  // and 64 KiB a workgroup go.
  int32_t nheld = 0;
  if (COPIES) {
    const Residency r = residency_of(ss_persistent_kernel<WT, COPIES>, threads);
    const int64_t W = threads / kWave, block = (int64_t)std::min(wgs.even, wgs.wide) * W * kWave * 32;
    const int64_t room = std::min<int64_t>(65536, 163840 / std::max(r.per_cu, 1) - 2048) - r.lds;
    nheld = (int32_t)std::max<int64_t>(
        0, std::min<int64_t>((a.n + block - 1) / block - 1, room / (W * kWave * 4)));
  }
  const unsigned dyn = (unsigned)nheld * (unsigned)threads * 4u;
  void* ptrs[] = {&args, &info, &nheld, &wgs.even, &wgs.wide};
  hipError_t e;
  const PersistentGate gate(stream, grid);
  void* tk = capture ? nullptr : ktimer_begin(stream);
  if (!capture && dev_info().coop && tuning().coop) {
    e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&ss_persistent_kernel<WT, COPIES>),
                                   dim3(grid), dim3(threads), ptrs, dyn, stream);
  } else {
    hipLaunchKernelGGL((ss_persistent_kernel<WT, COPIES>), dim3(grid), dim3(threads), dyn, stream, args,
                       info, nheld, wgs.even, wgs.wide);
    e = hipGetLastError();
  }
  ktimer_end(tk, stream, 1);
  return hip_check(e, "persistent launch");
}

template <int WT>
static dawn_status ss_run_t(const SsArgs& A, const int32_t* rowptr, const int32_t* colidx,
                            const SsSeeds& seeds, const SsLayout& L, dawn_run_info* info,
                            hipStream_t stream, bool capture, int* wgs) {
  const Tuning& T = tuning();
  const DevInfo& di = dev_info();
  // mode 0 picks: one workgroup when m <= small_m; step launches first when
  // m >= step_min_m (by default never); otherwise the persistent launch alone.
  // Measured, persistent against step launches of 512-thread workgroups: R-MAT
  // scale 22 2.21 / 2.55 ms, scale 20 0.81 / 0.99 ms, 64 ER graphs (118M edges)
  // 5.74 / 6.10 ms, the 2048^2 grid 43.4 / 47.2 ms.
  int mode = T.mode;
  // (Pull steps need step launches: large graphs with a reverse graph keep them,
  // and so do captured runs of that size.)
  // One workgroup's LDS where it holds the run; past that, a kernel with the state
  // in global memory took 1606 us on an ER graph of 60,000 vertices and 120,000
  // edges, the persistent launch 404 us.  A captured run of so few edges takes the
  // persistent launch with one workgroup (1135 us): its replays are ordered by
  // nothing, and on several streams at once they would wait for each other's
  // workgroups at grid barriers.
  const bool capturing = stream_capturing(stream), small = (int64_t)A.m <= (int64_t)T.small_m;
  const bool lone = mode == 0 && small && capturing;
  if (mode == 0) mode = small && A.n <= kCuMaxN ? 3
                        : (int64_t)A.m >= (int64_t)T.step_min_m ||
                          ((A.pull_min >= 0 || capturing) && A.m >= 1 << 25)
                            ? 1 : 2;
  const int threads = T.wg_threads > 0 ? T.wg_threads : mode == 1 ? 512 : 1024;
  const int fill_blocks = (int)std::min<int64_t>(4096, (A.n + 255) / 256 + 1);
  dawn_status st;
  if (mode == 3) {
    // one workgroup, one launch (after the optional device validation)
    if (T.validate) {
      hipLaunchKernelGGL(ss_fill_kernel<WT>, dim3(fill_blocks), dim3(256), 0, stream, A.dist,
                         (int64_t)A.n, A.bm[0], A.bm[1], L.nwords, A.ctl, nullptr, nullptr, 0, nullptr, 0,
                         A.n1, (int64_t)-1, false, nullptr, A);
      const int vb = (int)std::min<int64_t>(4096, ((int64_t)A.m + 255) / 256 + 1);
      hipLaunchKernelGGL(ss_validate_kernel, dim3(vb), dim3(256), 0, stream, rowptr, colidx, A.w,
                         A.n, A.m, (int32_t)(WT == kWF32), &A.ctl->done, &A.ctl->converged);
    }
    void* tk = capture ? nullptr : ktimer_begin(stream);
    hipLaunchKernelGGL((ss_wg_kernel<WT, false>(A.n, A.m)), dim3(1),
                       dim3(ss_wg_whole(A.n, A.m) ? kLdsThreads : threads), 0, stream, A,
                       seeds.sources_dev, seeds.voff_dev, seeds.count, seeds.source,
                       (int32_t)(T.validate != 0), info);
    ktimer_end(tk, stream, 1);
    return hip_check(hipGetLastError(), "small-graph launch");
  }
  // (a validation that fails leaves every distance INF: it comes before the seed)
  const bool placed = !seeds.sources_dev && !T.validate;
  hipLaunchKernelGGL(ss_fill_kernel<WT>, dim3(fill_blocks), dim3(256), 0, stream, A.dist,
                     (int64_t)A.n, A.bm[0], A.bm[1], L.nwords, A.ctl, rowptr, A.hv, A.t_lane, A.w,
                     (int64_t)A.m, A.n1, placed ? (int64_t)seeds.source : (int64_t)-1,
                     seeds.voff_dev != nullptr, nullptr, A);
  if (T.validate) {
    const int vb = (int)std::min<int64_t>(4096, ((int64_t)A.m + 255) / 256 + 1);
    hipLaunchKernelGGL(ss_validate_kernel, dim3(vb), dim3(256), 0, stream, rowptr, colidx, A.w,
                       A.n, A.m, (int32_t)(WT == kWF32), &A.ctl->done, &A.ctl->converged);
  }
  if (!placed)
    hipLaunchKernelGGL(ss_seed_kernel<WT>, dim3(1), dim3(256), 0, stream, A, seeds.sources_dev,
                       seeds.voff_dev, seeds.count, seeds.source);
  if ((st = hip_check(hipGetLastError(), "init launch")) != DAWN_OK) return st;

  // Mode 1: `step_launches` step launches, then one persistent launch for
  // whatever steps remain.  Nothing waits on the host: every launch after the
  // run has ended returns at once, so the call is a fixed launch sequence that
  // a HIP graph can capture.
  if (mode == 1) {
    const int grid = T.grid > 0 ? T.grid : 4 * di.cus;
    auto stepk = A.pull_min >= 0 ? ss_step_kernel<WT, true> : ss_step_kernel<WT, false>;
    const int chunk = (int)std::min<int64_t>(T.step_launches, (int64_t)A.n + 1);
    void* tk = capture ? nullptr : ktimer_begin(stream);
    for (int s = 0; s < chunk; s++)
      hipLaunchKernelGGL(stepk, dim3(grid), dim3(threads), 0, stream, A);
    ktimer_end(tk, stream, chunk);
    if ((st = hip_check(hipGetLastError(), "step launches")) != DAWN_OK) return st;
  }
  SsArgs a = A;
  a.counted = mode == 1 && A.pull_min >= 0;
  ss_persistent_tiers(a);
  a.pull_min = -1;  // pull steps need step launches (the last workgroup clears the bitmap)
  SsWgs pw = ss_persistent_wgs<WT, false>(A.n, A.m, threads);
  if (T.ss_tail_grid > 0) pw.limit(T.ss_tail_grid);
  if (lone) pw.limit(1);
  if (wgs) *wgs = (int)std::max(pw.even, pw.wide);
  if ((st = ss_launch_persistent<WT, false>(a, pw, threads, info, stream, capture)) != DAWN_OK)
    return st;
  if constexpr (WT == kWI32) {
    hipLaunchKernelGGL(ss_decode_i32_kernel, dim3(fill_blocks), dim3(256), 0, stream, A.dist,
                       (int64_t)A.n);
    st = hip_check(hipGetLastError(), "decode launch");
  }
  return st;
}

// ---------------------------------------------------------------------------
// a few sources on one graph: copies
//
// k sources run as one single-source run on k copies of the graph: vertex v of
// source j has the id j * n + v in the distances (the [k x n] output itself),
// the bitmaps and the queues, and the rows are read from the one CSR.  Every
// step then serves all sources with one barrier, rows are deferred as in a
// single-source run, and there is no tile to fill, scan or transpose.
// ---------------------------------------------------------------------------
// A source outside [0, n) ends the run before its first step (converged = -1),
// as in a tile, whose distances then hold the sources' zeros, of hop counts nothing.
template <int WT>
__global__ void ss_copy_seed_kernel(SsArgs A, const int32_t* sources, int32_t count) {
  SsCtl* C = A.ctl;
  bool bad = false;
  for (int j = threadIdx.x; j < count; j += blockDim.x) bad |= sources[j] < 0 || sources[j] >= A.n1;
  bad = __syncthreads_or(bad) != 0;
  if (bad && threadIdx.x == 0) {
    st_agent_i(&C->converged, -1);
    st_agent(&C->done, 1u);
  }
  if (bad && WT == kWUNIT) return;
  for (int j = threadIdx.x; j < count; j += blockDim.x) {
    const int32_t s = sources[j];
    if (s < 0 || s >= A.n1) continue;
    const int32_t x = j * A.n1 + s;
    A.dist[x] = zero_key<WT>();
    if (bad) continue;
    atomicOr(&A.bm[0][x >> 5], 1u << (x & 31));
    const int32_t start = A.rowptr[s], deg = A.rowptr[s + 1] - start;
    if (deg <= A.t_lane) continue;
    if (deg <= A.t_wave) {
      A.qwave[0][atomicAdd(&C->cnt[0][1].v, 1u)] = x;
    } else {
      const uint32_t nch = (deg + A.t_chunk - 1) / A.t_chunk;
      const uint32_t p = atomicAdd(&C->cnt[0][2].v, nch);
      for (uint32_t c = 0; c < nch; c++) {
        const int32_t off = (int32_t)c * A.t_chunk;
        if (p + c < A.cap_wg)
          A.qwg[0][p + c] = make_int4(x, start + off, min(A.t_chunk, deg - off), c == 0);
      }
    }
  }
}

// Workspace of a run on copies: the queues hold each long row of each copy once
// per step.
static SsLayout ss_copies_layout(int64_t n, int64_t m, int64_t k) {
  const Tuning& T = tuning();
  SsLayout L{};
  Carver c;
  L.cap_v = (uint32_t)(k * std::min<int64_t>(n, m / (T.t_lane + 1)) + 1);
  SsArgs A{};
  ss_persistent_tiers(A);
  L.cap_wg = (uint32_t)(k * (m / (A.t_wave + 1) + m / A.t_chunk) + 1);
  L.nwords = (k * n + 31) / 32;
  L.ctl = c.take(sizeof(SsCtl));
  for (int i = 0; i < 2; i++) L.qwave[i] = c.take((size_t)L.cap_v * 4);
  for (int i = 0; i < 2; i++) L.qwg[i] = c.take((size_t)L.cap_wg * 16);
  for (int i = 0; i < 2; i++) L.bm[i] = c.take((size_t)L.nwords * 4);
  L.hv = c.take((size_t)L.nwords * 4);
  L.df = c.take((size_t)L.nwords * 4);
  L.total = c.off;
  return L;
}

// The work of a run on copies grows with k; a tile reads each row once for all
// its sources, but pays for whole 64-column rows and scans every vertex each
// step.  So copies win where a call is short of work: with few sources, and in
// long runs of small steps (grids) at any of the k here.  Long runs show when the
// tile's step launches are over: what is left of a run then goes on on copies.
// Measured (us, copies / tile; weighted): k = 8: ER of 6 to 12 edges per vertex, n =
// 100,000 and 600,000, 0.75 to 0.9 of the tile's time; R-MAT scales 18 and 20, 8 to
// 30 edges per vertex, 0.94 to 1.09; k = 2: ER 0.59 to 0.87, R-MAT 0.69 to 0.97.  k
// = 16: ER 0.88 to 1.08, R-MAT 1.35 to 1.87; k = 24: ER 1.02 to 1.23, R-MAT 1.62 to
// 2.37.  Fewer edges per vertex, copies / tile first: R-MAT scale 20 with 3, k = 4 786
// / 906, k = 8 1257 / 1248, scale 20 with 5, k = 4 1077 / 1107, k = 8 1738 / 1574; ER n
// = 100,000 with 3, k = 4 666 / 727, n = 600,000, k = 4 1418 / 1469, k = 8 2518 / 2063;
// hop counts R-MAT scale 20 with 5, k = 4 556 / 720, k = 8 924 / 744.  Hop counts:
// R-MAT scale 20 with 8, k = 4 651 / 745, k = 8 1160 / 793; with 16, k = 2 558 / 840,
// k = 4 1014 / 869; with 5, k = 32 3452 / 850; ER n = 1,000,000 with 8, k = 4 758 /
// 1053, k = 8 1375 / 1255.  Grids, tile / copies / tile first: 1000 x 1021, k = 8
// 77.7 / 38.2 / 38.3 ms, k = 32 157.4 / 58.7 / 58.9 ms; 200 x 221, k = 8 - / 4.06 /
// 4.41 ms.  Tile first where copies alone lose: R-MAT scale 20 with 3, k = 32 1.81
// ms, ER n = 100,000 with 3, k = 8 837 us.
static int ss_copies_most(int64_t n, int64_t m, bool unit) {
  if (m < 6 * n) return 4;
  if (m < 12 * n) return unit ? 4 : 8;
  return unit ? 3 : 8;
}
// The most sources whose runs go on on copies (hop counts of many edges per vertex
// are over by then).
static int ss_handover_most(int64_t n, int64_t m, bool unit) {
  if (m < 6 * n) return 32;
  if (m < 12 * n) return unit ? 8 : 24;
  return 0;
}

// The frontier records of a step after which a run goes on on copies: a tile shares
// the rows of a dense step among its sources.
uint32_t ss_handover_rows(int64_t n) { return (uint32_t)std::max<int64_t>(n / 16, 16384); }

static bool ss_copies_sizes(int64_t n, int64_t m, int32_t k, size_t ws_bytes) {
  const Tuning& T = tuning();
  return T.mode == 0 && T.tile_step_launches > 0 && T.validate == 0 && k >= 2 && n >= 1024 &&
         k * n <= (int64_t)1 << 30 && ss_copies_layout(n, m, k).total <= ws_bytes;
}

bool ss_copies_fit(int64_t n, int64_t m, int32_t k, bool unit, size_t ws_bytes) {
  return k <= ss_copies_most(n, m, unit) && ss_copies_sizes(n, m, k, ws_bytes);
}

bool ss_handover_fits(int64_t n, int64_t m, int32_t k, bool unit, size_t ws_bytes) {
  return k <= ss_handover_most(n, m, unit) && ss_copies_sizes(n, m, k, ws_bytes);
}

// The arguments of a run on copies, laid out at ws.
static SsArgs ss_copies_args(const int32_t* rowptr, const int32_t* colidx, const void* w, int32_t n,
                             int32_t m, int32_t k, const SsLayout& L, void* dist, void* ws) {
  const Tuning& T = tuning();
  char* base = static_cast<char*>(ws);
  SsArgs A{};
  A.rowptr = rowptr;
  A.colidx = colidx;
  A.w = static_cast<const uint32_t*>(w);
  A.dist = static_cast<uint32_t*>(dist);
  A.n = k * n;
  A.n1 = n;
  A.inv1 = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)n);
  A.nf_work = kNfWork * copies_work(k);
  A.m = m;
  A.src = -1;
  A.skip = T.ss_skip;
  A.pull_min = -1;
  A.t_lane = T.t_lane;
  ss_persistent_tiers(A);
  for (int i = 0; i < 2; i++) {
    A.qwave[i] = reinterpret_cast<int32_t*>(base + L.qwave[i]);
    A.qwg[i] = reinterpret_cast<int4*>(base + L.qwg[i]);
    A.bm[i] = reinterpret_cast<uint32_t*>(base + L.bm[i]);
  }
  A.hv = reinterpret_cast<uint32_t*>(base + L.hv);
  A.df = reinterpret_cast<uint32_t*>(base + L.df);
  A.cap_v = L.cap_v;
  A.cap_wg = L.cap_wg;
  A.ctl = reinterpret_cast<SsCtl*>(base + L.ctl);
  A.bar_ticks = (unsigned long long)T.barrier_ms * kTicksPerMs;
  A.latch = dev_info().latch;
  return A;
}

// The launches of a run on copies: `start` (placing its frontier) between the fill
// and the persistent launch.
template <int WT, typename F>
static dawn_status ss_copies_launch(const SsArgs& A, const SsLayout& L, uint32_t* dist, int32_t k,
                                    const uint32_t* over, dawn_run_info* info, hipStream_t stream,
                                    F&& start) {
  const int threads = tuning().wg_threads > 0 ? tuning().wg_threads : 1024;
  const int fill_blocks = (int)std::min<int64_t>(4096, ((int64_t)A.n + 255) / 256 + 1);
  hipLaunchKernelGGL(ss_fill_kernel<WT>, dim3(fill_blocks), dim3(256), 0, stream, dist,
                     (int64_t)A.n, A.bm[0], A.bm[1], L.nwords, A.ctl, A.rowptr, A.hv, A.t_lane, A.w,
                     (int64_t)A.m, A.n1, (int64_t)-1, false, over, A);
  start();
  return ss_launch_persistent<WT, true>(A, ss_persistent_wgs<WT, true>(A.n, (int64_t)k * A.m, threads),
                                        threads, info, stream, false);
}

template <int WT>
static dawn_status ss_copies_run_t(const SsArgs& A, const SsLayout& L, const int32_t* sources,
                                   int32_t k, dawn_run_info* info, hipStream_t stream) {
  return ss_copies_launch<WT>(A, L, A.dist, k, nullptr, info, stream, [&] {
    hipLaunchKernelGGL(ss_copy_seed_kernel<WT>, dim3(1), dim3(64), 0, stream, A, sources, k);
  });
}

dawn_status ss_copies_run(const int32_t* rowptr, const int32_t* colidx, const void* w, int wt,
                          int32_t n, int32_t m, const int32_t* sources, int32_t k, void* dist,
                          void* ws, dawn_run_info* info, hipStream_t stream) {
  const SsLayout L = ss_copies_layout(n, m, k);
  const SsArgs A = ss_copies_args(rowptr, colidx, w, n, m, k, L, dist, ws);
  if (wt == kWF32) return ss_copies_run_t<kWF32>(A, L, sources, k, info, stream);
  if (wt == kWUNIT) return ss_copies_run_t<kWUNIT>(A, L, sources, k, info, stream);
  return ss_copies_run_t<kWU32>(A, L, sources, k, info, stream);
}

// From a tile (one segment) that is not done to a run on copies: the frontier's
// masks become bits, rows longer than t_lane are queued, and the counters and the
// step go on.  The tile's distances have been stored; of hop counts those of the
// frontier, which a tile takes down in its next compaction, are stored here.
template <int WT>
__global__ void __launch_bounds__(256) ss_handover_kernel(SsArgs A, TileArgs t, int32_t k) {
  SsCtl* C = A.ctl;
  const TileCtl* T = t.ctl;
  if (T->done) return;  // (every read here is of an earlier launch's words)
  const uint32_t step = T->step;
  const int cur = step & 1, rc = step % kRot;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    unsigned long long fe = 0, es = 0, im = 0, sa = 0, se = 0;
    for (int i = 0; i < kCtrStripes; i++) {
      fe += T->ctr[i].fe;
      es += T->ctr[i].es;
      im += T->ctr[i].im;
      sa += T->ctr[i].sa;
      se += T->ctr[i].se;
    }
    C->step = step;
    C->ctr.fe = sa;
    C->ctr.es = se;
    C->ctr.im = im;
    C->u_rows = fe - sa;
    C->u_edges = es - se;
    if (T->overflow) atomicOr(&C->overflow, 1u);
  }
  const unsigned long long* mk = t.mk[step % 3];
  const int lane = lane_id();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; v0 < A.n1; v0 += stride) {
    const int64_t v = v0 + lane;
    const unsigned long long m = v < A.n1 ? mk[v] : 0ull;
    if (__ballot(m != 0ull) == 0ull) continue;
    int32_t start = 0, deg = 0;
    if (m) {
      start = A.rowptr[v];
      deg = A.rowptr[v + 1] - start;
    }
    for (int j = 0; j < k; j++) {
      const bool on = (m >> j) & 1ull;
      const unsigned long long b = __ballot(on);
      if (b == 0ull) continue;
      // 64 bits from bit j * n1 + v0 on: parts of up to three words
      const int64_t bit0 = (int64_t)j * A.n1 + v0;
      const int sh = (int)(bit0 & 31);
      const uint32_t part = lane == 0   ? (uint32_t)(b << sh)
                            : lane == 1 ? (uint32_t)(b >> (32 - sh))
                            : lane == 2 && sh ? (uint32_t)(b >> (64 - sh))
                                              : 0u;
      if (part) atomicOr(&A.bm[cur][(bit0 >> 5) + lane], part);
      if (!on) continue;
      const int32_t x = j * A.n1 + (int32_t)v;
      if (WT == kWUNIT) A.dist[x] = step;
      if (deg <= A.t_lane) continue;
      if (deg <= A.t_wave) {
        const uint32_t p = atomicAdd(&C->cnt[rc][1].v, 1u);
        if (p < A.cap_v) A.qwave[cur][p] = x;
        else atomicOr(&C->overflow, 1u);
      } else {
        const uint32_t nch = (uint32_t)((deg + A.t_chunk - 1) / A.t_chunk);
        const uint32_t p = atomicAdd(&C->cnt[rc][2].v, nch);
        for (uint32_t c = 0; c < nch; c++) {
          const int32_t off = (int32_t)c * A.t_chunk;
          if (p + c < A.cap_wg)
            A.qwg[cur][p + c] = make_int4(x, start + off, min(A.t_chunk, deg - off), c == 0);
          else
            atomicOr(&C->overflow, 1u);
        }
      }
    }
  }
}

template <int WT>
static dawn_status ss_handover_t(const SsArgs& A, const SsLayout& L, const TileArgs& tile, int32_t k,
                                 dawn_run_info* info, hipStream_t stream) {
  return ss_copies_launch<WT>(A, L, nullptr, k, &tile.ctl->done, info, stream, [&] {
    const int blocks = (int)std::min<int64_t>(2048, ((int64_t)A.n1 + 255) / 256);
    hipLaunchKernelGGL(ss_handover_kernel<WT>, dim3(blocks), dim3(256), 0, stream, A, tile, k);
  });
}

dawn_status ss_handover(const TileArgs& tile, int wt, int32_t k, void* dist, void* ws,
                        dawn_run_info* info, hipStream_t stream) {
  const SsLayout L = ss_copies_layout(tile.n, tile.m, k);
  const SsArgs A =
      ss_copies_args(tile.rowptr, tile.colidx, tile.w, tile.n, tile.m, k, L, dist, ws);
  if (wt == kWF32) return ss_handover_t<kWF32>(A, L, tile, k, info, stream);
  if (wt == kWUNIT) return ss_handover_t<kWUNIT>(A, L, tile, k, info, stream);
  return ss_handover_t<kWU32>(A, L, tile, k, info, stream);
}

dawn_status ss_run(const int32_t* rowptr, const int32_t* colidx, const void* w, int wt,
                   int32_t n, int32_t m, const SsSeeds& seeds, bool guard_source, void* dist,
                   void* ws, dawn_run_info* info, hipStream_t stream, bool capture,
                   const void* tgraph, int* wgs) {
  if (wgs) *wgs = 1;
  const Tuning& T = tuning();
  const SsLayout L = ss_layout(n, m);
  char* base = static_cast<char*>(ws);
  SsArgs A{};
  A.rowptr = rowptr;
  A.colidx = colidx;
  A.w = static_cast<const uint32_t*>(w);
  A.dist = static_cast<uint32_t*>(dist);
  A.n = n;
  A.n1 = n;
  A.nf_work = kNfWork;
  A.m = m;
  A.src = guard_source ? seeds.source : -1;
  A.t_lane = T.t_lane;
  A.skip = T.ss_skip;
  A.T = TGraph{};
  A.pull_min = -1;
  if (tgraph && T.ss_pull <= 1000) {
    A.T = tgraph_view(tgraph, n, m);
    A.pull_min = (long long)m * T.ss_pull / 1000;
  }
  A.t_wave = T.t_wave;
  A.t_chunk = T.t_chunk;
  for (int i = 0; i < 2; i++) {
    A.qwave[i] = reinterpret_cast<int32_t*>(base + L.qwave[i]);
    A.qwg[i] = reinterpret_cast<int4*>(base + L.qwg[i]);
    A.bm[i] = reinterpret_cast<uint32_t*>(base + L.bm[i]);
  }
  A.hv = reinterpret_cast<uint32_t*>(base + L.hv);
  A.df = reinterpret_cast<uint32_t*>(base + L.df);
  A.cap_v = L.cap_v;
  A.cap_wg = L.cap_wg;
  A.ctl = reinterpret_cast<SsCtl*>(base + L.ctl);
  A.bar_ticks = (unsigned long long)T.barrier_ms * kTicksPerMs;
  A.latch = dev_info().latch;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
    capture = true;
  if (wt == kWF32) return ss_run_t<kWF32>(A, rowptr, colidx, seeds, L, info, stream, capture, wgs);
  if (wt == kWUNIT) return ss_run_t<kWUNIT>(A, rowptr, colidx, seeds, L, info, stream, capture, wgs);
  if (wt == kWI32) return ss_run_t<kWI32>(A, rowptr, colidx, seeds, L, info, stream, capture, wgs);
  return ss_run_t<kWU32>(A, rowptr, colidx, seeds, L, info, stream, capture, wgs);
}

}  // namespace dawn
