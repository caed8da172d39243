// Shared tail of the assignment kernels: writes the admitted requests into their workers'
// lists, emits the per-entry outputs in arrival order, compacts the waiting queue in place and
// stores worker state and statistics.  Everything here is lane-parallel over arrival positions; `bound` (by arrival
// position: worker << 16 | slot, or -1) comes from the round.  An entry's words are read once, whether it leaves for a
// list or stays in the queue: one memory round trip per group of four blocks of 64 entries.
#pragma once

#include <type_traits>

#include "br_advance_seg.h"
#include "br_device.h"
#include "br_score_wave.h"

#define BR_STAT(o, inst, k) (o).stats[(int64_t)(inst) * 16 + (k)]

struct BrRoundCounts {
  int admitted, stage1, pops, guard, wdrop;
  long long I_before;
};

// What the tail needs of the kernel arguments.  The assignment kernels take (BrParams, BrArr,
// BrOut) by value; keeping all of that in scalar registers across the admission loops starves
// them, so the tail reads its own copy from the kernel-argument segment when it starts.
struct BrTailArgs {
  int32_t *L, *n, *kv, *rem;
  float *pred;
  int32_t *qlen, *qs, *qo, *qid;
  float *qpred;
  const int32_t *as, *ao, *aid;
  const float *apred;
  int32_t *assign, *assign_id;
  long long *stats;
  int32_t G, B, Bs, Q, P, Pq, C, arr_cap, adv_t;
};

static_assert(sizeof(BrParams) == 272 && sizeof(BrArr) == 48 && sizeof(BrOut) == 48, "kernel argument layout");

__device__ __forceinline__ BrTailArgs br_tail_args() {
  typedef __attribute__((address_space(4))) const char kchar_t;
  typedef __attribute__((address_space(4))) const BrParams kparams_t;
  typedef __attribute__((address_space(4))) const BrArr karr_t;
  typedef __attribute__((address_space(4))) const BrOut kout_t;
  kchar_t *ka = (kchar_t *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(ka));  // the loads below may not move above this point
  kparams_t *kp = (kparams_t *)ka;
  karr_t *kaa = (karr_t *)(ka + sizeof(BrParams));
  kout_t *ko = (kout_t *)(ka + sizeof(BrParams) + sizeof(BrArr));
  BrTailArgs t;
  t.L = kp->L, t.n = kp->n, t.kv = kp->kv, t.rem = kp->rem, t.pred = kp->pred;
  t.qlen = kp->qlen, t.qs = kp->qs, t.qo = kp->qo, t.qid = kp->qid, t.qpred = kp->qpred;
  t.as = kaa->s, t.ao = kaa->o, t.aid = kaa->id, t.apred = kaa->pred;
  t.assign = ko->assign, t.assign_id = ko->assign_id, t.stats = ko->stats;
  t.G = kp->G, t.B = kp->B, t.Bs = kp->Bs, t.Q = kp->Q, t.P = kp->P, t.Pq = kp->Pq, t.C = kp->C, t.adv_t = kp->adv_t;
  t.arr_cap = kaa->arr_cap;
  return t;
}

// ---- pieces of the epilogue, each over GR blocks of 64 arrival positions starting at block j0 ----

// How prediction rows travel with the requests: not at all, by single floats, or as 16-byte words where rows are whole ones
// and lie on such boundaries (the workspace's always do, the caller's arrivals may not).  One cluster, rows of eight, a queue of
// 2048: whole pass 43.0 us by single floats, 37.0 so.  Decided once per cluster: decided per row, the two forms share
// registers and every row is waited for (whole pass of two clusters, rows of
// five, a queue of 723 55.7 us so, 54.7 without; of the one cluster with a queue of 2048 34.1 and 33.0).
#define BR_ROWS_NONE 0
#define BR_ROWS_FLOAT 1
#define BR_ROWS_WIDE 2
template <bool PRED, typename F>
__device__ __forceinline__ void br_with_rows(const BrTailArgs &t, F &&body) {
  if constexpr (!PRED)
    body(std::integral_constant<int, BR_ROWS_NONE>{});
  else if ((t.Pq & 3) == 0 && ((uintptr_t)t.apred & 15u) == 0)
    body(std::integral_constant<int, BR_ROWS_WIDE>{});
  else
    body(std::integral_constant<int, BR_ROWS_FLOAT>{});
}

// What those positions hold and where they went.
template <int GR, int ROWS, int NQ = BR_HP>  // NQ: words of a row at most
struct BrQueueGroup {
  int bound[GR], id[GR], sq[GR], oq[GR];
  float pr[ROWS != BR_ROWS_NONE ? GR : 1][NQ];
};

template <int ROWS, int NQ>
__device__ __forceinline__ void br_row_load(const float *src, int Pq, float (&r)[NQ]) {
  if constexpr (ROWS == BR_ROWS_WIDE) {
#pragma unroll
    for (int q = 0; q < NQ; q += 4)
      if (q < Pq) {
        const float4 v = *reinterpret_cast<const float4 *>(src + q);
        r[q] = v.x, r[q + 1] = v.y, r[q + 2] = v.z, r[q + 3] = v.w;
      }
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (q < Pq) r[q] = src[q];
  }
}
template <int ROWS, int NQ>
__device__ __forceinline__ void br_row_store(float *dst, int Pq, const float (&r)[NQ]) {
  if constexpr (ROWS == BR_ROWS_WIDE) {
#pragma unroll
    for (int q = 0; q < NQ; q += 4)
      if (q < Pq) *reinterpret_cast<float4 *>(dst + q) = make_float4(r[q], r[q + 1], r[q + 2], r[q + 3]);
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (q < Pq) dst[q] = r[q];
  }
}

// An entry's words (length, output length, id) of those positions.  Queues of up to 512: requested before the round, so
// that they arrive while the list is sorted and the epilogue starts without a memory trip of its own (1024 clusters, round
// and decode step on two waves: whole pass 23.4 -> 22.4 us; one cluster on host arrays 37.9 -> 37.0).
template <int GR>
struct BrQueueWords {
  int id[GR], sq[GR], oq[GR];
};

template <int GR>
__device__ __forceinline__ void br_queue_words(const int32_t *qs, const int32_t *qo, const int32_t *qid, const int32_t *as,
                                               const int32_t *ao, const int32_t *aid, int64_t qrow, int64_t arow, int lane,
                                               int j0, int q0, int qn, BrQueueWords<GR> &v) {
#pragma unroll
  for (int u = 0; u < GR; ++u) {
    const int i = (j0 + u) * BR_WAVE + lane;
    v.id[u] = -1, v.sq[u] = 1, v.oq[u] = 1;
    if (i < qn) {
      const bool old = i < q0;
      const int64_t aat = arow + (i - q0);
      v.sq[u] = *(old ? qs + (qrow + i) : as + aat);
      v.oq[u] = *(old ? qo + (qrow + i) : ao + aat);
      v.id[u] = old ? qid[qrow + i] : (aid ? aid[aat] : i - q0);
    }
  }
}

// Where they went (from LDS) and their prediction rows; `words` as read before, or null: read here.
template <int GR, int ROWS, int NQ>
__device__ __forceinline__ void br_queue_load(const BrTailArgs &t, int inst, int lane, int j0, int q0, int qn, const int *bound,
                                              BrQueueGroup<GR, ROWS, NQ> &v, const BrQueueWords<GR> *words = nullptr) {
  const int64_t qrow = (int64_t)inst * t.Q, arow = (int64_t)inst * t.arr_cap;
  BrQueueWords<GR> w;
  if (words)
    w = *words;
  else
    br_queue_words<GR>(t.qs, t.qo, t.qid, t.as, t.ao, t.aid, qrow, arow, lane, j0, q0, qn, w);
#pragma unroll
  for (int u = 0; u < GR; ++u) {
    const int i = (j0 + u) * BR_WAVE + lane;
    v.bound[u] = -1, v.id[u] = w.id[u], v.sq[u] = w.sq[u], v.oq[u] = w.oq[u];
    if (i < qn) {
      v.bound[u] = bound[i];
      if constexpr (ROWS != BR_ROWS_NONE) {
        const bool old = i < q0;
        const float *src = old ? t.qpred + (qrow + i) * t.Pq : t.apred + (arow + (i - q0)) * t.Pq;
        br_row_load<ROWS>(src, t.Pq, v.pr[u]);
      }
    }
  }
}

// ---- BR-H with decode steps in the call: the projection's pass over the lists has applied them to the old entries
// (br_k_project_advance), and the round's epilogue appends its admissions behind the survivors, already advanced.  Same final
// state as the round followed by the decode steps (see the split step below).
// Admitted requests whose output is used up within the decode steps leave at once.  Who they are is collected in bit masks
// by order of admission, a worker's from word `at` on, as many words as its admissions take, so that the others go straight to
// their final slots.  lds: [0..64) `at` per worker, [64..128) kv that leaves, then the masks (64 words and one per 32 entries that wait).
#define BR_DEAD_WORDS(E) (3 * BR_WAVE + 2 * (E))
struct BrAhead {
  const int *lost, *n0;  // null: no decode steps
  int *dead;             // null: everybody outlives them
  int t;
};

__device__ __forceinline__ void br_dead_clear(int lane, int a_g, int words, int *dead) {
  const int mine = (a_g + 31) >> 5;
  dead[lane] = br_scan_sum(mine) - mine;
  dead[BR_WAVE + lane] = 0;
  for (int k = lane; k < words; k += BR_WAVE) dead[2 * BR_WAVE + k] = 0;
}

__device__ __forceinline__ void br_dead_mark(const BrAhead &h, int bound, int s, int o) {
  if (bound >= 0 && max(o, 1) <= h.t) {
    const int g = (bound >> 16) & 63, k = (bound & 0xffff) - h.n0[g];
    atomicOr(&h.dead[2 * BR_WAVE + h.dead[g] + (k >> 5)], 1 << (k & 31));
    atomicAdd(&h.dead[BR_WAVE + g], min(max(s, 1), BR_MAX_S_DEV));
  }
}

// the admissions before the k-th of worker g that leave at once
__device__ __forceinline__ int br_dead_before(const BrAhead &h, int g, int k) {
  const int *m = h.dead + 2 * BR_WAVE + h.dead[g];
  int c = __builtin_popcount((unsigned)m[k >> 5] & ((1u << (k & 31)) - 1u));
  for (int i = 0; i < k >> 5; ++i) c += __builtin_popcount((unsigned)m[i]);
  return c;
}

// load and length of worker `lane` after the decode steps: Lcur, nn right after the round
__device__ __forceinline__ void br_ahead_workers(const BrTailArgs &t, int inst, int lane, int Lcur, int nn, const int *ahead,
                                                 const BrAhead &h) {
  int a_g = nn - ahead[2 * BR_WAVE + lane], n = nn - ahead[lane], L = Lcur + ahead[BR_WAVE + lane];
  if (h.dead) {
    int gone = 0;
    for (int k = 0; k < (a_g + 31) >> 5; ++k) gone += __builtin_popcount((unsigned)h.dead[2 * BR_WAVE + h.dead[lane] + k]);
    a_g -= gone, n -= gone, L -= h.dead[BR_WAVE + lane];
  }
  if (lane < t.G) {
    t.L[(int64_t)inst * t.G + lane] = L + a_g * h.t;
    t.n[(int64_t)inst * t.G + lane] = n;
  }
}

// List entries of the requests that were bound.
template <int GR, int ROWS, int NQ>
__device__ __forceinline__ void br_commit_store(const BrTailArgs &t, int inst, const BrQueueGroup<GR, ROWS, NQ> &v, float c0,
                                                const BrAhead &h = BrAhead{nullptr, nullptr, nullptr, 0}) {
#pragma unroll
  for (int u = 0; u < GR; ++u) {
    const int g = v.bound[u] >> 16, slot = v.bound[u] & 0xffff;
    if (v.bound[u] >= 0 && g < t.G && slot < t.B && max(v.oq[u], 1) > h.t) {
      int64_t row = ((int64_t)inst * t.G + g) * t.Bs + slot;
      if (h.lost) row -= h.lost[g];  // behind the old survivors
      if (h.dead) row -= br_dead_before(h, g, slot - h.n0[g]);
      t.kv[row] = min(max(v.sq[u], 1), BR_MAX_S_DEV) + h.t;
      t.rem[row] = max(v.oq[u], 1) - h.t;
      if constexpr (ROWS != BR_ROWS_NONE) {
        br_row_store<ROWS>(t.pred + row * t.P, t.Pq, v.pr[u]);
        if (t.P == 3 && t.Pq == 0) {  // maintained estimate: first query at age 0, nothing generated yet
          t.pred[row * 3] = c0;
          t.pred[row * 3 + 1] = 0.0f;
          t.pred[row * 3 + 2] = 0.0f;
        }
      }
    }
  }
}

// Outputs of those positions in arrival order, and their deferred requests to queue positions `kept`
// onwards (order preserved); `kept` moves on by the number stored.
template <int GR, int ROWS, int NQ>
__device__ __forceinline__ void br_queue_store(const BrTailArgs &t, int inst, int lane, int j0, int q0, int qn,
                                               const BrQueueGroup<GR, ROWS, NQ> &v, int &kept) {
  const int64_t qrow = (int64_t)inst * t.Q;
#pragma unroll
  for (int u = 0; u < GR; ++u) {
    const int i = (j0 + u) * BR_WAVE + lane;
    if ((j0 + u) * BR_WAVE < t.Q) {
      if (i < t.Q) {
        if (t.assign) t.assign[qrow + i] = v.bound[u] >> 16;
        if (t.assign_id) t.assign_id[qrow + i] = v.id[u];
      }
      const bool keep = i < qn && v.bound[u] < 0;
      const unsigned long long bal = br_ballot(keep);
      const int ni = kept + br_rank_below(bal);
      if (keep && (ni != i || i >= q0)) {
        t.qs[qrow + ni] = min(max(v.sq[u], 1), BR_MAX_S_DEV);
        t.qo[qrow + ni] = max(v.oq[u], 1);
        t.qid[qrow + ni] = v.id[u];
        if constexpr (ROWS != BR_ROWS_NONE) br_row_store<ROWS>(t.qpred + (qrow + ni) * t.Pq, t.Pq, v.pr[u]);
      }
      kept += __builtin_popcountll(bal);
    }
  }
}

// Worker state and the statistics of the round (one wave).
__device__ __forceinline__ void br_write_state(const BrTailArgs &t, int inst, int lane, int q0, int qn, int cnt, int kept,
                                               int Lcur, int nn, const BrRoundCounts &rc, bool store_workers = true) {
  const int G = t.G;
  const bool act = lane < G;
  const int64_t wrow = (int64_t)inst * G + lane;
  if (act && store_workers) {
    t.L[wrow] = Lcur;
    t.n[wrow] = nn;
  }
  const int Lact = Lcur;
  const int Lmax = br_wave_max(Lact);
  const int Lmin = br_wave_min(act ? Lact : INT32_MAX);
  const int over = __builtin_popcountll(br_ballot(act && t.C > 0 && Lact > t.C));
  const int wide = __builtin_popcountll(br_ballot(act && Lact >= (1 << 25)));  // beyond what the packed worker keys order
  long long sumL = 0;
  if (t.stats) {
    const int L0 = act ? Lcur : 0;
    sumL = ((long long)br_wave_sum(L0 >> 16) << 16) + br_wave_sum(L0 & 0xffff);
  }
  if (lane == 0) {
    t.qlen[inst] = kept;
    if (t.stats) {
      BR_STAT(t, inst, 0) = rc.admitted;
      BR_STAT(t, inst, 1) = kept;
      BR_STAT(t, inst, 2) = cnt - (qn - q0);
      BR_STAT(t, inst, 3) = rc.stage1;
      BR_STAT(t, inst, 4) = rc.pops;
      BR_STAT(t, inst, 5) = rc.guard;
      BR_STAT(t, inst, 6) = over;
      BR_STAT(t, inst, 7) = rc.I_before;
      BR_STAT(t, inst, 8) = (long long)G * Lmax - sumL;
      BR_STAT(t, inst, 9) = (long long)Lmax - Lmin;
      BR_STAT(t, inst, 10) = qn;
      BR_STAT(t, inst, 11) = rc.wdrop;
      BR_STAT(t, inst, 12) = wide;
      for (int k = 13; k < 16; ++k) BR_STAT(t, inst, k) = 0;
    }
  }
}

// The epilogue on the wave that ran the round.  The queue is compacted in place: a deferred entry moves to a position
// at or below its own, inside or before its group, and later groups read only beyond it.
template <int E, bool PRED>
__device__ __forceinline__ void br_assign_epilogue(int inst, int lane, int q0, int qn, int cnt, const int *bound, int Lcur, int nn,
                                                   const BrRoundCounts &rc, float c0, const BrQueueWords<E> *words = nullptr) {
  const BrTailArgs t = br_tail_args();
  constexpr int GR = E < 4 ? E : 4;
  int kept = 0;
  br_with_rows<PRED>(t, [&](auto rows) {
#pragma unroll
    for (int j0 = 0; j0 < E; j0 += GR) {
      if (j0 * BR_WAVE < t.Q) {
        BrQueueGroup<GR, decltype(rows)::value> v;
        if (words) {
          BrQueueWords<GR> w;
#pragma unroll
          for (int u = 0; u < GR; ++u) w.id[u] = words->id[j0 + u], w.sq[u] = words->sq[j0 + u], w.oq[u] = words->oq[j0 + u];
          br_queue_load(t, inst, lane, j0, q0, qn, bound, v, &w);
        } else {
          br_queue_load(t, inst, lane, j0, q0, qn, bound, v);
        }
        br_commit_store(t, inst, v, c0);
        br_queue_store(t, inst, lane, j0, q0, qn, v, kept);
      }
    }
  });
  br_write_state(t, inst, lane, q0, qn, cnt, kept, Lcur, nn, rc);
}

// The same for BR-H, whose decode steps may have been applied to the old entries ahead of the round.  dead: BR_DEAD_WORDS(E).
// The first rows are requested with the entries' words: a wait for a load waits for the stores before it too.
template <int E, int NQ>
__device__ __forceinline__ void br_assign_epilogue_ahead(int inst, int lane, int q0, int qn, int cnt, const int *bound, int Lcur,
                                                         int nn, const BrRoundCounts &rc, float c0, const int *ahead, int *dead) {
  const BrTailArgs t = br_tail_args();
  constexpr int GR = E < 4 ? E : 4;
  BrAhead h{nullptr, nullptr, nullptr, t.adv_t};
  BrQueueWords<E> words;
  br_queue_words<E>(t.qs, t.qo, t.qid, t.as, t.ao, t.aid, (int64_t)inst * t.Q, (int64_t)inst * t.arr_cap, lane, 0, q0, qn, words);
  int kept = 0;
  br_with_rows<true>(t, [&](auto rows) {
    BrQueueGroup<GR, decltype(rows)::value, NQ> v;
    auto load = [&](int j0) {
      BrQueueWords<GR> w;
#pragma unroll
      for (int u = 0; u < GR; ++u) w.id[u] = words.id[j0 + u], w.sq[u] = words.sq[j0 + u], w.oq[u] = words.oq[j0 + u];
      br_queue_load(t, inst, lane, j0, q0, qn, bound, v, &w);
    };
    load(0);
    if (h.t > 0) {
      h.lost = ahead, h.n0 = ahead + 2 * BR_WAVE;
      int b[E];
      bool short_one = false;
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int i = u * BR_WAVE + lane;
        b[u] = i < qn ? bound[i] : -1;
        short_one |= b[u] >= 0 && max(words.oq[u], 1) <= h.t;
      }
      if (br_ballot(short_one) != 0ull) {
        h.dead = dead;
        br_dead_clear(lane, nn - h.n0[lane], BR_WAVE + 2 * E, dead);
        br_wave_sync();
#pragma unroll
        for (int u = 0; u < E; ++u) br_dead_mark(h, b[u], words.sq[u], words.oq[u]);
        br_wave_sync();
      }
    }
#pragma unroll
    for (int j0 = 0; j0 < E; j0 += GR) {
      if (j0 * BR_WAVE < t.Q) {
        if (j0 > 0) load(j0);
        br_commit_store(t, inst, v, c0, h);
        br_queue_store(t, inst, lane, j0, q0, qn, v, kept);
      }
    }
  });
  br_write_state(t, inst, lane, q0, qn, cnt, kept, Lcur, nn, rc, h.t == 0);  // statistics: the state right after the round
  if (h.t > 0) br_ahead_workers(t, inst, lane, Lcur, nn, ahead, h);
}

// The epilogue on the four waves of a block (queues of up to 2048 entries): wave w owns the arrival positions
// [w*512, (w+1)*512).  Every wave requests all it will read of the queue before the barrier that precedes the first
// store, so the in-place compaction needs no order between waves; the counts of deferred requests per wave go through
// `sh` (4 words of LDS).  With `share_workers` wave 0's per-worker (load, count) are handed to every wave through `wk`
// (2 x 64 words, for a decode step split among the waves) and wave 0 leaves their store to that step.
template <bool PRED>
__device__ __forceinline__ void br_assign_epilogue_block4(int inst, int lane, int w, int q0, int qn, int cnt, const int *bound,
                                                          int *sh, int *wk, int &Lcur, int &nn, const BrRoundCounts &rc, float c0,
                                                          bool share_workers) {
  const BrTailArgs t = br_tail_args();
  if (share_workers && w == 0) wk[lane] = Lcur, wk[BR_WAVE + lane] = nn;
  __syncthreads();  // the round is over: bound[] is complete
  if (share_workers) Lcur = wk[lane], nn = wk[BR_WAVE + lane];
  int total = 0;
  br_with_rows<PRED>(t, [&](auto rows) {
    BrQueueGroup<4, decltype(rows)::value> va, vb;
    br_queue_load(t, inst, lane, w * 8, q0, qn, bound, va);
    br_queue_load(t, inst, lane, w * 8 + 4, q0, qn, bound, vb);
    int mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      mine += __builtin_popcountll(br_ballot((w * 8 + u) * BR_WAVE + lane < qn && va.bound[u] < 0)) +
              __builtin_popcountll(br_ballot((w * 8 + 4 + u) * BR_WAVE + lane < qn && vb.bound[u] < 0));
    // the loaded values must have arrived before any wave stores
    asm volatile("" ::"v"(va.sq[0]), "v"(va.sq[1]), "v"(va.sq[2]), "v"(va.sq[3]), "v"(vb.sq[0]), "v"(vb.sq[1]), "v"(vb.sq[2]),
                 "v"(vb.sq[3])
                 : "memory");
    __builtin_amdgcn_s_waitcnt(0);
    if (lane == 0) sh[w] = mine;
    __syncthreads();
    int kept = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = sh[k];
      kept += k < w ? c : 0;
      total += c;
    }
    br_commit_store(t, inst, va, c0);
    br_commit_store(t, inst, vb, c0);
    br_queue_store(t, inst, lane, w * 8, q0, qn, va, kept);
    br_queue_store(t, inst, lane, w * 8 + 4, q0, qn, vb, kept);
  });
  if (w == 0) br_write_state(t, inst, lane, q0, qn, cnt, total, Lcur, nn, rc, !share_workers);
  if (share_workers) __syncthreads();  // the lists that a wave goes on to hold entries stored by the others
}

// Late copy of the whole parameter block from the kernel-argument segment (same reason as above).
__device__ __forceinline__ BrParams br_late_params() {
  typedef __attribute__((address_space(4))) const char kchar_t;
  typedef __attribute__((address_space(4))) const BrParams kparams_t;
  kchar_t *ka = (kchar_t *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(ka));
  BrParams p;
  __builtin_memcpy(&p, (kparams_t *)ka, sizeof(BrParams));
  return p;
}

// Likewise the outputs.
__device__ __forceinline__ BrOut br_late_out() {
  typedef __attribute__((address_space(4))) const char kchar_t;
  typedef __attribute__((address_space(4))) const BrOut kout_t;
  kchar_t *ka = (kchar_t *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(ka));
  BrOut o;
  __builtin_memcpy(&o, (kout_t *)(ka + sizeof(BrParams) + sizeof(BrArr)), sizeof(BrOut));
  return o;
}

// Decode steps of one BR-0 cluster by the wave that has just routed it.  `Lcur`, `nn`: load and list length of worker `lane`
// after the round; lists [g0, g1) are this wave's; lds: BR_PLAIN_WORDS of the wave's.
// LONG as for br_advance_lists_any.
// STORE = false: loads and counts are not stored; what list g loses and its load change go to split[4 + g] and
// split[4 + 64 + g] instead (the split kernels, where another wave owns the workers' final state).
#define BR_PLAIN_WORDS (2 * BR_SEG_WORDS(0))
template <int LONG, bool STORE = true>
__device__ __forceinline__ void br_advance_cluster(int inst, int lane, int Lcur, int nn, int *lds, int g0 = 0, int g1 = 64,
                                                   int *split = nullptr) {
  const BrParams p = br_late_params();
  const int t = p.adv_t;
  br_wave_sync();  // the round's own writes into the lists are read back below
  const int G = min(p.G, g1);
  const int64_t row0 = (int64_t)__builtin_amdgcn_readfirstlane(inst) * p.G;  // scalar: list bases stay in SGPRs
  if (p.Bs <= 256) {
    const BrSegBase b = br_seg_base(p, row0);
    br_advance_lists_any<LONG>(p, t, b, lane, g0, G, nn, lds, [&](int g, const BrSegPlan &d, bool whole) {
      if constexpr (STORE) {
        const int L = __builtin_amdgcn_ds_bpermute(g << 2, Lcur);
        if (whole) {
          br_seg_at<int>(b.L, 4u * (unsigned)g) = L + d.kept * t - d.gone;
          br_seg_at<int>(b.n, 4u * (unsigned)g) = d.kept;
        }
      } else {
        const int n = __builtin_amdgcn_ds_bpermute(g << 2, nn);
        if (whole) split[4 + g] = n - d.kept, split[4 + BR_WAVE + g] = d.kept * t - d.gone;
      }
    });
    return;
  }
  // longer lists: br_adv_apply over (list, 256-slot chunk) units, UB units requested before the first is used
  constexpr int UB = 8;
  const int NC = (p.Bs + 255) >> 8, U = max(G - g0, 0) * NC;
  const int64_t rowa = row0 + g0;
  int dLw = 0, nw = nn;     // lane g: load change and new length of worker g
  int kept = 0, gone = 0;   // running state of the list in progress: survivors, kv that left
  int gl = g0, cl = 0, gp = g0, cp = 0;  // (list, chunk) cursors of the load and the update pass
  const int32_t *kl = p.kv + rowa * p.Bs, *rl = p.rem + rowa * p.Bs;  // list the load pass is at
  int32_t *kw = p.kv + rowa * p.Bs, *rw = p.rem + rowa * p.Bs;        // list the update pass is at
  for (int u0 = 0; u0 < U; u0 += UB) {
    int4 kv[UB], rem[UB];
#pragma unroll
    for (int k = 0; k < UB; ++k) {
      kv[k] = make_int4(0, 0, 0, 0), rem[k] = make_int4(0, 0, 0, 0);
      if (gl < G) br_adv_load(kl, rl, cl * 256 + 4 * lane, __builtin_amdgcn_readlane(nn, gl), kv[k], rem[k]);
      if (++cl == NC) cl = 0, ++gl, kl += p.Bs, rl += p.Bs;
    }
#pragma unroll
    for (int k = 0; k < UB; ++k) {
      if (gp < G) {
        const int ng = __builtin_amdgcn_readlane(nn, gp);
        if (cp * 256 < ng) {
          int from;
          br_adv_apply<0>(p, t, cp * 256 + 4 * lane, ng, cp * 256, kv[k], rem[k], kw, rw, nullptr, kept, gone, nullptr, from);
        }
        if (++cp == NC) {
          if (lane == gp) dLw = kept * t - gone, nw = kept;  // survivors gain t tokens each
          kept = 0, gone = 0, cp = 0, ++gp;
          kw += p.Bs, rw += p.Bs;
        }
      }
    }
  }
  if constexpr (STORE) {
    if (lane >= g0 && lane < G) {
      p.L[row0 + lane] = Lcur + dLw;
      p.n[row0 + lane] = nw;
    }
  } else {
    split[4 + lane] = nn - nw;
    split[4 + BR_WAVE + lane] = dLw;
  }
}

// Decode steps of a BR-H cluster by the wave that has just routed it (lists of up to 256 slots whose prediction rows move
// along; a SIMD's waves end their rounds one after the other, so the memory works for some while others route): Lcur, nn: load and list length of worker `lane` after the round; lds: BR_TAIL_WORDS of the wave's.
#define BR_TAIL_WORDS (2 * BR_SEG_WORDS(1))
__device__ __forceinline__ void br_advance_cluster_rows(int inst, int lane, int Lcur, int nn, int *lds) {
  const BrParams p = br_late_params();
  br_wave_sync();  // the round's own writes into the lists are read back below
  br_with_row_unit(p.P, [&](auto unit, auto upr) {
    using V = decltype(unit);
    constexpr int UPR = decltype(upr)::value;
    if (p.Bs <= 64)
      br_advance_lists<16, 2, UPR, V>(p, p.adv_t, inst, lane, Lcur, nn, lds);
    else if (p.Bs <= 128)
      br_advance_lists<32, 2, UPR, V>(p, p.adv_t, inst, lane, Lcur, nn, lds);
    else
      br_advance_lists<64, 2, UPR, V>(p, p.adv_t, inst, lane, Lcur, nn, lds);
  });
}

// ---------------------------------------------------------------- split step: round and decode step on two waves
// In the split kernels (BR-0, queues of up to 512) the decode steps of a cluster's lists as they stand at the
// start of the step are applied by a second wave (the helper) while the first runs the round; the wave that ran
// the round then appends its admissions behind the survivors, already advanced.  Same final state as the round
// followed by the decode steps: a list holds its old survivors in order, then the new survivors in admission
// order; L_g = sum of the kv held; a request whose output is used up within the t steps leaves at once.
// LDS area of one cluster: [0] flag (lists advanced), [1] flag (a third wave has read what it needs, or there is none), [4..68) per worker: entries its list lost (old length - kept),
// [68..132) per worker: load change of the old entries.
#define BR_SPLIT_WORDS 132

// The decode steps of a cluster's lists as they stand, what they lost and by how much their loads change, then the flag.
// lds: BR_PLAIN_WORDS of the wave's.
template <int LONG>
__device__ __forceinline__ void br_split_advance(const BrParams &p, int inst, int lane, int *split, int *lds) {
  const bool act = lane < p.G;
  const int n_raw = p.n[(int64_t)inst * p.G + (act ? lane : 0)];
  const int n0 = act ? min(max(n_raw, 0), p.B) : 0;
  br_advance_cluster<LONG, false>(inst, lane, 0, n0, lds, 0, 64, split);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // the lists are in place before the flag is seen
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) split[0] = 1;
}

// The epilogue of the wave that ran the round where the decode steps of the old entries are (being) applied apart: by
// another wave (split kernels), or by this one before the round.  nn0: list lengths at the start of the step.
// Admitted requests whose output is used up within the t steps leave at once: who they are per worker is collected in
// bit masks (by order of admission) in `lds` (320 words), so that the others go straight to their final slots.
template <int E>
__device__ __forceinline__ void br_assign_epilogue_split(int inst, int lane, int q0, int qn, int cnt, const int *bound, int Lcur,
                                                         int nn, int nn0, const BrRoundCounts &rc, int *split, int *lds,
                                                         const BrQueueWords<E> *words) {
  const BrTailArgs t = br_tail_args();
  const int G = t.G, tt = t.adv_t;
  BrQueueGroup<E, BR_ROWS_NONE> v;
  br_queue_load(t, inst, lane, 0, q0, qn, bound, v, words);
  // the helpers are done with this cluster's lists and queue (they never wait for anything: the flags always come)
  while (__atomic_load_n(split, __ATOMIC_RELAXED) == 0 || __atomic_load_n(split + 1, __ATOMIC_RELAXED) == 0)
    __builtin_amdgcn_s_sleep(4);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // (or this wave's own stores to the lists)
  const int lost = split[4 + lane], dold = split[4 + BR_WAVE + lane];  // lane g: worker g
  const int kept0 = nn0 - lost, a_g = nn - nn0;                        // old survivors, admissions of this round
  int nfin = kept0 + a_g, Lfin = Lcur + dold + a_g * tt;               // if every admitted request outlives the t steps
  bool slow = false;
  if (rc.admitted > 0) {
    int *dead = lds, *dead_kv = lds + 2 * BR_WAVE, *first = lds + 3 * BR_WAVE;  // per worker
    bool short_one = false, far = false;
#pragma unroll
    for (int u = 0; u < E; ++u) short_one |= v.bound[u] >= 0 && max(v.oq[u], 1) <= tt;
    const bool some = br_ballot(short_one) != 0ull;
    if (some) {
      dead[2 * lane] = 0, dead[2 * lane + 1] = 0, dead_kv[lane] = 0, first[lane] = nn0;
      br_wave_sync();
#pragma unroll
      for (int u = 0; u < E; ++u) {
        if (v.bound[u] >= 0 && max(v.oq[u], 1) <= tt) {
          const int g = (v.bound[u] >> 16) & 63, k = (v.bound[u] & 0xffff) - first[g];
          far |= k >= BR_WAVE;
          if (k < BR_WAVE) {
            atomicOr(&dead[2 * g + (k >> 5)], 1 << (k & 31));
            atomicAdd(&dead_kv[g], min(max(v.sq[u], 1), BR_MAX_S_DEV));
          }
        }
      }
      slow = br_ballot(far) != 0ull;  // beyond the masks: the lists are compacted below
      br_wave_sync();
      if (!slow) {
        const int gone = __builtin_popcount(dead[2 * lane]) + __builtin_popcount(dead[2 * lane + 1]);
        nfin -= gone;
        Lfin = Lcur + dold - dead_kv[lane] + (a_g - gone) * tt;
      }
    }
    const int add = slow ? 0 : tt;
#pragma unroll
    for (int u = 0; u < E; ++u) {
      const int g = v.bound[u] >> 16, slot = v.bound[u] & 0xffff;
      if (v.bound[u] >= 0 && g < G && slot < t.B) {
        int64_t row = ((int64_t)inst * G + g) * t.Bs + (slot - split[4 + g]);  // behind the old survivors
        bool live = true;
        if (some && !slow) {
          const int k = slot - first[g];
          const unsigned lo = (unsigned)dead[2 * g], hi = (unsigned)dead[2 * g + 1];
          live = max(v.oq[u], 1) > tt;
          row -= k >= 32 ? __builtin_popcount(lo) + __builtin_popcount(k < 64 ? hi & ((1u << (k & 31)) - 1u) : hi)
                         : __builtin_popcount(lo & ((1u << k) - 1u));
        }
        if (live) {
          t.kv[row] = min(max(v.sq[u], 1), BR_MAX_S_DEV) + add;
          t.rem[row] = max(v.oq[u], 1) - add;
        }
      }
    }
  }
  int keptq = 0;
  br_queue_store(t, inst, lane, 0, q0, qn, v, keptq);
  br_write_state(t, inst, lane, q0, qn, cnt, keptq, Lcur, nn, rc, false);  // statistics: the state right after the round
  if (slow) {
    // The admissions sit behind the old survivors as admitted (kv = s, rem = o); per worker the decode steps
    // now run over that stretch alone: who outlives them moves up and gains t tokens, the others leave.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the stores above are read back below
    __builtin_amdgcn_wave_barrier();
    for (int g = 0; g < G; ++g) {
      const int ag = __builtin_amdgcn_readlane(a_g, g);
      if (ag <= 0) continue;
      const int64_t base = ((int64_t)inst * G + g) * t.Bs + __builtin_amdgcn_readlane(kept0, g);
      int keptn = 0, gone = 0;
      for (int c0 = 0; c0 < ag; c0 += BR_WAVE) {
        const int j = c0 + lane;
        const bool in = j < ag;
        const int kv = in ? t.kv[base + j] : 0, rem = in ? t.rem[base + j] : 0;
        const bool stay = in && rem > tt;
        const unsigned long long bal = br_ballot(stay);
        const int dst = keptn + br_rank_below(bal);
        if (stay) {  // at or below its own position; the chunk was read whole before
          t.kv[base + dst] = kv + tt;
          t.rem[base + dst] = rem - tt;
        }
        gone += br_wave_sum((in && !stay) ? kv : 0);
        keptn += (int)__builtin_popcountll(bal);
      }
      if (lane == g) {
        nfin = kept0 + keptn;
        Lfin = Lcur + dold - gone + keptn * tt;
      }
    }
  }
  if (lane < G) {
    const int64_t wrow = (int64_t)inst * G + lane;
    t.L[wrow] = Lfin;
    t.n[wrow] = nfin;
  }
}

