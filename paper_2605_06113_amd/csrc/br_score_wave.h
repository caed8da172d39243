// K2 + K3 on one wavefront per cluster: the snapshot reductions best_g (best worker of each waiting request) and best_i
// (best request of each worker), without scoring every pair where the scores' shape decides.
//
// best_g, lanes = requests in arrival order.  BR-0: eq. (br0-Fscore) does not fall with the margin, and every worker
// whose margin the request does not exceed gives it the same score, its length.  So the best worker is the one of lowest
// index among the eligible workers with L_g <= M - s, and if there is none the lightest eligible one (lowest index on
// ties): two instructions per (worker, register) instead of a score.  BR-H: likewise the worker of lowest index whose
// horizon-min margin the request does not exceed (br_penalty_shows); the few requests that exceed all of them are scored,
// one at a time with the workers side by side, or against one worker after the other where they are many.
// best_i, lanes = workers: over the sorted list (br_list.h, copied to LDS) each worker finds the neighbours of its
// smallest margin by binary search and compares their two scores, all workers side by side (why those two: see pick in
// br_assign_kernel.h); where the peak of eq. (brh-Fscore) may be elsewhere the worker's requests are all scored.
// The round of the same wave goes on with the sorted list.
// 4096 clusters, G = 32, H = 4, 250 waiting: whole pass 297 us with every pair scored for best_g, 281.5 by the margins;
// 1531 clusters, G = 13, queues of 307, BR-0: 17.7 us in a block per cluster that scored all pairs twice, 8.8 so.
#pragma once

#include <type_traits>

#include "br_device.h"
#include "br_list.h"

// Worker state of a round: lane g holds worker g; envelope and totals are uniform.  HB: offsets beyond h = 0 that are
// carried (0: BR-0, 4: H <= 4, BR_HP); those beyond H repeat offset H, so that a minimum over all of them is one over
// the horizon (their discount is zero).
template <int HB>
struct BrRoundState {
  static constexpr int NH = HB + 1;
  int nn, cap;        // requests held, free slots
  int Lh[NH], Mh[NH]; // projected loads, envelope
  int S_tot;
};

// BR-H: bounds used where only the neighbours of the smallest margin are scored.  e = 8e-7 (alpha D + beta D) s_max bounds
// the distance of a computed score of a single request from the exact one: at most H + 5 <= 13 roundings, each relative
// 2^-24 on terms of at most (alpha D + beta D) Delta.  Offsets h <= ho have beta d_h - alpha D > 2 e: exceeding the margin
// there alone makes the score fall by more than rounding can hide, per token.
template <int HB>
__device__ __forceinline__ void br_peak_bounds(const BrParams &p, int s_max, float &e2, int &ho) {
  e2 = 1.6e-6f * (p.aD + p.beta * p.dsum) * (float)s_max;
  ho = -1;
#pragma unroll
  for (int h = 0; h <= HB; ++h) ho = (h <= p.H && p.beta * p.d[h] - p.aD > e2) ? h : ho;  // (d falls with h)
  ho = br_uniform(ho);
}

// BR-H: does a request that exceeds any one margin compute strictly below alpha D s, what it scores within all of them?
// The penalty then sums to at least d_H (rounding keeps order), so it is enough that fl(beta d_H) reaches one unit in the
// last place of the longest request's alpha D s, 2^-23 alpha D 32768 = 0.0039 alpha D.
__device__ __forceinline__ bool br_penalty_shows(const BrParams &p) {
  float d_H = p.d[0];
#pragma unroll
  for (int h = 1; h <= BR_HP; ++h) d_H = h <= p.H ? p.d[h] : d_H;
  return p.beta * d_H >= 0.004f * p.aD;
}

// x: keys in arrival order (position first + j * 64 + lane)
template <int E, int HB>
__device__ __forceinline__ void br_snapshot_best_g(const BrParams &p, const BrOut &o, int inst, int lane, int first, int qn,
                                                   const unsigned (&x)[E], const BrRoundState<HB> &st) {
  const int G = p.G;
  const int64_t qrow = (int64_t)inst * p.Q;
  int bg[E];
#pragma unroll
  for (int j = 0; j < E; ++j) bg[j] = -1;
  const unsigned long long freem = br_ballot(lane < G && st.cap > 0);
  if constexpr (HB == 0) {
    const int Lmin = br_wave_min((freem >> lane) & 1ull ? st.Lh[0] : INT32_MAX);
    if (freem != 0ull) {
      const int glight = (int)__builtin_ctzll(br_ballot(((freem >> lane) & 1ull) && st.Lh[0] == Lmin));
      int thr[E];  // eligible and safe below it (the watermark bounds both)
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int s = (int)(x[j] >> BR_IDX_BITS);
        thr[j] = st.Mh[0] - s;
        if (p.W > 0) thr[j] = min(thr[j], p.W - s);
        bg[j] = p.W <= 0 || Lmin + s <= p.W ? glight : -1;
      }
      for (unsigned long long m = freem; m != 0ull;) {  // from the highest index down: the lowest one stays
        const int g = 63 - (int)__builtin_clzll(m);
        m &= ~(1ull << g);
        const int Lg = __builtin_amdgcn_readlane(st.Lh[0], g);
#pragma unroll
        for (int j = 0; j < E; ++j) bg[j] = Lg <= thr[j] ? g : bg[j];
      }
    }
  } else {
    const int n_free = __builtin_popcountll(freem);
    int m[HB + 1], safe = INT32_MAX;  // of the worker this lane holds: margins; the longest request within all of them
#pragma unroll
    for (int h = 0; h <= HB; ++h) m[h] = max(st.Mh[h] - st.Lh[h], 0), safe = min(safe, m[h]);
    const int room = p.W > 0 ? p.W - st.Lh[0] : INT32_MAX;
    safe = min(safe, room);
    const bool exact = br_penalty_shows(p);
    if (exact) {
      for (unsigned long long f = freem; f != 0ull;) {  // from the highest index down: the lowest one stays
        const int g = 63 - (int)__builtin_clzll(f);
        f &= ~(1ull << g);
        const int Tg = __builtin_amdgcn_readlane(safe, g);
#pragma unroll
        for (int j = 0; j < E; ++j) bg[j] = (int)(x[j] >> BR_IDX_BITS) <= Tg ? g : bg[j];
      }
    }
    bool many[E], any = false;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      many[j] = false;
      if (first + j * BR_WAVE >= qn) continue;
      const int s = (int)(x[j] >> BR_IDX_BITS);
      unsigned long long left = br_ballot(bg[j] < 0 && x[j] != 0u);
      many[j] = !exact || 2 * __builtin_popcountll(left) > n_free;
      any |= many[j];
      if (many[j]) continue;
      for (; left != 0ull; left &= left - 1ull) {  // a few: one at a time, all workers side by side
        const int l = (int)__builtin_ctzll(left);
        const int sl = __builtin_amdgcn_readlane(s, l);
        const int k = ((freem >> lane) & 1ull) && sl <= room ? br_ord(br_scoreh(p, m, sl)) : BR_KEY_NONE;
        const int km = br_wave_max(k);
        const int g = km == BR_KEY_NONE ? -1 : (int)__builtin_ctzll(br_ballot(k == km));
        bg[j] = lane == l ? g : bg[j];
      }
    }
    if (any) {  // one worker after the other, 64 requests side by side
      int bk[E];
#pragma unroll
      for (int j = 0; j < E; ++j) bk[j] = BR_KEY_NONE;
      for (unsigned long long f = freem; f != 0ull; f &= f - 1ull) {
        const int g = (int)__builtin_ctzll(f);
        int mg[HB + 1];
#pragma unroll
        for (int h = 0; h <= HB; ++h) mg[h] = __builtin_amdgcn_readlane(m[h], g);
        const int room_g = __builtin_amdgcn_readlane(room, g);
#pragma unroll
        for (int j = 0; j < E; ++j) {
          if (!many[j]) continue;
          const int s = (int)(x[j] >> BR_IDX_BITS);
          const int k = br_ord(br_scoreh(p, mg, s));
          const bool better = s <= room_g && k > bk[j];
          bk[j] = better ? k : bk[j];
          bg[j] = better ? g : bg[j];
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int i = first + j * BR_WAVE + lane;
    if (i < p.Q) o.best_g[qrow + i] = i < qn ? bg[j] : -1;
  }
}

// positions from `first` on that hold no request
__device__ __forceinline__ void br_snapshot_rest(const BrParams &p, const BrOut &o, int inst, int lane, int first) {
  for (int i = first + lane; i < p.Q; i += BR_WAVE) o.best_g[(int64_t)inst * p.Q + i] = -1;
}

// first position of the LDS list (n entries) whose key lies below T
template <int E>
__device__ __forceinline__ int br_list_first_below(const int *lst, int n, unsigned T) {
  int b = 0;
#pragma unroll
  for (int step = E * BR_WAVE; step > 0; step >>= 1) {
    const int q = b + step;
    const unsigned e = (unsigned)lst[br_list_at<E>(min(q, n) - 1)];
    b = q <= n && e >= T ? q : b;
  }
  return b;
}

// x: the sorted list, lst: its LDS copy; qn >= 1
template <int E, int HB>
__device__ __forceinline__ void br_snapshot_best_i(const BrParams &p, const BrOut &o, int inst, int lane, int qn,
                                                   const unsigned (&x)[E], const int *lst, const BrRoundState<HB> &st) {
  constexpr int IDX_MASK = (1 << BR_IDX_BITS) - 1;
  const int G = p.G;
  const bool act = lane < G && st.cap > 0;
  const int room = p.W > 0 ? p.W - st.Lh[0] : INT32_MAX;
  const int room1 = min(room, BR_MAX_S_DEV) + 1;  // lengths below it are admissible
  int m[HB + 1], mn;
#pragma unroll
  for (int h = 0; h <= HB; ++h) m[h] = max(st.Mh[h] - st.Lh[h], 0);
  mn = m[0];
#pragma unroll
  for (int h = 1; h <= HB; ++h) mn = min(mn, m[h]);
  bool two = true;
  if constexpr (HB > 0) {
    float e2;
    int ho;
    br_peak_bounds<HB>(p, br_uniform((int)(x[0] >> BR_IDX_BITS)), e2, ho);
    int mo = INT32_MAX;
#pragma unroll
    for (int h = 0; h <= HB; ++h) mo = h <= ho ? min(mo, m[h]) : mo;
    two = mo == mn;
  } else {
    if (G == 1) mn = BR_MAX_S_DEV + 1;  // every score is zero: the first admissible entry
  }
  const unsigned T = (unsigned)max(min(mn, room1), 1) << BR_IDX_BITS;
  const int b = br_list_first_below<E>(lst, qn, T);
  const unsigned lo = b < qn ? (unsigned)lst[br_list_at<E>(b)] : 0u;
  unsigned hi = b > 0 ? (unsigned)lst[br_list_at<E>(b - 1)] : 0u;
  const int sh = (int)(hi >> BR_IDX_BITS), sl = (int)(lo >> BR_IDX_BITS);
  if (sh >= room1) hi = 0u;
  int kh, kl;
  if constexpr (HB > 0) {
    kh = br_ord(br_scoreh(p, m, sh)), kl = br_ord(br_scoreh(p, m, sl));
  } else {
    kh = sh - G * max(sh - mn, 0), kl = sl;
  }
  const bool useh = hi != 0u && (lo == 0u || kh >= kl);
  unsigned key = lo;
  if (br_ballot(useh && act) != 0ull) {  // the first of its length
    const int b2 = br_list_first_below<E>(lst, qn, (unsigned)(sh + 1) << BR_IDX_BITS);
    if (useh) key = (unsigned)lst[br_list_at<E>(min(b2, qn - 1))];
  }
  if constexpr (HB > 0) {
    for (unsigned long long bad = br_ballot(act && !two); bad != 0ull; bad &= bad - 1ull) {
      const int g = (int)__builtin_ctzll(bad);
      int mg[HB + 1];
#pragma unroll
      for (int h = 0; h <= HB; ++h) mg[h] = __builtin_amdgcn_readlane(m[h], g);
      const unsigned Tr = (unsigned)max(__builtin_amdgcn_readlane(room1, g), 1) << BR_IDX_BITS;
      int bk = BR_KEY_NONE;
      unsigned bx = 0u;
#pragma unroll
      for (int j = 0; j < E; ++j) {  // positions rise with j and with the lane: the first best stays
        const int k = br_ord(br_scoreh(p, mg, (int)(x[j] >> BR_IDX_BITS)));
        if (x[j] != 0u && x[j] < Tr && k > bk) bk = k, bx = x[j];
      }
      const int km = br_wave_max(bk);
      const unsigned best = km == BR_KEY_NONE ? 0u
                                              : (unsigned)__builtin_amdgcn_readlane((int)bx, (int)__builtin_ctzll(br_ballot(bk == km)));
      key = lane == g ? best : key;
    }
  }
  if (lane < G) o.best_i[(int64_t)inst * G + lane] = act && key != 0u ? IDX_MASK - (int)(key & IDX_MASK) : -1;
}

// nothing waits or no worker has a free slot
__device__ __forceinline__ void br_snapshot_none(const BrParams &p, const BrOut &o, int inst, int lane) {
  if (o.best_g)
    for (int i = lane; i < p.Q; i += BR_WAVE) o.best_g[(int64_t)inst * p.Q + i] = -1;
  if (o.best_i && lane < p.G) o.best_i[(int64_t)inst * p.G + lane] = -1;
}

// Worker state of a cluster (step-start loads or projections), envelope and totals; lanes beyond G hold no worker.
template <int HB>
__device__ __forceinline__ void br_round_state(const BrParams &p, int lane, int n_raw, const int (&L_raw)[HB + 1],
                                               BrRoundState<HB> &st) {
  const bool act = lane < p.G;
  st.nn = act ? min(max(n_raw, 0), p.B) : p.B;
  st.cap = p.B - st.nn;
#pragma unroll
  for (int h = 0; h <= HB; ++h) st.Lh[h] = act ? L_raw[h] : BR_LOW;
#pragma unroll
  for (int h = 0; h <= HB; ++h) st.Mh[h] = st.Lh[h];
  br_wave_maxs(st.Mh);
  st.S_tot = br_wave_sum(st.cap);
}

// The step-start envelope M_h, margins m_{g,h} = (M_h - L_g(k+h))_+ and min_h m_{g,h} as the workspace shows them, from the
// registers of the wave that runs the round.  (A launch of their own took 5 us of 4096 clusters with G = 32, H = 4 and
// 3.7 us of a single cluster: whole pass 281.5 -> 275.0 and 57.5 -> 52.9 us.)
template <int HB>
__device__ __forceinline__ void br_store_margins(const BrParams &p, int inst, int lane, const BrRoundState<HB> &st) {
  const int64_t wrow = (int64_t)inst * p.G + lane;
  int mn = INT32_MAX;
#pragma unroll
  for (int h = 0; h <= HB; ++h) {
    if (h <= p.H) {
      const int m = st.Mh[h] - st.Lh[h];
      mn = min(mn, m);
      if (lane < p.G) p.mh[wrow * (p.H + 1) + h] = m;
      if (lane == 0) p.Mh[(int64_t)inst * (p.H + 1) + h] = st.Mh[h];
    }
  }
  if (lane < p.G) p.minm[wrow] = mn;
}

// Decode steps applied ahead of the round (br_k_project_advance): what a worker's list lost and its load change, handed to
// the round in the words of its margins, which the round is about to write (one offset at least beyond h = 0, so there are two).
__device__ __forceinline__ void br_ahead_store(const BrParams &p, int64_t row, int lost, int dL) {
  p.mh[row * (p.H + 1)] = lost;
  p.mh[row * (p.H + 1) + 1] = dL;
}
// LDS of a cluster: [0..64) per worker: entries its list lost ahead of the round, [64..128) load change of the old entries,
// [128..192) list length at the start of the step.
#define BR_AHEAD_WORDS 192

// Loads of a cluster's worker words and queue lengths: everything that does not need the queue length, requested before
// the first result is used (lanes without a worker read worker 0's words).  STEPS: with what br_ahead_store left, if it did.
template <int HB>
struct BrClusterIn {
  int q0, cnt, n, L[HB + 1], lost, dL;
};
template <int HB, bool STEPS = false>
__device__ __forceinline__ void br_cluster_load(const BrParams &p, const BrArr &a, int inst, int lane, BrClusterIn<HB> &in) {
  const int64_t wrow = (int64_t)inst * p.G + (lane < p.G ? lane : 0);
  const int q0 = p.qlen[inst], cnt = a.count ? a.count[inst] : 0;
  in.n = p.n[wrow];
  if constexpr (HB == 0) {
    in.L[0] = p.L[wrow];
  } else {
#pragma unroll
    for (int h = 0; h <= HB; ++h) in.L[h] = p.Lh[wrow * (p.H + 1) + min(h, p.H)];
  }
  in.lost = 0, in.dL = 0;
  if constexpr (STEPS) {
    if (p.adv_t > 0) in.lost = p.mh[wrow * (p.H + 1)], in.dL = p.mh[wrow * (p.H + 1) + 1];
  }
  in.q0 = br_uniform(min(max(q0, 0), p.Q));
  in.cnt = br_uniform(min(max(cnt, 0), a.arr_cap));
}

// Keys of the waiting set in arrival order (E * 64 of them from position `first` on, the set's qn first), straight from
// the queue and the arrivals: one batch of unconditional loads (addresses by select, an entry beyond the set reads the
// cluster's first queue word).
template <int E>
__device__ __forceinline__ void br_keys_load(const BrParams &p, const BrArr &a, int inst, int q0, int qn, int first, int lane,
                                             unsigned (&x)[E]) {
  constexpr int IDX_MASK = (1 << BR_IDX_BITS) - 1;
  const int64_t qrow = (int64_t)inst * p.Q, arow = (int64_t)inst * a.arr_cap;
  int v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int i = first + j * BR_WAVE + lane;
    const bool ina = i >= q0 && i < qn;
    v[j] = *(ina ? a.s + (arow + (i - q0)) : p.qs + (qrow + (i < q0 ? i : 0)));
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int i = first + j * BR_WAVE + lane;
    const int s = min(max(v[j], 1), BR_MAX_S_DEV);
    x[j] = i < qn ? ((unsigned)s << BR_IDX_BITS) | (unsigned)(IDX_MASK - i) : 0u;
  }
}

// The list of a cluster of qn >= 1 requests, sorted (and copied to `lst` where `copy` or best_i asks for it), with the
// snapshot reductions on the way if they are asked for.
template <int E, int HB, bool SCORES>
__device__ __forceinline__ void br_list_build(const BrParams &p, const BrArr &a, const BrOut &o, int inst, int lane, int q0,
                                              int qn, int *lst, const BrRoundState<HB> &st, unsigned (&x)[E]) {
  br_keys_load<E>(p, a, inst, q0, qn, 0, lane, x);
  if constexpr (SCORES) {
    if (o.best_g) {
      br_snapshot_best_g<E, HB>(p, o, inst, lane, 0, qn, x, st);
      br_snapshot_rest(p, o, inst, lane, E * BR_WAVE);
    }
  }
  br_list_sort<E>(x, lane);
  if constexpr (SCORES) {
    if (o.best_i) {
      br_list_store<E>(x, lst, lane);
      br_wave_sync();
      br_snapshot_best_i<E, HB>(p, o, inst, lane, qn, x, lst, st);
      br_wave_sync();
    }
  }
}

// BR-0 scores of 64 requests (from position i0 on, n of them) against every worker, as a wave writes them into the matrix:
// four neighbours per lane and store (element e of the cluster's rows is request e / G, worker e % G; recip_g: the
// rounded-up reciprocal of G, exact for e < 2^17).  s, m: length of the request, margin of the worker this lane holds;
// t: 128 words of LDS.
__device__ __forceinline__ void br_matrix_rows(const BrParams &p, const BrOut &o, int inst, int lane, int i0, int n, int s, int m,
                                               unsigned recip_g, int *t) {
  const int G = p.G, total = n * G;
  int *F = (int *)o.F + ((int64_t)inst * p.Q + i0) * G;
  t[lane] = s, t[BR_WAVE + lane] = m;
  br_wave_sync();
  auto score = [&](int e) -> int {
    const int i = G == 1 ? e : (int)__umulhi((unsigned)e, recip_g);
    return br_score0(G, t[BR_WAVE + (e - i * G)], t[i & 63]);
  };
  if (((uintptr_t)F & 15u) == 0) {  // (64 rows are whole 16-byte units: so for all of a cluster's or none)
    for (int e = 4 * lane; e < total; e += 4 * BR_WAVE) {
      if (e + 3 < total) {
        *reinterpret_cast<int4 *>(F + e) = make_int4(score(e), score(e + 1), score(e + 2), score(e + 3));
      } else {
        for (int k = e; k < total; ++k) F[k] = score(k);
      }
    }
  } else {
    for (int e = lane; e < total; e += BR_WAVE) F[e] = score(e);
  }
  br_wave_sync();
}

// What a round's caller asked for beside it (matrix, best_g, best_i), on wave h of the nh that a cluster's block has for it
// while another wave runs the round: none of it is on the round's path, and nothing here is read after the return.
// lst: BR_LIST_WORDS(EM) + 128 words of LDS of this wave's.
template <int EM, int HB>
__device__ __forceinline__ void br_snapshot_helper(const BrParams &p, const BrArr &a, const BrOut &o, int inst, int lane, int h,
                                                   int nh, unsigned recip_g, int *lst) {
  BrClusterIn<HB> in;
  br_cluster_load<HB>(p, a, inst, lane, in);
  BrRoundState<HB> st;
  br_round_state<HB>(p, lane, in.n, in.L, st);
  const int qn = in.q0 + min(in.cnt, p.Q - in.q0);
  const bool none = st.S_tot == 0 || qn == 0;
  if constexpr (HB == 0) {
    if (o.F) {
      const int m = st.Mh[0] - st.Lh[0];
      for (int i0 = h * BR_WAVE; i0 < qn; i0 += nh * BR_WAVE) {
        unsigned x[1];
        br_keys_load<1>(p, a, inst, in.q0, qn, i0, lane, x);
        br_matrix_rows(p, o, inst, lane, i0, min(qn - i0, BR_WAVE), (int)(x[0] >> BR_IDX_BITS), m, recip_g, lst + BR_LIST_WORDS(EM));
      }
    }
  }
  if (none) {
    if (h == 0) br_snapshot_none(p, o, inst, lane);
    return;
  }
  // one wave: both reductions off one list; more: the last one sorts, the others share out the requests
  BrOut mine = o;
  if (nh > 1) {
    if (h < nh - 1) {
      if (o.best_g) {
        for (int i0 = h * 2 * BR_WAVE; i0 < p.Q; i0 += (nh - 1) * 2 * BR_WAVE) {
          unsigned x[2];
          br_keys_load<2>(p, a, inst, in.q0, qn, i0, lane, x);
          br_snapshot_best_g<2, HB>(p, o, inst, lane, i0, qn, x, st);
        }
      }
      return;
    }
    mine.best_g = nullptr;
  }
  if (!mine.best_g && !mine.best_i) return;
  auto with = [&](auto e) {
    constexpr int E = decltype(e)::value;
    unsigned x[E];
    br_list_build<E, HB, true>(p, a, mine, inst, lane, in.q0, qn, lst, st, x);
  };
  if (qn <= BR_WAVE)
    with(std::integral_constant<int, 1>{});
  else if (EM == 4 || qn <= 4 * BR_WAVE)
    with(std::integral_constant<int, 4>{});
  else if constexpr (EM > 4)
    with(std::integral_constant<int, EM>{});
}

// The snapshot reductions of a cluster whose round has a block of four waves (queues beyond 1024, shorter ones where br_block_serves)
// on the three that do not run it
// (h = 0..2): requests shared out 128 at a time, best_i on the last one.  lst: the sorted list where more than 256 wait, else
// room for it.
template <int HB>
__device__ __forceinline__ void br_snapshot_coop(const BrParams &p, const BrArr &a, const BrOut &o, int inst, int lane, int h,
                                                 int q0, int qn, bool run, int *lst, const BrRoundState<HB> &st) {
  if (!run) {
    if (h == 0) br_snapshot_none(p, o, inst, lane);
    return;
  }
  if (o.best_g) {
    for (int i0 = h * 2 * BR_WAVE; i0 < p.Q; i0 += 3 * 2 * BR_WAVE) {
      unsigned x[2];
      br_keys_load<2>(p, a, inst, q0, qn, i0, lane, x);
      br_snapshot_best_g<2, HB>(p, o, inst, lane, i0, qn, x, st);
    }
  }
  if (!o.best_i || h != 2) return;
  if (qn > 4 * BR_WAVE) {
    unsigned x[32];
    br_list_load<32>(x, lst, lane, 0, qn);
    br_snapshot_best_i<32, HB>(p, o, inst, lane, qn, x, lst, st);
  } else {
    BrOut mine = o;
    mine.best_g = nullptr;
    unsigned x[4];
    br_list_build<4, HB, true>(p, a, mine, inst, lane, q0, qn, lst, st, x);
  }
}
