// Sequential two-stage assignment of one scheduling round (Appendix, Alg. BR-0 / Alg. BR-H),
// one wavefront per cluster.
//
// The round is a dependent chain: every admission changes L_g, possibly the envelope M and
// with it every margin.  The chain therefore stays inside one wave, with no block barrier and
// no HBM access on its critical path, and what bounds it is the number of instructions on it:
//   - lane g holds worker g's state (free slots, projected loads L_g(k+h), request count);
//   - the waiting set, ordered by prefill length (largest first, arrival order among equals), is a dense
//     sorted list in registers (br_list.h), E entries per lane, E chosen by the number of requests that wait: a
//     list of up to 64 is one register;
//   - "pick a worker" is a DPP reduction on packed int32 keys; Stage-2 subsets are enumerated one subset mask per lane;
//   - "pick a request" is two neighbours in the list.  Eq. (br0-Fscore) rises with the length up to the margin and (G > 1)
//     falls beyond it, so argmax_i F_g({i}) is the longest request below the margin or the shortest at or above it
//     (earliest arrival among equals).  Eq. (brh-Fscore) is concave; where exceeding any one of the smallest margins already
//     outweighs the gain (below), its peak is the smallest margin and the same two requests are compared, by their
//     computed scores; otherwise all are scored.
//
// Stage 1 is taken a whole capacity level at a time where that is provably the same as the
// one-by-one loop: the workers that share the largest free-slot count are picked once each in
// order of load, and as long as the largest waiting request still fits the next worker's
// (horizon-min) margin its score is the largest one (score = const * s in the safe regime of
// eq. (br0-Fscore) / eq. (brh-Fscore)), the envelope does not move, and the k-th lightest worker
// takes the k-th largest waiting request.  The rest of the level goes one worker at a time, except where no waiting
// request is shorter than the next worker's margin: then the workers in turn take the shortest ones, in one step
// (tail_bulk).
//
// Stage 2 of BR-0 (G > 1, no token watermark) takes the consecutive guard pops of one free-slot count in one step of
// that kind while the window stays untouched.  Stage 2 skips the subset enumeration when the window's
// smallest entry alone scores <= 0 (the starvation guard is then certain), and under a watermark sets aside in one step
// the workers for which even the shortest waiting request is too long.
//
// Ties: Stage 1 worker (most free slots, then lightest, then lowest index); Stage 2 worker
// (most free slots, then largest horizon-min margin, then lowest index); equal request scores
// resolve to the lowest sorted position; equal subset scores to the lowest mask.
//
// ADV: the wave goes on to apply the decode steps to the lists of the cluster it has routed
// (br_route_advance); a separate instantiation, so that the two kinds of launch carry distinct
// kernel names in profiles.
#pragma once

#include <type_traits>

#include "br_device.h"
#include "br_launch.h"
#include "br_list.h"
#include "br_sort.h"
#include "br_assign_common.h"
#include "br_subset_dp.h"
#include "br_subset_few.h"
#include "br_subset_halves.h"
#include "br_subset_list.h"
#include "br_score_wave.h"

// LDS of a cluster whose queue holds up to EM * 64 entries: bound [EM * 64], list copy, slots [64], what BR-H lists lost ahead of the round, Stage-2 window and
// table (BIGR), then the mailbox of shared subset searches and the bit rows of br_subset_dp.h where they are used
#define BR_SEARCH_WORDS 1344
#define BR_ROUND_WORDS(EM, HB, BIGR) ((EM) * BR_WAVE + BR_LIST_WORDS(EM) + BR_WAVE + ((EM) <= 8 && (HB) > 0 && !(BIGR) ? BR_AHEAD_WORDS : 0) + ((BIGR) ? 32 + BR_SEARCH_WORDS : 0))
// the same where the wave goes on to apply decode steps to its cluster's lists (BR-0)
#define BR_ROUND_ADV_WORDS(EM) (BR_ROUND_WORDS(EM, 0, false) > BR_PLAIN_WORDS ? BR_ROUND_WORDS(EM, 0, false) : BR_PLAIN_WORDS)
static_assert(BR_ROUND_WORDS(32, 0, false) + BR_LIST_WORDS(32) >= 4 * BR_PLAIN_WORDS, "four waves share the lists' LDS");
static_assert(BR_SEARCH_WORDS >= BR_HALVES_WORDS && BR_SEARCH_WORDS >= BR_FEW_WORDS && BR_SEARCH_WORDS >= 1024, "LDS of a subset search");

// Trips of 256 masks from which a block's four waves share a search: fewer are not worth two barriers.
#define BR_SHARE_TRIPS 4
// BR-0, limits beyond BR_FEW_MAX: trips from which the sums of the window's halves decide instead (br_subset_halves.h: about
// 6300 cycles at kmax = 6 and 200 more per request beyond; a trip is 350 to 600 cycles on one wave).
#define BR_HALVES_TRIPS 6

// Subset search of a window of up to 16 requests (Stage 2, BIGR), this wave's share of it: the best key and its lowest
// mask (uniform).  With at most half of the window per subset the admissible masks are taken from a list
// (br_subset_list.h; `hitab`: its byte tables, made here with `build`).
// Otherwise a scan over all masks: lane l keeps the lower six mask bits, the upper bits c run as passes over the table
// `hitab` of their partial sums, four passes per trip; the wave takes the trips wv, wv + nwv, ... (trips whose upper bits
// alone exceed the cardinality limit are skipped).  A lane sees its masks in ascending order and keeps the first best.
template <bool BRH, int N>
__device__ __forceinline__ void br_bigr_scan(const BrParams &p, const int (&mg)[N], const int *win, int *hitab, int w, int kmax,
                                             int room, int lane, int wv, int nwv, bool build, int &best, int &mask) {
  if (br_list_serves(w, kmax)) {
    br_list_walk(win, hitab, w, kmax, room, lane, wv, nwv, build,
                 [&](const int(&delta)[4], int(&key)[4]) {
#pragma unroll
                   for (int u = 0; u < 4; ++u) key[u] = br_score_key<BRH>(p, mg, delta[u]);
                 },
                 best, mask);
    return;
  }
  const int nhi = w > 6 ? 1 << (w - 6) : 1;
  const int nmask = 1 << w;
  int base = 0;
  for (int b = 0; b < min(w, 6); ++b) base += ((lane >> b) & 1) * (win[b] >> BR_IDX_BITS);
  const int klim = kmax - __builtin_popcount(lane);  // bits the upper part of a mask may still add on this lane
  const bool lane_ok = lane < nmask;                  // (windows below six requests use the lower lanes only)
  int bk = BR_KEY_NONE, bm = INT32_MAX;
  for (int c0 = 4 * wv; c0 < nhi; c0 += 4 * nwv) {  // four passes per trip: one 16-byte table read, independent scores
    if (__builtin_popcount(c0) > kmax) continue;     // c0 + u has at least the bits of c0: too many for every lane
    const int4 h4 = *reinterpret_cast<const int4 *>(hitab + c0);
    const int hd[4] = {h4.x, h4.y, h4.z, h4.w};
    int key[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u;
      const int delta = base + hd[u];
      bool ok = lane_ok && c < nhi && __builtin_popcount(c) <= klim && delta <= room;
      if (c == 0) ok = ok && lane != 0;  // the empty subset
      const int k = br_score_key<BRH>(p, mg, ok ? delta : 0);
      key[u] = ok ? k : BR_KEY_NONE;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (key[u] > bk) {
        bk = key[u];
        bm = (c0 + u) * BR_WAVE + lane;
      }
  }
  best = br_wave_max(bk);
  mask = best == BR_KEY_NONE ? INT32_MAX : br_wave_min(bk == best ? bm : INT32_MAX);
}


// The two stages on one wave.  x: the qn waiting requests as a sorted list.  bound [arrival position]: worker << 16 | slot
// of the requests admitted (the others keep what is there).  lst, slots, win, hitab: LDS (see BR_ROUND_WORDS).
// svc (BIGR, shared): mailbox of the block's other three waves, which serve the subset searches.
// DP (BIGR, BR-0): windows of 17 to 32 as well, by reachable sums; a kernel of its own, which the searches of every sum stay out
// of (3 clusters, G = 7, window 24, whole pass: 367 us, 376 with both in one).
template <int E, int HB, bool BIGR, bool DP = false>
__device__ __forceinline__ void br_round(const BrParams &p, int inst, int lane, int qn, unsigned (&x)[E], int *bound, int *lst,
                                         int *slots, int *win, int *hitab, int *svc, int *dprows, bool shared,
                                         BrRoundState<HB> &st, BrRoundCounts &rc) {
  constexpr int NP = E * BR_WAVE;
  constexpr bool BRH = HB > 0;
  constexpr int NH = HB + 1;
  // (what ends a level's turns is looked up at each: carried along it put the kernels of queues beyond 256 two to four words a lane into scratch memory.  4096
  // clusters, G = 16, H = 8, queues of 512, 8 steps, whole pass 181.5 -> 180.1 us, without reductions 172.1 -> 171.3; with shorter queues 188 against 179, 2048 clusters, 40 steps)
  constexpr bool LESS = HB == 8 && E == 8;
  constexpr int IDX_MASK = (1 << BR_IDX_BITS) - 1;
  constexpr int BIAS2 = 1 << 24;               // subset of <= 8 requests: score in (-2^24, 2^18]
  const int G = p.G;
  int Lh[NH], Mh[NH], nn = st.nn, cap = st.cap, S_tot = st.S_tot;
#pragma unroll
  for (int h = 0; h < NH; ++h) Lh[h] = st.Lh[h], Mh[h] = st.Mh[h];
  const bool small = G <= 16;  // every worker sits in the first row of 16 lanes: row reductions serve
  // largest free-slot count among the workers: free slots only shrink during a round, so the value is tracked
  // downwards with ballots instead of a reduction per pick
  int capmax_cur = br_wave_max(cap);
  auto cap_max = [&]() -> int {
    while (capmax_cur > 0 && br_ballot(cap == capmax_cur) == 0ull) --capmax_cur;
    return capmax_cur;
  };
  // rank of each member among the members by (load, index): lanes that are no members hold INT32_MAX
  auto rank_of = [&](int wkey) -> int {
    if (small) return br_row_rank(wkey);
    return br_wave_rank(wkey, G > 32);
  };

  int n_alive = qn;
  int head = 0;        // entries consumed from the front (they read BR_ENTRY_GONE); the list is [head, head + n_alive)
  bool stale = true;   // the LDS copy of the list is out of date (consumed entries aside)
  int pops = 0, guard = 0, wdrop = 0;

  auto list_to_lds = [&]() {
    if (stale) {
      br_list_store<E>(x, lst, lane);
      stale = false;
    }
    br_wave_sync();
  };

  float e2 = 0.0f, dscale = 0.0f;
  int ho = -1;
  if constexpr (BRH) {
    dscale = p.aD + p.beta * p.dsum;
    br_peak_bounds<HB>(p, br_uniform((int)(x[0] >> BR_IDX_BITS)), e2, ho);
  }

  // argmax_i F_g({i}) over the waiting, admissible requests (lowest position on ties) as a list entry; false when none
  // is admissible.  `none_below`: no waiting request is shorter than the margin.
  auto pick = [&](const int(&mg)[NH], int room, unsigned &key, bool &none_below) -> bool {
    const int room1 = min(room, BR_MAX_S_DEV) + 1;  // lengths below it are admissible
    int m = mg[0];
    bool two = true;
    if constexpr (BRH) {
#pragma unroll
      for (int h = 1; h < NH; ++h) m = min(m, mg[h]);
      if (ho < p.H) {
        int mo = INT32_MAX;
#pragma unroll
        for (int h = 0; h < NH; ++h) mo = h <= ho ? min(mo, mg[h]) : mo;
        two = mo == m;  // the smallest margin is one of those that end the rise
      }
    } else {
      if (G == 1) m = BR_MAX_S_DEV + 1;  // one worker is its own envelope: every score is zero, the first entry wins
    }
    if (!BRH || two) {
      const unsigned T = (unsigned)max(min(m, room1), 1) << BR_IDX_BITS;
      unsigned hi, lo;
      br_list_around<E>(x, T, hi, lo);
      none_below = lo == 0u;
      const int sh = (int)(hi >> BR_IDX_BITS), sl = (int)(lo >> BR_IDX_BITS);
      // each below zero where it speaks against the longer one: no such entry (0 or gone), too long; scored below the shorter one (equal: the lower position)
      int longer = min((int)hi - 1, room1 - 1 - sh);
      if constexpr (BRH) {
        const int F = br_ord(br_scoreh(p, mg, lane == 0 ? sh : sl));
        longer = (lo == 0u) | (__builtin_amdgcn_readlane(F, 0) >= __builtin_amdgcn_readlane(F, 1)) ? longer : -1;
      } else {
        longer = min(longer, sh - G * (sh - m) - (lo != 0u ? sl : -(1 << 30)));
      }
      const bool useh = longer >= 0;
      key = lo;
      if (useh) {  // the first of its length
        unsigned before;
        br_list_around<E>(x, (unsigned)(sh + 1) << BR_IDX_BITS, before, key);
      }
      return key != 0u;
    }
    if constexpr (BRH) {
      none_below = false;
      const unsigned Tr = (unsigned)max(room1, 1) << BR_IDX_BITS;
      if constexpr (E >= 16) {
        // Bracket first: the lanes' first entries are probes every E positions.  A probe before the best one that scores
        // below it by more than 2 e is beaten by it in exact arithmetic, by concavity so is everything before the
        // probe, and all of that computes strictly below what the best probe computes; likewise behind it.  What
        // lies strictly between the nearest such probes is scored: 64 positions at most, else all of the list.
        const bool live = x[0] != 0u && x[0] != BR_ENTRY_GONE;
        const int F1 = br_ord(br_scoreh(p, mg, live ? (int)(x[0] >> BR_IDX_BITS) : 0));
        const int km1 = br_wave_max(live && x[0] < Tr ? F1 : BR_KEY_NONE);
        if (km1 != BR_KEY_NONE) {
          const int ls = (int)__builtin_ctzll(br_ballot(live && x[0] < Tr && F1 == km1));
          const unsigned long long out = br_ballot(live && br_unord(F1) < br_unord(km1) - 2.0f * e2);
          const unsigned long long before = out & ((1ull << ls) - 1ull);
          const unsigned long long after = ls < 63 ? out >> (ls + 1) : 0ull;
          const int from = before != 0ull ? (63 - (int)__builtin_clzll(before)) * E + 1 : head;
          const int to = after != 0ull ? (ls + 1 + (int)__builtin_ctzll(after)) * E : head + n_alive;
          if (to - from <= BR_WAVE) {
            list_to_lds();
            const unsigned e = (unsigned)lst[br_list_at<E>(min(from + lane, NP - 1))];
            const int F2 = br_ord(br_scoreh(p, mg, (int)(e >> BR_IDX_BITS)));
            const bool ok = from + lane < to && e < Tr;
            const int km2 = br_wave_max(ok ? F2 : BR_KEY_NONE);
            key = (unsigned)__builtin_amdgcn_readlane((int)e, (int)__builtin_ctzll(br_ballot(ok && F2 == km2)));
            br_wave_sync();
            return true;
          }
        }
      }
      int bk = BR_KEY_NONE;
      unsigned bx = 0u;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int k = br_score_key<BRH>(p, mg, (int)(x[j] >> BR_IDX_BITS) & 0xffff);
        const bool ok = x[j] != 0u && x[j] < Tr;
        if (ok && k > bk) bk = k, bx = x[j];  // positions rise with j: the first best stays
      }
      const int km = br_wave_max(bk);
      if (km == BR_KEY_NONE) return false;
      key = (unsigned)__builtin_amdgcn_readlane((int)bx, (int)__builtin_ctzll(br_ballot(bk == km)));  // and with the lane
      return true;
    }
    return false;
  };

  // length of the shortest waiting request (looked up again once its entry has left)
  unsigned tail_key = 0u;
  bool tail_dirty = true;
  auto tail_len = [&]() -> int {
    if (tail_dirty) {
      unsigned below;
      br_list_around<E>(x, 1u << BR_IDX_BITS, tail_key, below);
      tail_dirty = false;
    }
    return (int)(tail_key >> BR_IDX_BITS);
  };

  // margins of worker g against the current envelope
  auto margins_of = [&](int g, int(&Lg)[NH], int(&mg)[NH]) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      Lg[h] = __builtin_amdgcn_readlane(Lh[h], g);
      mg[h] = max(Mh[h] - Lg[h], 0);
    }
  };

  // horizon-min margin of the worker each lane holds
  auto lane_minm = [&]() {
    int mn = INT32_MAX;
#pragma unroll
    for (int h = 0; h < NH; ++h) mn = min(mn, max(Mh[h] - Lh[h], 0));
    return mn;
  };

  // sticky binding of list entry `key` to worker g
  auto take = [&](unsigned key, int g, int slot) {
    bound[IDX_MASK - (int)(key & IDX_MASK)] = (g << 16) | slot;  // every lane stores the same word: no lane masking needed
    br_list_remove<E>(x, key);
    if constexpr (BRH && E >= 16) stale = true;  // (pick reads the copy)
  };
  // where the copy of the list and its shortest entry are looked at again
  auto bind = [&](unsigned key, int g, int slot) {
    take(key, g, slot);
    stale = true;
    tail_dirty |= key == tail_key;
  };

  // load update: the admitted length enters every horizon offset; envelope follows
  auto add_load = [&](int g, const int(&Lg)[NH], int delta, int k) {
    const int d = lane == g ? delta : 0;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      Lh[h] += d;
      Mh[h] = max(Mh[h], Lg[h] + delta);
    }
    const int dk = lane == g ? k : 0;
    cap -= dk;
    nn += dk;
    S_tot -= k;
    n_alive -= k;
  };

  auto drop_worker = [&](int g, int capg) {
    S_tot -= capg;
    cap = (lane == g) ? 0 : cap;
    ++wdrop;
  };

  // Admission of the K shortest waiting requests, in order of (length, arrival), to the workers of
  // rank r0 .. r0+K-1 (one each; ranks order the workers in question by load, then index), given that the first of them
  // has no shorter request than its margin waiting.  `smax` >= 0 limits K to the requests no longer than smax.
  //   BR-0: eq. (br0-Fscore) is G m - (G-1) s on the whole waiting set, so the worker takes the shortest one.  The envelope
  // becomes its new load; the next worker is at least as loaded, so its margin is at most that length and the same
  // holds for it, and so on down the ranks.
  //   BR-H: where the peak is the smallest margin (pick), the same request wins.  The k-th worker's margins are those
  // against the envelope that the admissions before it leave, a running maximum of L_j(h) + s_j over the ranks; K ends
  // before the first worker whose smallest margin exceeds the shortest request then left, or is not where the peak is.
  // Returns the number admitted, or 0 when the order cannot be read off the 64 shortest requests (a run of equal
  // lengths crossing that edge).  Loads, free slots, the envelope and the list are updated; counters are the caller's.
  auto tail_bulk = [&](int rank, int r0, int K, int smax) -> int {
    list_to_lds();
    const int end = head + n_alive;
    const int nA = min(n_alive, BR_WAVE);
    const bool valid = lane < nA;
    const int e = lst[br_list_at<E>(max(end - 1 - lane, 0))];  // the 64 shortest, shortest first
    const int st_ = e >> BR_IDX_BITS;
    const int sprev = __builtin_amdgcn_update_dpp(0, st_, 0x138, 0xF, 0xF, false);  // lane - 1
    const int snext = __builtin_amdgcn_update_dpp(0, st_, 0x130, 0xF, 0xF, false);  // lane + 1
    // requests of equal length are contiguous; within such a run the order of admission is by
    // arrival, the reverse of the order of the lanes
    const unsigned long long last = 1ull << (nA - 1), here = last | (last - 1ull);
    const unsigned long long sm = (br_ballot(sprev != st_) | 1ull) & here, em = (br_ballot(snext != st_) & here) | last;
    int T = BR_WAVE, ga = BR_WAVE;
    if (valid) {
      ga = 63 - (int)__builtin_clzll(sm & ((2ull << lane) - 1ull));
      const int gb = lane + (int)__builtin_ctzll(em >> lane);
      T = ga + gb - lane;
    }
    if (smax >= 0) K = min(K, (int)__builtin_popcountll(br_ballot(T < K && st_ <= smax)));  // lengths rise with T
    if (K <= 0) return 0;
    // a run cut by the edge of the 64 requests at hand has an unknown order here
    if (__builtin_expect(n_alive > BR_WAVE && __builtin_amdgcn_readlane(ga, BR_WAVE - 1) < K, 0)) return 0;
    if (T < K) slots[T] = e;
    br_wave_sync();
    if constexpr (BRH) {
      // lane k: the k-th of these workers (src: the lane that holds it) and the request it would take
      const int rel = rank - r0;
      const int src = br_ranks_to_lanes(rel >= 0 && rel < K, rel, lane);
      const int s_k = slots[min(lane, K - 1)] >> BR_IDX_BITS;
      int mn = INT32_MAX, mo = INT32_MAX;
      int Lk[NH], Mk[NH];
#pragma unroll
      for (int h = 0; h < NH; ++h) Lk[h] = __builtin_amdgcn_ds_bpermute(src << 2, Lh[h]);
      // envelope before the k-th admission: running maximum over the lanes below
#pragma unroll
      for (int h = 0; h < NH; ++h) Mk[h] = lane < K ? Lk[h] + s_k : BR_LOW;
      br_scan_maxs(Mk);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int m = max(max(Mh[h], br_dpp<0x138>(BR_LOW, Mk[h])) - Lk[h], 0);  // wave_shr:1
        mn = min(mn, m);
        mo = h <= ho ? min(mo, m) : mo;
      }
      const unsigned long long bad = br_ballot(lane < K && !(s_k >= mn && mo == mn));
      if (bad != 0ull) K = (int)__builtin_ctzll(bad);
      if (K < 2) return 0;
    }
    const bool cand = rank >= r0 && rank < r0 + K;
    const int mine = slots[cand ? rank - r0 : 0];
    const int s_k = cand ? mine >> BR_IDX_BITS : 0;
    if (cand) bound[IDX_MASK - (mine & IDX_MASK)] = (lane << 16) | nn;
#pragma unroll
    for (int h = 0; h < NH; ++h) Lh[h] += s_k;
    nn += cand ? 1 : 0;
    cap -= cand ? 1 : 0;
    // gone: the last K entries, except that of the run that holds the K-th one its first q (by arrival) go
    const int tK = (int)__builtin_ctzll(br_ballot(T == K - 1));
    const int gaK = __builtin_amdgcn_readlane(ga, tK);
    const int run0 = end - 1 - (tK + (K - 1) - gaK);  // list position of the run's first entry (its last lane)
    const int q = K - gaK;                            // entries of the run that go
    const int newend = end - K;
    const bool part = run0 < newend;                  // some of the run stays: it moves up over those that go
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int pos = lane * E + j;
      unsigned v = x[j];
      if (part) {
        const unsigned after = (unsigned)lst[br_list_at<E>(min(pos + q, NP - 1))];
        v = pos >= run0 ? after : v;
      }
      x[j] = pos < newend ? v : 0u;
    }
    stale |= part;
    if constexpr (BRH) {
#pragma unroll
      for (int h = 0; h < NH; ++h) Mh[h] = Lh[h];
      br_wave_maxs(Mh);
    } else {  // each of them became the envelope
      Mh[0] = __builtin_amdgcn_readlane(Lh[0], (int)__builtin_ctzll(br_ballot(rank == r0 + K - 1)));
    }
    S_tot -= K;
    n_alive -= K;
    tail_dirty = true;
    br_wave_sync();
    return K;
  };
  const bool tail_bulk_ok = G > 1 && p.W <= 0;  // argued without the watermark

  const int bound_it = qn + G + 1;  // every iteration admits a request or sets a worker aside

  // ---- Stage 1: greedy fill while free capacity is abundant
  for (int it = 0; it < bound_it; ++it) {
    if (!(S_tot > p.S_greedy && n_alive > 0)) break;
    const int capmax = cap_max();
    if (capmax <= 0) break;
    // the level: workers sharing the largest free-slot count, ranked by (load, index); each is
    // picked exactly once, in rank order, before any other worker can reach this free-slot count
    const unsigned long long members = br_ballot(cap == capmax);
    const bool member = __builtin_amdgcn_inverse_ballot_w64(members);
    const int wkey = member ? (int)(((unsigned)Lh[0] << 6) | (unsigned)lane) : INT32_MAX;
    int rank = rank_of(wkey);
    rank = member ? rank : BR_WAVE;  // (no member has rank 64)
    const int level = __builtin_popcountll(members);
    const int kmaxp = min(level, min(S_tot - p.S_greedy, n_alive));
    list_to_lds();
    const bool cand = rank < kmaxp;
    const int mine = lst[br_list_at<E>(head + (cand ? rank : 0))];
    const int s_k = mine >> BR_IDX_BITS;
    int lim = lane_minm();
    if (p.W > 0) lim = min(lim, p.W - Lh[0]);
    const int k0 = br_wave_min((cand && s_k > lim) ? rank : kmaxp);
    if (k0 > 0) {  // ranks 0..k0-1 are in the safe regime: k-th lightest worker takes k-th largest request
      const bool take = cand && rank < k0;
      if (take) bound[IDX_MASK - (mine & IDX_MASK)] = (lane << 16) | nn;
      const int d = take ? s_k : 0;
#pragma unroll
      for (int h = 0; h < NH; ++h) Lh[h] += d;
      nn += take ? 1 : 0;
      cap -= take ? 1 : 0;
      head += k0;
#pragma unroll
      for (int j = 0; j < E; ++j) x[j] = lane * E + j < head ? BR_ENTRY_GONE : x[j];
      S_tot -= k0;
      n_alive -= k0;
    }
    br_wave_sync();
    // the rest of the level in rank order
    for (int r = k0, end = kmaxp; LESS ? r < level && S_tot > p.S_greedy && n_alive > 0 : r < end;) {  // (every admission takes one off what ends the stage and off the level alike)
      const int g = (int)__builtin_ctzll(br_ballot(rank == r));
      int Lg[NH], mg[NH];
      margins_of(g, Lg, mg);
      const int room = p.W > 0 ? p.W - Lg[0] : INT32_MAX;
      unsigned key = 0u;
      bool none_below = false;
      if (__builtin_expect(!pick(mg, room, key, none_below), 0)) {
        drop_worker(g, capmax);
        ++r;
        end = r + min(level - r, min(S_tot - p.S_greedy, n_alive));
        continue;
      }
      if constexpr (LESS) end = r + min(level - r, min(S_tot - p.S_greedy, n_alive));
      if (none_below && tail_bulk_ok && end - r >= 3) {
        const int done = tail_bulk(rank, r, end - r, -1);
        if (done > 0) {
          r += done;
          continue;
        }
      }
      take(key, g, __builtin_amdgcn_readlane(nn, g));
      stale = true;
      add_load(g, Lg, (int)(key >> BR_IDX_BITS), 1);
      ++r;
    }
  }
  const int stage1 = qn - n_alive;
  tail_dirty = true;

  // ---- Stage 2: refined allocation over the workers that still have free slots
  if (head > 0 && n_alive > 0) {  // the window is read off the front of the list
    list_to_lds();
    br_list_load<E>(x, lst, lane, head, n_alive);
    head = 0;
    stale = true;
    br_wave_sync();
  }
  // Windows of up to four requests: 16 masks, one per lane of the wave's first row, which alone decides.  A loop of its own:
  // a pop is a chain of about 100 instructions on one wave, in which a taken branch costs 25 to 85 cycles (seven to twenty
  // instructions) and a scalar instruction that reads a vector result waits for four, so what is common goes straight
  // down.  In one loop with the window of eight a pop took 2400 to 3000 cycles alone on its SIMD, so 1250 to 1500 (1500 to 2000
  // through the guard).  Whole pass: 1531 clusters, G = 13, 10 admissions each 46.6 -> 42.7 us; 4096, G = 16, 6 admissions
  // 48.9 -> 47.1; one, G = 64, a queue of 2048 under a watermark 52.9 -> 49.1.  With the turns' shared state cut down, lane masks formed
  // by ballots alone and the score in one full-rate multiply-add (below) 1040 to 1330 and 1500 to 1800: 1531 clusters 33.6 -> 32.3, 4096
  // 41.5 -> 41.2, with 250 admissions each and 48 steps 104.8 -> 103.3.
  if (!BIGR && p.R_max <= 4) {
    // all ones at the length of window entry b on the lanes whose mask holds it (an entry beyond R_max never; one beyond
    // the list reads as zero, so its masks repeat lower ones, which win)
    unsigned len[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) len[b] = ((lane >> b) & 1) && b < p.R_max ? ~(unsigned)IDX_MASK : 0u;
    const int bits = __builtin_popcount(lane & 15);
    const int limit = p.W > 0 ? p.W : 1 << 29;           // of a load (none: beyond every load and length)
    // length of the shortest waiting request as last looked up: it only rises, so a worker that cannot take a request of
    // this length is out for good; one that turns out to be too full when its turn comes has it looked up again
    auto shortest_now = [&]() {
      tail_dirty = true;
      return tail_len();
    };
    int shortest = p.W > 0 ? shortest_now() : 0;
    // What the turns carry on is kept to what they read, since what differs between their ends is copied at each: free slots in
    // all, whether the LDS copy stands, which entry is the shortest are formed where they are asked for.
    // (every turn admits a request, sets a worker aside, or goes on to a lower free-slot count after such a turn)
    for (int turns = 2 * bound_it; min(min(n_alive, capmax_cur), turns) > 0; --turns) {
      // priority (free slots, horizon-min margin), lowest index on ties.  Workers for which even the shortest request is
      // too long are set aside when their turn comes; those whose turn comes before the first other one's go together
      // (nothing is admitted in between).
      const int prio = (int)(((unsigned)lane_minm() << 6) | (unsigned)(63 - lane));
      const unsigned long long members = br_ballot(cap == capmax_cur), takes = br_ballot(limit - Lh[0] >= shortest);
      int top = br_wave_max(__builtin_amdgcn_inverse_ballot_w64(members & takes) ? prio : -1);
      const unsigned long long outm = members & ~takes & br_ballot(prio > top);
      if (__builtin_expect((outm | (unsigned long long)(unsigned)(top >> 31)) != 0ull, 0)) {  // (or no member)
        const int n_out = __builtin_popcountll(outm);
        cap = __builtin_amdgcn_inverse_ballot_w64(outm) ? 0 : cap;
        wdrop += n_out;
        pops += n_out;
        guard += n_out;
        if (top < 0) {
          const unsigned long long left = br_ballot(cap == capmax_cur);
          if (left == 0ull) {  // the next lower free-slot count that has a member
            cap_max();
            continue;
          }
          top = 63 - (int)__builtin_ctzll(left);  // (loads beyond what the priorities order: the lowest index)
        }
      }
      const int g = 63 - (top & 63);
      ++pops;
      int Lg[NH], mg[NH];
      margins_of(g, Lg, mg);
      const int room = p.W > 0 ? p.W - Lg[0] : INT32_MAX;
      unsigned wv[4];  // the window: the first entries of the list
#pragma unroll
      for (int b = 0; b < 4; ++b) wv[b] = (unsigned)__builtin_amdgcn_readlane((int)x[b % E], b / E);
      const int delta =
          (int)(((wv[0] & len[0]) + (wv[1] & len[1]) + (wv[2] & len[2]) + (wv[3] & len[3])) >> BR_IDX_BITS);
      const bool ok = bits <= capmax_cur && delta <= room;
      unsigned mask;
      bool found;  // a subset scores above zero (the empty one scores zero: the guard's case like any other)
      if constexpr (!BRH) {
        int F;  // br_score0 (the compiler loses sight of the factors' 24 bits in the loop and multiplies in quarter rate)
        asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(F) : "v"(max(delta - mg[0], 0)), "v"(-G), "v"(delta));
        const int best = br_row0_max(ok ? F * 64 + (63 - lane) : INT32_MIN);
        found = best >= 64;
        mask = 63u - ((unsigned)best & 63u);
      } else {
        const int F = br_score_key<BRH>(p, mg, delta);
        const int best = br_row0_max(ok ? F : BR_KEY_NONE);
        found = best > 0;
        mask = (unsigned)__builtin_ctzll(br_ballot(ok && F == best) | (1ull << 63));
      }
      int slot = __builtin_amdgcn_readlane(nn, g);
      if (__builtin_expect(found, 1)) {
        const int sum = __builtin_amdgcn_readlane(delta, (int)mask);
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (__builtin_expect((mask >> b) & 1u, 1)) take(wv[b], g, slot++);  // slots follow the order of the window
        add_load(g, Lg, sum, __builtin_popcount(mask));
      } else {
        // starvation guard: the single best request anyway
        ++guard;
        unsigned key = 0u;
        bool none_below = false;
        const bool some = pick(mg, room, key, none_below);
        int done = 0;
        if constexpr (!BRH) {
          if (none_below && tail_bulk_ok) {
            // This worker takes the shortest waiting request through the guard and the envelope becomes
            // its new load.  The next pop goes to the next lightest worker that still has this many free
            // slots; its margin is at most the length just admitted.  While the lengths admitted stay
            // at or below (G-1)/G of the window's smallest entry, the window is untouched, that entry
            // still scores <= 0 for every such margin (so the guard fires again) and no waiting request
            // is below the margin: the pops of this free-slot count follow in one step.
            const int w = min(p.R_max, n_alive);
            int s_last = (int)(wv[0] >> BR_IDX_BITS);
#pragma unroll
            for (int b = 1; b < 4; ++b) s_last = b < w ? (int)(wv[b] >> BR_IDX_BITS) : s_last;
            const bool member = __builtin_amdgcn_inverse_ballot_w64(members);
            const int K = min((int)__builtin_popcountll(members), n_alive - w);
            if (K >= 3 && br_score0(G, mg[0], s_last) <= 0) {
              const int rank = rank_of(member ? (int)(((unsigned)Lh[0] << 6) | (unsigned)lane) : INT32_MAX);
              stale = true;
              done = tail_bulk(member ? rank : BR_WAVE, 0, K, (G - 1) * s_last / G);
              if (done > 0) pops += done - 1, guard += done - 1;
            }
          }
        }
        if (done == 0) {
          if (some) {
            take(key, g, slot);
            add_load(g, Lg, (int)(key >> BR_IDX_BITS), 1);
          } else {
            drop_worker(g, capmax_cur);
            shortest = shortest_now();
          }
        }
      }
    }
  } else {
  // lane-constant pieces of the subset enumeration: lane l of pass c stands for mask c*64 + l
  int lbit[6];
#pragma unroll
  for (int b = 0; b < 6; ++b) lbit[b] = (lane >> b) & 1;
  const int lpop = __builtin_popcount(lane);
  for (int it = 0; it < bound_it; ++it) {
    if (n_alive <= 0) break;
    const int capmax = cap_max();
    if (capmax <= 0) break;
    // priority (free slots, horizon-min margin), lowest index on ties
    int kc = (cap == capmax) ? (int)(((unsigned)lane_minm() << 6) | (unsigned)(63 - lane)) : -1;
    if (p.W > 0) {
      // workers for which even the shortest request is too long are set aside when their turn comes; those whose turn
      // comes before the first other one's go together (nothing is admitted in between)
      const int shortest = tail_len();  // (looked up by the whole wave)
      const bool none = kc >= 0 && p.W - Lh[0] < shortest;
      const int kfirst = br_wave_max(none ? -1 : kc);
      const bool out = none && kc > kfirst;
      const int n_out = __builtin_popcountll(br_ballot(out));
      if (n_out > 0) {
        cap = out ? 0 : cap;
        S_tot -= capmax * n_out;
        wdrop += n_out;
        pops += n_out;
        guard += n_out;
        if (kfirst < 0) continue;
        kc = out ? -1 : kc;
      }
    }
    const int g = 63 - (br_wave_max(kc) & 63);
    ++pops;
    int Lg[NH], mg[NH];
    margins_of(g, Lg, mg);
    const int room = p.W > 0 ? p.W - Lg[0] : INT32_MAX;

    // candidate window: the first min(R_max, |R_wait|) entries of the list
    const int w = min(p.R_max, n_alive);
    unsigned wv[8];
    int ws[8];
    int s_last = 0;  // smallest length in the window (its w-th entry)
    int wl = 0;      // BIGR: the window, entry l on lane l (BR-0 up to 16 requests: on lane l of each row)
    constexpr bool W16 = !BRH && !DP;
    if constexpr (BIGR) {
#pragma unroll
      for (int j = 0; j < E; ++j)
        if (lane * E + j < 32) win[lane * E + j] = (int)x[j];
      br_wave_sync();
      wl = win[lane & (W16 ? 15 : 31)];  // (read once: what a pop looks up of it comes from here)
      s_last = __builtin_amdgcn_readlane(wl, w - 1) >> BR_IDX_BITS;
    } else {
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        wv[b] = 0u, ws[b] = 0;
        if (b < 4 || w > 4) {
          wv[b] = (unsigned)__builtin_amdgcn_readlane((int)x[b % E], b / E);
          ws[b] = b < w ? (int)(wv[b] >> BR_IDX_BITS) : 0;
          s_last = b < w ? ws[b] : s_last;
        }
      }
    }
    // BR-0: every subset of the window sums to at least its smallest entry, and eq. (br0-Fscore)
    // falls beyond the margin; if that entry alone scores <= 0 (then it exceeds the margin), no
    // subset scores above 0 and the round goes to the starvation guard without the enumeration.
    // BR-H: eq. (brh-Fscore) is concave in Delta with F(0) = 0, so F(Delta) <= F(s) Delta / s for every
    // Delta >= s.  The scores are compared as computed in fp32: each of the at most H + 5 roundings of
    // one evaluation is relative 2^-24 on terms bounded by (alpha D + beta D) Delta, under 8e-7 of that in
    // all.  If the smallest entry's computed score is below -8e-6 (alpha D + beta D) s, its exact score
    // is below -7e-6 of it, every subset's exact score below the same fraction of its own Delta, and
    // every subset's computed score below zero: the guard is certain here too.
    bool guard_sure = false;
    if constexpr (!BRH) {
      guard_sure = br_score0(G, mg[0], s_last) <= 0;
    } else {
      guard_sure = br_scoreh(p, mg, s_last) <= -8e-6f * dscale * (float)s_last;
    }
    unsigned bestmask = 0u;
    int bestkey = BR_KEY_NONE;
    if (!guard_sure) {
      if constexpr (BIGR) {
        int kmax = min(min(capmax, p.R_max), w);
        {
          const int sum = br_rest_sums(wl, w, lane);
          float F, slack;
          if constexpr (BRH) {
            F = br_scoreh(p, mg, sum);
            slack = 3.2e-6f * dscale * (float)(kmax * (__builtin_amdgcn_readlane(wl, 0) >> BR_IDX_BITS));
          } else {  // (scores of sums below 2^20 times G <= 64 stay below 2^26: rounded to float they keep their order up
            F = (float)br_score0(G, mg[0], min(sum, 1 << 20)), slack = 32.0f;  // to units of 8, and the slack covers those)
          }
          kmax = br_useful_rest(sum, F, slack, w > 16 ? min(room, BR_DP_MAX_SUM) : room, kmax, w, lane);
        }
        if ((BRH || DP) && w > 16) {
          // windows of 17..32 requests: reachable sums instead of masks (br_subset_dp.h)
          br_subset_dp<BRH>(p, mg, win, w, kmax, room, lane, dprows,
                            p.dp + (size_t)inst * br_dp_cluster_words(min(p.B, p.R_max)), bestmask, bestkey,
                            shared ? svc : nullptr);
        } else {
          auto score4 = [&](const int(&delta)[4], int(&key)[4]) {
#pragma unroll
            for (int u = 0; u < 4; ++u) key[u] = br_score_key<BRH>(p, mg, delta[u]);
          };
          const bool listed = br_list_serves(w, kmax);
          // trips of 256 masks each (asked for only beyond the searches of few requests: a load from constant memory)
          auto trips = [&]() { return ((listed ? br_list_size(w, kmax) : 1 << w) + 255) >> 8; };
          if (!BRH && !DP && br_few_serves(w, kmax)) {
            br_subset_few(G, mg[0], wl, w, kmax, room, lane, hitab, bestkey, bestmask);
          } else if (kmax <= 3) {
            int mbest;
            br_wave_sync();
            br_small_search<BRH || DP>(W16 ? wl : win[lane & 15], win, w, kmax, room, lane, score4, bestkey, mbest);
            bestmask = bestkey == BR_KEY_NONE ? 0u : (unsigned)mbest;
          } else if (!BRH && trips() >= BR_HALVES_TRIPS) {
            br_subset_halves<!DP>(G, mg[0], wl, w, kmax, room, lane, hitab, bestkey, bestmask);
          } else {
            if (!listed) {
              const int nhi = w > 6 ? 1 << (w - 6) : 1;
              for (int c0 = 0; c0 < nhi; c0 += BR_WAVE) {
                const int c = c0 + lane;
                int sum = 0;
                for (int b = 6; b < w; ++b) sum += ((c >> (b - 6)) & 1) * (win[b] >> BR_IDX_BITS);
                if (c < nhi) hitab[c] = sum;
              }
            }
            int mbest;
            const bool shared_scan = shared && trips() >= BR_SHARE_TRIPS;
            if (shared_scan) {
              if (listed) br_list_tables(win, w, hitab, lane);
#pragma unroll
              for (int h = 0; h < NH; ++h) svc[1 + h] = mg[h];
              svc[2 + BR_HP] = room, svc[3 + BR_HP] = w, svc[4 + BR_HP] = kmax;
              svc[0] = 1;
              __syncthreads();
              br_bigr_scan<BRH>(p, mg, win, hitab, w, kmax, room, lane, 0, 4, false, bestkey, mbest);
            } else {
              br_wave_sync();
              br_bigr_scan<BRH>(p, mg, win, hitab, w, kmax, room, lane, 0, 1, true, bestkey, mbest);
            }
            if (shared_scan) {  // the best of the four shares: lowest mask among equal scores
              __syncthreads();
#pragma unroll
              for (int u = 1; u < 4; ++u) {
                const int ku = svc[16 + 2 * u], mu = svc[17 + 2 * u];
                if (ku > bestkey || (ku == bestkey && mu < mbest)) bestkey = ku, mbest = mu;
              }
            }
            bestmask = bestkey == BR_KEY_NONE ? 0u : (unsigned)mbest;
          }
        }
      } else {
        // exhaustive subset search, one subset mask per lane (ascending masks, strict improvement)
        const int kmax = min(capmax, p.R_max);
        const int nmask = 1 << w;
        int low = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) low += lbit[b] * ws[b];
        if (w > 4) low += lbit[4] * ws[4] + lbit[5] * ws[5];
        for (int c = 0; c * BR_WAVE < nmask; ++c) {
          const int delta = c == 0 ? low : low + (c & 1) * ws[6] + (c >> 1) * ws[7];
          const int mask = c * BR_WAVE + lane;
          const bool ok = mask != 0 && mask < nmask && lpop + __builtin_popcount(c) <= kmax && delta <= room;
          if constexpr (!BRH) {
            const int F = delta - (int)((unsigned)(max(delta - mg[0], 0) & 0x7ffff) * (unsigned)(G & 0x7f));
            const unsigned key = ok ? (((unsigned)(F + BIAS2) << 6) | (unsigned)(63 - lane)) : 0u;
            const unsigned km = w <= 4 ? (unsigned)br_row0_max((int)key) : br_wave_umax(key);  // (keys stay below 2^31)
            if (km != 0u) {
              const int Fm = (int)(km >> 6) - BIAS2;
              if (Fm > bestkey) {
                bestkey = Fm;
                bestmask = (unsigned)(c * BR_WAVE + (63 - (int)(km & 63u)));
              }
            }
          } else {
            int key = br_score_key<BRH>(p, mg, delta);
            key = ok ? key : BR_KEY_NONE;
            const int km = br_wave_max(key);
            if (km > bestkey) {
              bestkey = km;
              bestmask = (unsigned)(c * BR_WAVE + (int)__builtin_ctzll(br_ballot(key == km)));
            }
          }
        }
      }
    }

    if (bestmask == 0u || bestkey <= 0) {  // starvation guard: the single best request anyway
      unsigned key = 0u;
      bool none_below = false;
      const bool found = pick(mg, room, key, none_below);
      if constexpr (!BRH) {
        if (guard_sure && none_below && tail_bulk_ok) {
          // the pops of this free-slot count in one step, as argued for narrow windows above (one function for both: the batch
          // of 4096 clusters with 250 admissions each takes 114.7 us instead of 112.2)
          const bool member = cap == capmax;
          const int level = __builtin_popcountll(br_ballot(member));
          const int K = min(level, n_alive - w);
          if (K >= 3) {
            const int wkey = member ? (int)(((unsigned)Lh[0] << 6) | (unsigned)lane) : INT32_MAX;
            int rank = rank_of(wkey);
            rank = member ? rank : BR_WAVE;
            const int done = tail_bulk(rank, 0, K, (G - 1) * s_last / G);
            if (done > 0) {
              pops += done - 1;
              guard += done;
              continue;
            }
          }
        }
      }
      ++guard;
      if (!found) {
        drop_worker(g, capmax);
        continue;
      }
      bind(key, g, __builtin_amdgcn_readlane(nn, g));
      add_load(g, Lg, (int)(key >> BR_IDX_BITS), 1);
    } else {
      // slots follow the order of the window
      int slot = __builtin_amdgcn_readlane(nn, g);
      int delta = 0;
      if constexpr (BIGR) {
        for (unsigned m = bestmask; m != 0u; m &= m - 1u) {
          const unsigned key = (unsigned)__builtin_amdgcn_readlane(wl, __builtin_ctz(m));
          bind(key, g, slot++);
          delta += (int)(key >> BR_IDX_BITS);
        }
        br_wave_sync();  // the window has been read before a later pop rewrites it
      } else {
#pragma unroll
        for (int b = 0; b < 8; ++b)
          if ((bestmask >> b) & 1u) {
            bind(wv[b], g, slot++);
            delta += ws[b];
          }
      }
      add_load(g, Lg, delta, __builtin_popcount(bestmask));
    }
  }
  }
#pragma unroll
  for (int h = 0; h < NH; ++h) st.Lh[h] = Lh[h];
  st.nn = nn;
  rc.admitted = qn - n_alive;
  rc.stage1 = stage1;
  rc.pops = pops;
  rc.guard = guard;
  rc.wdrop = wdrop;
}

// One cluster's round on one wave.  EM: the queue holds up to EM * 64 entries; the list is made for 64 or 256 where no
// more are waiting.  COOP (EM = 32): the block has four waves; all of them sort a long waiting set together
// (br_sort_desc_block4) and share the epilogue and the decode step, wave 0 runs the round; the others compute the snapshot
// reductions meanwhile (one cluster, G = 64, H = 8, a queue of 2048: whole pass 49.1 -> 43.0 us against a launch of tiles and one that folds them).
// ADV: decode steps after the round, on its wave (0: none; BR-0: that many long lists at a time, see br_advance_lists_any).
// SCORES: the snapshot reductions (best_g / best_i where asked for) are taken on the way (br_score_wave.h).
// `split`: the cluster's BR_SPLIT_WORDS of LDS where the decode steps of the old list entries are applied apart (by
// another wave meanwhile, or by this one before the round), or null.
// `shared` (BIGR without COOP, one cluster per block of four waves): waves 1-3 serve the subset searches of wave 0
// (every fourth trip of a mask scan, every fourth run of 64 words of the rows of reachable sums) through the
// mailbox `svc` and two block barriers per search.
// HELPED: the block's other waves read the cluster's step-start state meanwhile (br_snapshot_helper); the block meets before
// this wave's epilogue changes it.
// SPLIT: the decode steps of the old entries are applied by another wave in every call, so the other epilogue is left out: with both
// in the kernel the words requested ahead of a queue of 257..512 went through 100 bytes of scratch memory per lane (2000 clusters,
// G = 16, queues of 500: whole pass 31.0 us, 26.1 without; one cluster 12.5 and 11.8).
template <int EM, int HB, int ADV, bool COOP = false, bool BIGR = false, bool SCORES = false, bool HELPED = false,
          bool SPLIT = false, bool DP = false>
__device__ __forceinline__ void br_assign_body(const BrParams &p, const BrArr &a, const BrOut &o, int *lds, int inst,
                                               int w = 0, int *split = nullptr,
                                               bool shared = false) {
  static_assert(!COOP || EM == 32, "the four-wave sort covers 4 x 512 keys");
  constexpr bool BRH = HB > 0;
  constexpr int NH = HB + 1;
  constexpr bool STEPS = BRH && EM <= 8 && !BIGR && !ADV;  // decode steps may have been applied ahead of the round
  static_assert(!STEPS || BR_DEAD_WORDS(EM) <= BR_LIST_WORDS(EM), "the epilogue's bit masks take the list's place");
  if (inst >= p.N) return;
  int *bound = lds;                              // [EM * 64] by arrival position: worker << 16 | slot, or -1
  int *lst = bound + EM * BR_WAVE;               // copy of the list
  int *slots = lst + BR_LIST_WORDS(EM);          // [64] requests of a bulk step in order of admission
  int *ahead = slots + BR_WAVE;                  // STEPS: [BR_AHEAD_WORDS] (br_ahead_store)
  int *win = ahead;                              // BIGR: [32] Stage-2 candidate window
  int *hitab = win + 32;                         // BIGR: [BR_SEARCH_WORDS] subset-sum tables
  int *svc = hitab + BR_SEARCH_WORDS;            // BIGR, shared: [32] mailbox
  int *dprows = svc + (shared ? 32 : 0);         // BIGR, R_max > 16: bit rows of the subset search
  // COOP: [BR_LIST_WORDS(32)] the sorted list as it was at the start
  int *lst2 = lds + BR_ROUND_WORDS(EM, HB, BIGR) + (BIGR && p.R_max > 16 ? BR_DP_LDS_WORDS : 0);

  const int lane = br_lane();
  if constexpr (BIGR && !COOP) {
    if (shared && w != 0) {  // one pass per scan; every wave of the block meets at both barriers, wave 0 ends the loop
      for (;;) {
        __syncthreads();
        const int cmd = svc[0];
        if (cmd == 0) break;
        if (cmd == 2) {  // this wave's words of the rows of reachable sums
          br_dp_build_helper(p, win, svc, dprows, p.dp + (size_t)inst * br_dp_cluster_words(min(p.B, p.R_max)), lane, w);
        } else {         // this wave's trips of a mask scan
          int mgq[NH];
#pragma unroll
          for (int h = 0; h < NH; ++h) mgq[h] = svc[1 + h];
          int km, mm;
          const int w_q = br_uniform(svc[3 + BR_HP]), k_q = br_uniform(svc[4 + BR_HP]), room_q = br_uniform(svc[2 + BR_HP]);
          br_bigr_scan<BRH>(p, mgq, win, hitab, w_q, k_q, room_q, lane, w, 4, false, km, mm);
          if (lane == 0) svc[16 + 2 * w] = km, svc[17 + 2 * w] = mm;
        }
        __syncthreads();
      }
      return;
    }
  }
  const int G = p.G;
  // two memory round trips for the cluster: these words, then the waiting set
  BrClusterIn<HB> in;
  br_cluster_load<HB, STEPS>(p, a, inst, lane, in);
  const int q0 = in.q0, cnt = in.cnt;
  const int qn = q0 + min(cnt, p.Q - q0);

  // first estimate of a newly admitted request when the library maintains c_hat (age 0)
  float c0 = 0.0f;
  if constexpr (BRH) {
    if (p.pred_mode == 2) c0 = *p.c0;
  }

  // (not where four waves share a SIMD anyway: 4096 clusters with decode steps 47.2 us without, 47.9 with)
  constexpr bool AHEAD = !COOP && !BRH && !ADV && EM <= 8;
  BrQueueWords<EM> words;
  if constexpr (AHEAD)
    br_queue_words<EM>(p.qs, p.qo, p.qid, a.s, a.o, a.id, (int64_t)inst * p.Q, (int64_t)inst * a.arr_cap, lane, 0, q0, qn, words);

  // ---- worker state, one worker per lane
  BrRoundState<HB> st;
  br_round_state<HB>(p, lane, in.n, in.L, st);
  const int nn_start = st.nn;
  if constexpr (BRH) {
    if (w == 0) {
      if (STEPS && p.adv_t > 0) ahead[lane] = in.lost, ahead[BR_WAVE + lane] = in.dL, ahead[2 * BR_WAVE + lane] = st.nn;  // (the margins replace it in memory)
      br_store_margins<HB>(p, inst, lane, st);
    }
  }

  BrRoundCounts rc = {};
  if (o.stats) {  // sum of loads in two 16-bit halves (each partial sum fits int32 for loads below 2^25)
    const int L0 = lane < G ? st.Lh[0] : 0;
    rc.I_before = (long long)G * st.Mh[0] - (((long long)br_wave_sum(L0 >> 16) << 16) + br_wave_sum(L0 & 0xffff));
  }

  // ---- waiting set: sorted list, made for the number that wait; then the two stages
  const bool run = st.S_tot > 0 && qn > 0;
  bool lead = true;  // this wave runs the round
  if constexpr (COOP) {
    lead = w == 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) bound[w * 512 + j * BR_WAVE + lane] = -1;
    if (run && qn > 256) {  // same for every wave of the block
      unsigned x8[8];
      br_keys_load<8>(p, a, inst, q0, qn, w * 512, lane, x8);
      br_sort_desc_block4(x8, lst, w, lane, qn);
      // (every wave is past its last read of the exchange buffer: the block meets inside the sort after that; up to 512 waiting nothing
      // is exchanged and each wave writes its own part only)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int at = br_list_at<32>(w * 512 + lane * 8 + j);
        lst[at] = (int)x8[j], lst2[at] = (int)x8[j];
      }
    }
    __syncthreads();
    // the snapshot reductions on the waves that have nothing to do until the epilogue (which starts with a block barrier)
    if (w != 0 && (o.best_g || o.best_i)) br_snapshot_coop<HB>(p, a, o, inst, lane, w - 1, q0, qn, run, lst2, st);
  } else {
#pragma unroll
    for (int j = 0; j < EM; ++j)
      if (j * BR_WAVE < qn) bound[j * BR_WAVE + lane] = -1;
  }
  if constexpr (SCORES) {
    if (!run) br_snapshot_none(p, o, inst, lane);
  }
  if (run && lead) {
    auto with = [&](auto e) {
      constexpr int E = decltype(e)::value;
      unsigned x[E];
      if constexpr (COOP && E >= 16) {
        br_list_load<E>(x, lst, lane, 0, qn);
      } else {
        br_list_build<E, HB, SCORES>(p, a, o, inst, lane, q0, qn, lst, st, x);
      }
      br_wave_sync();
      br_round<E, HB, BIGR, DP>(p, inst, lane, qn, x, bound, lst, slots, win, hitab, svc, dprows, shared, st, rc);
    };
    if (qn <= BR_WAVE)
      with(std::integral_constant<int, 1>{});
    else if (EM == 4 || qn <= 4 * BR_WAVE)
      with(std::integral_constant<int, 4>{});
    else if (COOP && qn <= 16 * BR_WAVE)
      with(std::integral_constant<int, COOP ? 16 : EM>{});
    else if constexpr (EM > 4)
      with(std::integral_constant<int, EM>{});
  }
  br_wave_sync();

  if constexpr (BIGR && !COOP) {
    if (shared) {
      svc[0] = 0;  // the round is over: the waves that served the scans leave
      __syncthreads();
    }
  }
  if constexpr (HELPED) __syncthreads();
  if constexpr (COOP) {
    int Lw = st.Lh[0];
    br_assign_epilogue_block4<BRH>(inst, lane, w, q0, qn, cnt, bound, slots, lst, Lw, st.nn, rc, c0, ADV > 0);
    if constexpr (ADV) {
      const int per = (G + 3) >> 2;
      br_advance_cluster<ADV>(inst, lane, Lw, st.nn, lds + w * BR_PLAIN_WORDS, min(w * per, G), min(w * per + per, G));
    }
  } else {
    bool done = false;
    if constexpr (SPLIT) {
      br_assign_epilogue_split<EM>(inst, lane, q0, qn, cnt, bound, st.Lh[0], st.nn, nn_start, rc, split, lst, &words);
      return;
    } else if constexpr (!BRH && !BIGR && EM <= 8) {
      if (split != nullptr) {
        br_assign_epilogue_split<EM>(inst, lane, q0, qn, cnt, bound, st.Lh[0], st.nn, nn_start, rc, split, lst, AHEAD ? &words : nullptr);
        done = true;
      }
    }
    if (!done) {
      if constexpr (STEPS)
        br_assign_epilogue_ahead<EM, HB>(inst, lane, q0, qn, cnt, bound, st.Lh[0], st.nn, rc, c0, ahead, lst);
      else
        br_assign_epilogue<EM, BRH>(inst, lane, q0, qn, cnt, bound, st.Lh[0], st.nn, rc, c0, AHEAD ? &words : nullptr);
      if constexpr (ADV && BRH)
        br_advance_cluster_rows(inst, lane, st.Lh[0], st.nn, bound);
      else if constexpr (ADV)
        br_advance_cluster<ADV>(inst, lane, st.Lh[0], st.nn, lds);
    }
  }
}

// every wave of the block owns one cluster and its own slice of LDS; waves never meet at a barrier
// The BR-H kernels need one or two registers more than let four waves share a SIMD
// (a batch of 4096 clusters is four waves per SIMD): they are asked to fit, and so is that for H <= 4 and queues of up to 256 (two
// registers too many for five).  H = 5..8, queues of up to 256, no reductions, 130 registers and three waves / 128 and four, whole pass, us: 4096 clusters, G = 16,
// overloaded, H = 8, one step 107.3 / 99.7, H = 6, 16 steps 183.8 / 174.4; 3500, G = 40 142.4 / 134.6.
// BIGR: candidate windows of 9..16 requests (R_max > 8); a separate instantiation so that the kernels for
// the deployed window sizes keep their registers and code size.
template <int E, int HB, int ADV, bool BIGR = false, bool DP = false>
// `share` (BIGR, queues of up to 1024; BR-0: reachable sums only): one cluster per block, its four waves share the searches
__global__ __launch_bounds__(256, (HB > 0 && E == 8 && !BIGR) ? 4 : (HB > 0 && E == 4 && !BIGR) ? (HB == 4 ? 5 : 4) : ADV == 4 ? 6 : 1) void br_k_assign(BrParams p, BrArr a, BrOut o, int share) {
  extern __shared__ int lds_all[];
  constexpr int WORDS = ADV ? BR_ROUND_ADV_WORDS(E) : BR_ROUND_WORDS(E, HB, BIGR);
  const int w = threadIdx.x >> 6;
  if constexpr (E == 32) {  // one cluster per block, four waves for the sort
    br_assign_body<E, HB, ADV, true, BIGR, false, false, false, DP>(p, a, o, lds_all, (int)blockIdx.x, w);
    return;
  }
  // (in the kernel for BR-0 windows of up to 16, which never shares, the second copy of the round cost scalar registers and four vector
  // ones, with queues of 257..512 the third wave per SIMD: 3000 clusters, window 16, queues of 512, whole pass 102 us, 79 without)
  if constexpr (BIGR && (HB > 0 || DP)) {
    if (share) {
      br_assign_body<E, HB, ADV, false, BIGR, false, false, false, DP>(p, a, o, lds_all, (int)blockIdx.x, w, nullptr, true);
      return;
    }
  }
  if constexpr (E != 32)
    br_assign_body<E, HB, ADV, false, BIGR, false, false, false, DP>(p, a, o, lds_all + w * WORDS, (int)(blockIdx.x * (blockDim.x >> 6)) + w);
}

// Small batches without decode steps in the launch: a block per cluster, its first wave runs the round, the others compute
// what was asked for beside it (the reductions, BR-0 also the matrix) meanwhile.  Two of them: one shares out the requests,
// one sorts.  1531 clusters, G = 13, queues of 307, matrix and reductions asked for, whole pass: 42.7 us with the reductions on the
// round's wave and the matrix as a launch before it, 36.5 / 35.6 / 39.1 us with 1 / 2 / 3 such waves.
#define BR_HELPERS 2
template <int E, int HB>
__global__ __launch_bounds__((1 + BR_HELPERS) * BR_WAVE) void br_k_route_helped(BrParams p, BrArr a, BrOut o, unsigned recip_g) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6, inst = (int)blockIdx.x;
  if (w == 0) {
    br_assign_body<E, HB, 0, false, false, false, true>(p, a, o, lds_all, inst);
  } else {
    br_snapshot_helper<E, HB>(p, a, o, inst, br_lane(), w - 1, BR_HELPERS, recip_g,
                              lds_all + BR_ROUND_WORDS(E, HB, false) + (w - 1) * (BR_LIST_WORDS(E) + 2 * BR_WAVE));
    __builtin_amdgcn_s_waitcnt(0);  // every read has returned
    __syncthreads();
  }
}

static inline unsigned br_recip(int G) { return (unsigned)((0x100000000ull + (unsigned)G - 1u) / (unsigned)G); }  // ceil(2^32 / G)

template <int E, int HB>
static void br_launch_helped_one(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const size_t lds = (BR_ROUND_WORDS(E, HB, false) + (size_t)BR_HELPERS * (BR_LIST_WORDS(E) + 2 * BR_WAVE)) * sizeof(int);
  hipLaunchKernelGGL((br_k_route_helped<E, HB>), dim3((unsigned)p.N), dim3(BR_WAVE * (1 + BR_HELPERS)), lds, st, p, a, o,
                     br_recip(p.G));
}

// Clusters of one wave each per block (one where the queues are long and so the LDS of a cluster is large).
static inline int br_clusters_per_block(int N, int E) { return E <= 8 ? br_waves_per_block(N) : 1; }

template <int E, int HB, bool BIGR = false>
static void br_launch_assign_one(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const bool dp = BIGR && p.R_max > 16;   // windows beyond 16 requests: one cluster per block, with LDS for the bit rows
  const int wpb = dp ? 1 : br_clusters_per_block(p.N, E);
  const bool adv = HB == 0 && !BIGR && p.adv_t > 0;
  const size_t lds = ((size_t)wpb * (adv ? BR_ROUND_ADV_WORDS(E) : BR_ROUND_WORDS(E, HB, BIGR)) + (dp ? BR_DP_LDS_WORDS : 0) +
                      (E == 32 ? BR_LIST_WORDS(32) : 0)) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(E == 32 ? 4 * BR_WAVE : BR_WAVE * wpb);
  // (decode steps ride along for BR-0 with windows of up to 8 requests only; elsewhere the caller launches the decode kernel)
  if constexpr (BIGR) {
    // windows beyond 8 requests on a batch that leaves room on the chip: a block of four waves per cluster, the searches
    // shared (BR-0 up to a window of 16 has none that is long enough).  Registers let two of these waves share a SIMD, so
    // up to 512 clusters are resident at once; beyond, what a search costs decides.  Whole pass, us, shared / one wave each
    // (G = 8, B = 48, 5 pops a round), queues of 256 | 1024:
    //   H = 4, window 12    512 clusters 42 / 42 | 58 / 60      768: 57 / 45 | 83 / 65      1024: 64 / 46 | 98 / 68
    //   H = 8, window 16    512 clusters 50 / 75 | 69 / 97      768: 68 / 83 | 96 / 105     1024: 75 / 102 | 113 / 111
    //   H = 0, window 24    512 clusters 229 / 438 | 193 / 510  768: 225 / 444 | 224 / 558  1024: 285 / 513 | 289 / 574
    // The lines: 768 / 512 / 256 clusters for BR-H with queues of up to 256 / 512 / 1024, 1024 / 768 / 512 for reachable sums.
    const long long room = 1024ll * max(1, (E == 4 ? 4 : E == 8 ? 3 : 2) - (HB > 0 ? 1 : 0));
    if ((HB > 0 || dp) && E <= 16 && (long long)p.N * 4 <= room) {
      const size_t lds1 = ((size_t)BR_ROUND_WORDS(E, HB, true) + 32 + (dp ? BR_DP_LDS_WORDS : 0)) * sizeof(int);
      if (HB == 0)  // (reachable sums)
        hipLaunchKernelGGL((br_k_assign<E, HB, 0, true, HB == 0>), dim3((unsigned)p.N), dim3(4 * BR_WAVE), lds1, st, p, a, o, 1);
      else
        hipLaunchKernelGGL((br_k_assign<E, HB, 0, true>), dim3((unsigned)p.N), dim3(4 * BR_WAVE), lds1, st, p, a, o, 1);
    } else if (HB == 0 && dp) {
      hipLaunchKernelGGL((br_k_assign<E, HB, 0, true, HB == 0>), grid, block, lds, st, p, a, o, 0);
    } else {
      hipLaunchKernelGGL((br_k_assign<E, HB, 0, true>), grid, block, lds, st, p, a, o, 0);
    }
  } else if constexpr (HB > 0) {
    hipLaunchKernelGGL((br_k_assign<E, HB, 0>), grid, block, lds, st, p, a, o, 0);
  } else {
    // (six waves per SIMD with four long lists at a time, five with eight, 80 and 94 registers: 6000 clusters, G = 16, B = 144, eight /
    // four, us: one step 75.8 / 70.9, 48 steps 142 / 129; 5120 clusters 58.7 / 60.4; two words per lane in scratch memory, three instructions)
    if (adv && E <= 8 && p.N > 5 * 1024 && p.N <= 6 * 1024)
      hipLaunchKernelGGL((br_k_assign<E, HB, E <= 8 ? 4 : 8>), grid, block, lds, st, p, a, o, 0);
    else if (adv)
      hipLaunchKernelGGL((br_k_assign<E, HB, 8>), grid, block, lds, st, p, a, o, 0);
    else
      hipLaunchKernelGGL((br_k_assign<E, HB, 0>), grid, block, lds, st, p, a, o, 0);
  }
}

template <int HB, bool BIGR = false>
static void br_launch_assign_sized(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    br_launch_assign_one<4, HB, BIGR>(p, a, o, st);
  else if (p.Q <= 512)
    br_launch_assign_one<8, HB, BIGR>(p, a, o, st);
  else if (p.Q <= 1024 && (BIGR || !br_block_serves(p, o.F != nullptr)))
    br_launch_assign_one<16, HB, BIGR>(p, a, o, st);
  else
    br_launch_assign_one<32, HB, BIGR>(p, a, o, st);
}
