// Two-stage assignment of one scheduling round for horizons beyond the offsets the register kernel
// carries (Appendix, Alg. BR-H; H up to 128, the deployed value of Sec. 6 is 80), one wavefront per
// cluster runs the round (others may serve its searches, below).
//
// The round is the loop of Alg. BR-H: Stage 1 gives the worker with the most free slots (then the
// lightest, then the lowest index) its best single request while free capacity exceeds S_greedy (taken a
// level of equal free-slot counts at a time where that is provably the same, see below); Stage 2 pops
// workers by (free slots, horizon-min margin), searches the subsets of the top-R_max window and falls
// back to the single best request when no subset scores above zero.
//
// What differs from the short-horizon kernel is where the per-offset state lives:
//   - the step-start projections L_g(k+h) stay in LDS, sL[h][g] (row stride G | 1 words: odd, so that both
//     "lane = worker" and "lane = offset" reads spread over the banks, and no wider than the cluster needs:
//     with few workers several clusters then share a CU's LDS) and are never rewritten: an
//     admission adds its length at every offset (constant-s approximation of Sec. 4.1), so worker g's
//     current projection is sL[h][g] + add_g with one register add_g per lane;
//   - the envelope M_h and the margins of the worker in hand are LDS arrays maintained with lanes
//     mapped to offsets (lane l also keeps the envelope at offsets l, l + 64, l + 128 and the projections of
//     the worker in hand in registers, so that the update after an admission needs no LDS read);
//   - a score walks the offsets in order with margins and discounts broadcast from LDS, four per load, and
//     skips the groups of offsets whose margins no value in question reaches (exact zeros);
//   - the single best request argmax_i F_g({i}): in queues of up to 256 first read off the requests around the peak of the
//     score (pick_quick); where rounding could reorder those, and in longer queues, found by bracketing (pick_single: the
//     score is concave in the length, the waiting set is sorted by length); only where more than 64 requests are left
//     between the brackets is the whole waiting set scored.  2048 clusters, G = 8, H = 80, overloaded, with the
//     register sort and margins kept while the envelope stands: whole pass 75.1 -> 71.2 us, one cluster 27.3 -> 26.0;
//   - with queues of up to 256 and several waves a cluster the block forms the projections itself, before the round
//     (br_long_projects): one cluster, G = 8, H = 80, whole pass 20.6 -> 18.8 us, 2048 clusters 69.4 -> 65.7;
//   - Stage 2 goes straight to the starvation guard when the window's smallest entry scores clearly below
//     zero (then every subset does).
// Waiting set, sticky binding and epilogue are those of the short-horizon
// kernel (br_sort.h, br_assign_common.h).
//
// With fewer clusters than the chip has room for waves (NW = 2 or 4 waves per cluster) the searches, which
// are most of a round at these horizons, are shared: wave 0 runs the round and posts a command in LDS (the
// margins are there already), every wave does its share between two block barriers: of the probes' offset
// groups in a bracketing search (the order of that sum is free), or of the sorted positions in a full scan
// (wave 0 takes the best of the partial results; the share of a later wave holds higher positions, so only a
// strictly better score wins).  The helper waves leave when wave 0 posts the end of the round.
#pragma once

#include "br_device.h"
#include "br_launch.h"
#include "br_project.h"
#include "br_sort.h"
#include "br_assign_common.h"
#include "br_subset_list.h"

#define BR_LSTRIDE(G) ((G) | 1)  // words between offsets in sL (odd; one spare "no worker" column when G is even)

// Best (score key, sorted position) among the alive, admissible requests of NB blocks of 64 sorted positions
// (block jb + j in sv[J0 + j], alive bit J0 + j), lowest position on equal scores.  The longest alive request of
// a block is its first alive one: offsets whose margin it does not reach add nothing for any request of the
// block and are skipped for that block.
template <int NS, int J0, int NB>
__device__ __forceinline__ void br_long_slice_best(const BrParams &p, const float *smg, const float *sd, int HS, int lane,
                                                   int qn, const int (&sv)[NS], unsigned alive, int jb, int room, int &bk,
                                                   int &bp) {
  constexpr int NV = NB >= 4 ? 4 : NB;
  bk = BR_KEY_NONE, bp = INT32_MAX;
#pragma unroll
  for (int c = 0; c < NB; c += NV) {
    if ((jb + c) * BR_WAVE < qn) {
      int top[NV], dv[NV];
      int any = 0;
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const unsigned long long bal = br_ballot((alive >> (J0 + c + u)) & 1u);
        const int first = __builtin_amdgcn_readlane(sv[J0 + c + u], bal != 0ull ? (int)__builtin_ctzll(bal) : 0);
        top[u] = bal != 0ull ? first : 0;
        dv[u] = sv[J0 + c + u];
        any |= top[u];
      }
      if (any == 0) continue;
      float Fv[NV];
      br_scoreh_long_sel<NV>(p.aD, p.beta, smg, sd, HS, lane, top, dv, Fv);
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const bool ok = ((alive >> (J0 + c + u)) & 1u) && dv[u] <= room;
        const int key = ok ? br_ord(Fv[u]) : BR_KEY_NONE;
        if (key > bk) {  // positions rise with the block within a lane: the first best stays
          bk = key;
          bp = (jb + c + u) * BR_WAVE + lane;
        }
      }
    }
  }
}

// LDS of a wave for the snapshot reductions: margins of a worker, the best request it has seen for every worker, then the best
// worker it has seen for each request of a tile that waves share
#define BR_LONG_PART_AT(HS) ((HS) + 4)
#define BR_LONG_BEST_AT(HS, G) (BR_LONG_PART_AT(HS) + ((3 * (G) + 3) & ~3))
#define BR_LONG_RED_WORDS(HS, G) (BR_LONG_BEST_AT(HS, G) + 2 * BR_WAVE)

// Pairs (tile of 64 requests, worker with a free slot) that the helper waves take alone, per wave.  More (slots free nearly
// everywhere): wave 0 takes a share before its round, since its first shared search would wait for the helpers anyway
// (2048 clusters, all slots free, 256 waiting: whole pass 533 us with the helpers alone, 517 so, 524 with a launch of their own).
#define BR_LONG_ALONE 16

// The snapshot reductions of a cluster (K2 + K3) on its nh helper waves while wave 0 runs the round: wave h takes every nh-th
// tile of 64 requests against every worker with a free slot, or, of fewer tiles, one with `share` - 1 other waves, every
// so many-th of those workers; a worker's step-start margins are on their way from memory while the one before it is scored.
// best_g is written here, for shared tiles when the round is over (br_long_shared_best); what is best for a worker among these
// requests (score, then the longer request, then the earlier arrival) goes to `red`, where wave 0 finds it then.
template <bool MANY>
__device__ __forceinline__ void br_long_reductions(const BrParams &p, const BrArr &a, const BrOut &o, int inst, int lane, int h,
                                                   int nh, int share, int q0, int qn, const float *sd, float *red) {
  const int G = p.G, H1 = p.H + 1, HS = BR_HS(p.H);
  const int64_t wrow = (int64_t)inst * G, qrow = (int64_t)inst * p.Q;
  int *part = (int *)red + BR_LONG_PART_AT(HS), *best = (int *)red + BR_LONG_BEST_AT(HS, G);
  const int n_raw = p.n[wrow + min(lane, G - 1)], L = p.L[wrow + min(lane, G - 1)];
  const int tiles = (qn + BR_WAVE - 1) / BR_WAVE;
  unsigned long long freem = br_ballot(lane < G && n_raw < p.B);
  int first = h, step = nh;  // tiles of this wave
  if (share > 1) {           // (at most one)
    const int r = br_rank_below(freem);
    step = tiles;
    if constexpr (MANY) {
      first = h / share;
      freem = br_ballot(((freem >> lane) & 1ull) && r % share == h - first * share);
    } else {
      first = tiles <= 1 ? 0 : h >> 1;
      freem = br_ballot(((freem >> lane) & 1ull) && (share == 3 ? r % 3 : r & (share - 1)) == (share == 2 ? h & 1 : h));
    }
  }
  int ik = BR_KEY_NONE, is = 0, ii = -1;  // lane g: of worker g
  int mh[3] = {0, 0, 0};
  auto fetch = [&](int g) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int e = u * BR_WAVE + lane;
      if (u * BR_WAVE < HS) mh[u] = p.mh[(wrow + g) * H1 + min(e, H1 - 1)];
    }
  };
  for (int t = first; t < tiles; t += step) {
    const int i = t * BR_WAVE + lane;
    int bk = BR_KEY_NONE, bg = -1;
    if (freem != 0ull) {
      unsigned x[1];
      br_keys_load<1>(p, a, inst, q0, qn, t * BR_WAVE, lane, x);
      fetch((int)__builtin_ctzll(freem));
      const int s[1] = {(int)(x[0] >> BR_IDX_BITS)};
      const int top[1] = {br_wave_max(s[0])};
      for (unsigned long long f = freem; f != 0ull;) {
        const int g = (int)__builtin_ctzll(f);
        f &= f - 1ull;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const int e = u * BR_WAVE + lane;
          if (e < HS) red[e] = e < H1 ? (float)mh[u] : 0.0f;
        }
        br_wave_sync();
        if (f != 0ull) fetch((int)__builtin_ctzll(f));
        float F[1];
        br_scoreh_long_sel<1>(p.aD, p.beta, red, sd, HS, lane, top, s, F);
        br_wave_sync();
        const int room = p.W > 0 ? p.W - __builtin_amdgcn_readlane(L, g) : INT32_MAX;
        const int key = x[0] != 0u && s[0] <= room ? br_ord(F[0]) : BR_KEY_NONE;
        if (key > bk) bk = key, bg = g;  // workers in ascending order: the first best stays
        const int km = br_wave_max(key);
        if (km != BR_KEY_NONE) {
          const int sb = br_wave_max(key == km ? s[0] : -1);
          const int ib = br_wave_min(key == km && s[0] == sb ? i : INT32_MAX);
          const bool better = lane == g && (km > ik || (km == ik && (sb > is || (sb == is && ib < ii))));
          ik = better ? km : ik, is = better ? sb : is, ii = better ? ib : ii;
        }
      }
    }
    if (share > 1)
      best[lane] = bk, best[BR_WAVE + lane] = bg;
    else if (o.best_g && i < p.Q)
      o.best_g[qrow + i] = bg;
  }
  if (o.best_g)
    for (int i = (tiles + h) * BR_WAVE + lane; i < p.Q; i += nh * BR_WAVE) o.best_g[qrow + i] = -1;
  if (lane < G) part[lane] = ik, part[G + lane] = is, part[2 * G + lane] = ii;
}

// Waves that share a tile: with fewer tiles than waves (nh), two workers with a free slot or more to each.
// 229 clusters, G = 22, H = 73, at most 44 waiting, half of the slots free, whole pass: 44.1 us with a launch of its own, 55.2
// with a tile to a wave, 35.1 so.
template <bool MANY>  // more than four waves
__device__ __forceinline__ int br_long_sharers(int nh, int qn, int free) {
  if constexpr (MANY) {
    const int tiles = (qn + BR_WAVE - 1) / BR_WAVE;
    return 2 * tiles > nh ? 1 : max(min(nh / max(tiles, 1), free >> 1), 1);
  }
  return free < 2 * nh ? 1 : qn <= BR_WAVE ? nh : nh == 4 && qn <= 2 * BR_WAVE ? 2 : 1;
}

// best_g of shared tiles from what their waves have left, in the areas from `reds` on: score, then the first worker
__device__ __forceinline__ void br_long_shared_best(int32_t *best_g, int Q, int inst, int lane, int qn, int share, const int *reds, int words) {
  for (int i = lane; i < ((qn + BR_WAVE - 1) & ~(BR_WAVE - 1)); i += BR_WAVE) {
    int bk = BR_KEY_NONE, bg = -1;
    for (int u = 0; u < share; ++u, reds += words) {
      const int k = reds[lane], g = reds[BR_WAVE + lane];
      const bool better = g >= 0 && (bg < 0 || k > bk || (k == bk && g < bg));
      bk = better ? k : bk, bg = better ? g : bg;
    }
    if (i < Q) best_g[(int64_t)inst * Q + i] = bg;
  }
}

#define BR_LONG_EXTRA_MAX_N 256
// XW: waves beyond those that serve the searches, for the reductions only (few clusters).
template <int E, int NW, int XW = 0>
// (queues of up to 256: four waves per SIMD are asked for, which is what br_long_waves counts on.  Beyond, the compiler reserves 20 bytes
// of scratch memory with four waves a cluster that no instruction touches; asking for two waves per SIMD takes them away and is slower:
// H = 80, G = 8, queues of 1024, 100 clusters 65.0 us, 63.7 so)
__global__ __launch_bounds__(64 * (NW + XW), E == 4 && XW == 0 ? 4 : 1) void br_k_assign_long(BrParams p, BrArr a, BrOut o) {
  constexpr int RW = NW - 1 + XW;  // waves that have the reductions while wave 0 runs the round
  static_assert(E % NW == 0, "every wave takes whole blocks of 64 sorted positions");
  constexpr int EW = E / NW;  // blocks of 64 sorted positions per wave in a shared search
  // four-offset groups of wave 0 when the probes of a bracketing search are shared: every NW-th, wave w takes the
  // same pattern shifted by w
  constexpr unsigned long long SHARE = NW == 1 ? ~0ull : NW == 2 ? 0x5555555555555555ull : 0x1111111111111111ull;
  extern __shared__ int lds[];
  constexpr int NP = E * BR_WAVE;
  constexpr int IDX_MASK = (1 << BR_IDX_BITS) - 1;
  const int inst = (int)blockIdx.x;
  if (inst >= p.N) return;
  const int H1 = p.H + 1, HS = BR_HS(p.H);
  constexpr bool PROJECTS = E == 4 && NW > 1;  // (br_long_projects)
  if constexpr (PROJECTS) {
    if (p.project) {
      br_project_long<NW + XW>(p, inst, (int)threadIdx.x, lds);
      if (p.pred_mode == 2 && threadIdx.x >= 64 * (NW + XW - 1)) lds[p.project] = __float_as_int(br_survival_start(p, br_lane()));
      __syncthreads();  // what it wrote is in place, and its LDS free
    }
  }
  int *skey = lds;                  // [NP] sorted keys (s << 11 | 2047 - arrival position)
  int *adm = lds + NP;              // [NP] by sorted position: worker << 16 | slot, or -1
  int *who = lds + 2 * NP;          // [NP] by arrival position: worker << 16 | slot, or -1 (filled after the round)
  int *win = lds + 3 * NP;          // [64] Stage-1 level: k-th alive request (s << 11 | sorted position);
                                    //      Stage 2: the candidate window, same packing (16-byte aligned)
  int *pm = win + BR_WAVE;          // [64] partial horizon-min margins (offsets split over the lanes)
  int *sM = pm + BR_WAVE;           // [HS] envelope M_h
  float *smg = (float *)(sM + HS);  // [HS] margins of the worker in hand, as floats
  float *sd = smg + HS;             // [HS] discounts, zero beyond H
  const int LS = BR_LSTRIDE(p.G);
  int *sL = sM + 3 * HS;            // [HS][LS] step-start projections (rows beyond H: "no worker")
  int *hitab = sL + ((HS * LS + 3) & ~3);  // R_max > 8: [1024] sums of window entries 6.. by upper mask bits
  int *mbox = hitab + (p.R_max > 8 ? 1024 : 0);  // NW > 1: [16] search mailbox: command, admissible length; results from word 4; [12] how the reductions were shared out
  int *salive = pm;                 // alive words of the lanes of wave 0 during a search (pm is idle then)

  const int lane = br_lane();
  const int G = p.G;
  const int q0 = br_uniform(min(max(p.qlen[inst], 0), p.Q));
  int cnt = a.count ? a.count[inst] : 0;
  cnt = br_uniform(min(max(cnt, 0), a.arr_cap));
  const int qn = q0 + min(cnt, p.Q - q0);
  const int64_t qrow = (int64_t)inst * p.Q, arow = (int64_t)inst * a.arr_cap;

  // the step-start projections, as contiguous memory: all waves of the block, four words per thread in flight
  {
    const int32_t *src = p.Lh + (int64_t)inst * G * H1;
    const int words = G * H1, nt = 64 * (NW + XW);
    const unsigned inv = 0xffffffffu / (unsigned)H1 + 1u;  // e / H1 by a multiply-high (e < 2^14)
    for (int e0 = (int)threadIdx.x; e0 < words; e0 += 4 * nt) {
      int v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = src[min(e0 + u * nt, words - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = min(e0 + u * nt, words - 1);
        const int g = (int)__umulhi((unsigned)e, inv);
        sL[(e - g * H1) * LS + g] = v[u];
      }
    }
    for (int h = (int)threadIdx.x; h < HS; h += nt) {  // a column beyond G and offsets beyond H read as "no worker"
      if (LS > G) sL[h * LS + G] = BR_LOW;
      if (h >= H1)
        for (int g = 0; g < G; ++g) sL[h * LS + g] = BR_LOW;
    }
  }
  if constexpr (NW > 1) {
    const int w = (int)(threadIdx.x >> 6);
    if (w != 0) {  // serves wave 0's searches: every wave of the block meets at both barriers of each, wave 0 ends the loop
      __syncthreads();  // the sorted keys and the discounts are in LDS
      int svh[EW];
#pragma unroll
      for (int j = 0; j < EW; ++j) svh[j] = skey[(min(w, NW - 1) * EW + j) * BR_WAVE + lane] >> BR_IDX_BITS;
      const int sprobe = skey[lane * E] >> BR_IDX_BITS;  // the probe of this lane in a bracketing search
      if (o.best_g || o.best_i) {
        const int free = (int)__builtin_popcountll(br_ballot(lane < G && p.n[(int64_t)inst * G + min(lane, G - 1)] < p.B));
        const bool all = ((qn + BR_WAVE - 1) / BR_WAVE) * free > BR_LONG_ALONE * RW;
        const int skip = all ? 0 : 1;
        const int share = br_long_sharers<(XW > 0)>(RW + 1 - skip, qn, free);
        br_long_reductions<(XW > 0)>(p, a, o, inst, lane, w - skip, RW + 1 - skip, share, q0, qn, sd,
                           (float *)(mbox + 16) + w * BR_LONG_RED_WORDS(HS, G));
        if (w == RW) mbox[12] = 2 * share + skip;  // (for this wave, when the round is over)
        __builtin_amdgcn_s_waitcnt(0);  // every read has returned before the block meets for the last time
      }
      for (;;) {
        __syncthreads();
        const int cmd = mbox[0];
        if (cmd == 0) break;
        if (XW > 0 && w >= NW) {  // (has no part in searches)
        } else if (cmd == 2) {  // this wave's share of the probes' penalty sums
          who[w * BR_WAVE + lane] = __float_as_int(br_long_penalty_part(smg, sd, HS, lane, mbox[2], sprobe, SHARE << w));
        } else {         // this wave's share of a full scan
          const int roomq = mbox[1];
          const unsigned al = (unsigned)salive[lane] >> (w * EW);
          int bk, bp;
          br_long_slice_best<EW, 0, EW>(p, smg, sd, HS, lane, qn, svh, al, w * EW, roomq, bk, bp);
          const int km = br_wave_max(bk);
          const int pmn = km == BR_KEY_NONE ? INT32_MAX : br_wave_min(bk == km ? bp : INT32_MAX);
          if (lane == 0) mbox[4 + 2 * w] = km, mbox[5 + 2 * w] = pmn;
        }
        __syncthreads();
      }
      int32_t *best_g = br_late_out().best_g;
      if (w == RW && best_g && br_uniform(mbox[12]) > 3)
        br_long_shared_best(best_g, p.Q, inst, lane, qn, br_uniform(mbox[12]) >> 1,
                            mbox + 16 + (br_uniform(mbox[12]) & 1) * BR_LONG_RED_WORDS(HS, G) + BR_LONG_BEST_AT(HS, G), BR_LONG_RED_WORDS(HS, G));
      return;
    }
  }

  float c0 = 0.0f;  // first estimate of a newly admitted request when the library maintains c_hat
  if (p.pred_mode == 2) c0 = PROJECTS && p.project ? __int_as_float(lds[p.project]) : *p.c0;

  // ---- worker state: lane g holds worker g
  const bool act = lane < G;
  const int64_t wrow = (int64_t)inst * G + lane;
  int nn = act ? min(max(p.n[wrow], 0), p.B) : p.B;
  int cap = p.B - nn;
  int Lcur = act ? p.Lh[wrow * H1] : BR_LOW;  // L_g(k) + what this round admits
  int add = 0;                                // tokens admitted to this lane's worker in this round
  // envelope: lane l also keeps the offsets l, l + 64, l + 128 in registers (the LDS copy serves the reads that
  // need other lanes' offsets); Lg: the same offsets of the step-start projection of the worker in hand
  int Mr[3] = {0, 0, 0}, Lg[3] = {0, 0, 0};
  float mr[3] = {0.0f, 0.0f, 0.0f}, dr[3] = {0.0f, 0.0f, 0.0f};  // margins of the worker in hand and discounts, likewise
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int h = u * BR_WAVE + lane;
    if (h < HS) {
      Mr[u] = h < H1 ? p.Mh[(int64_t)inst * H1 + h] : 0;
      sM[h] = Mr[u];
      dr[u] = p.dl[h];
      sd[h] = dr[u];
      smg[h] = 0.0f;
    }
  }
  int S_tot = br_wave_sum(cap);
  long long I_before = 0;
  if (o.stats) {
    const int L0 = act ? Lcur : 0;
    const long long sumL = ((long long)br_wave_sum(L0 >> 16) << 16) + br_wave_sum(L0 & 0xffff);
    I_before = (long long)G * br_wave_max(Lcur) - sumL;
  }

  // ---- waiting set, sorted in registers (largest prefill first, arrival order among equals)
  const bool run = S_tot > 0 && qn > 0;
  unsigned xk[E];
  int s_raw[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {  // one batch of unconditional loads (an entry beyond the set reads the first queue word)
    const int i = j * BR_WAVE + lane;
    const bool ina = i >= q0 && i < qn;
    const int32_t *src = ina ? a.s + (arow + (i - q0)) : p.qs + (qrow + (i < q0 ? i : 0));
    s_raw[j] = *src;
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int i = j * BR_WAVE + lane;
    unsigned key = 0;
    if (i < qn) {
      const int s = min(max(s_raw[j], 1), BR_MAX_S_DEV);
      key = ((unsigned)s << BR_IDX_BITS) | (unsigned)(IDX_MASK - i);
    }
    xk[j] = key;
    adm[i] = -1;
    who[i] = -1;
  }
  if (run) br_sort_across<E>(xk, skey, lane, qn);
  int sv[E];
  unsigned alive = 0;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int pos = j * BR_WAVE + lane;
    skey[pos] = (int)xk[j];
    sv[j] = (int)(xk[j] >> BR_IDX_BITS);
    if (pos < qn) alive |= 1u << j;
  }
  br_wave_sync();
  if constexpr (NW > 1) {
    __syncthreads();  // the helper waves read their share of the sorted keys
    if (o.best_g || o.best_i) {
      float *red = (float *)(mbox + 16);
      const int free = (int)__builtin_popcountll(br_ballot(cap > 0));
      if (((qn + BR_WAVE - 1) / BR_WAVE) * free > BR_LONG_ALONE * RW) {
        br_long_reductions<(XW > 0)>(p, a, o, inst, lane, 0, RW + 1, br_long_sharers<(XW > 0)>(RW + 1, qn, free), q0, qn, sd, red);
      } else if (lane < G) {
        int *part = (int *)red + BR_LONG_PART_AT(HS);
        part[lane] = BR_KEY_NONE, part[G + lane] = 0, part[2 * G + lane] = -1;
      }
    }
  }

  int n_alive = qn;
  int stage1 = 0, pops = 0, guard = 0, wdrop = 0, admitted = 0;

  // margins of worker g against the current envelope, into smg (lanes = offsets)
  auto margins_of = [&](int g) {
    const int ag = __builtin_amdgcn_readlane(add, g);
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int h = u * BR_WAVE + lane;
      if (h < H1) {
        Lg[u] = sL[h * LS + g];
        mr[u] = (float)max(Mr[u] - (Lg[u] + ag), 0);
        smg[h] = mr[u];
      }
    }
    br_wave_sync();
  };

  // horizon-min margin of the worker each lane holds.  With few workers the offsets are split over the lanes:
  // lane c * GP + g takes every C-th group of four offsets of worker g (GP = workers rounded up to a power of
  // two, C = 64 / GP), the partial minima meet in LDS.  Padded offsets: envelope 0 against "no worker".
  const int GP = G <= 8 ? 8 : G <= 16 ? 16 : G <= 32 ? 32 : 64;
  const int C = BR_WAVE / GP;
  // Formed again only after an admission that raised the envelope somewhere.
  bool grew = true;  // (on any lane)
  int mn_kept = 0;
  auto lane_minm = [&]() {
    if (br_ballot(grew) == 0ull) return max(mn_kept - add, 0);
    const int g = lane & (GP - 1), c = lane / GP;
    int mn = INT32_MAX;
    const int *row = sL + min(g, LS - 1);  // lanes that stand for no worker read the last column (their result is never used)
    for (int h = 4 * c; h < HS; h += 4 * C) {
      const int4 M4 = *reinterpret_cast<const int4 *>(sM + h);
      const int l0 = row[(h + 0) * LS], l1 = row[(h + 1) * LS];
      const int l2 = row[(h + 2) * LS], l3 = row[(h + 3) * LS];
      mn = min(mn, min(min(M4.x - l0, M4.y - l1), min(M4.z - l2, M4.w - l3)));
    }
    if (C > 1) {
      pm[lane] = mn;
      br_wave_sync();
      for (int cc = 0; cc < C; ++cc) mn = min(mn, pm[cc * GP + g]);
      br_wave_sync();
    }
    mn_kept = mn, grew = false;
    return max(mn - add, 0);  // min_h (M_h - sL_h) - add, clamped once: the same as clamping every offset
  };

  // Rounding of one evaluation of eq. (brh-Fscore) in fp32: at most H + 5 roundings, each relative 2^-24 on terms
  // bounded by (alpha D + beta D) Delta, so a computed score differs from the exact one by at most
  // err_unit * Delta (a quarter of slack on top covers the rounding of this bound itself).
  const float err_unit = 1.25f * (float)(p.H + 5) * 5.9604645e-8f * (p.aD + p.beta * p.dsum);

  // argmax_i F_g({i}) over alive, admissible requests against the margins in smg (lowest sorted
  // position on ties); false when no request is admissible.
  //
  // The exact score is concave in the request's length, and the waiting set is sorted by length: the search
  // brackets the maximum instead of scoring every request.  Probes: every E-th sorted position from the first
  // request in question on (up to 64 lanes), waiting or not, scored by the order-free evaluation (br_long_penalty_part, shared out by offset groups when
  // several waves serve the cluster); Fb is the best probe among the requests in question.  With e =
  // err_unit times the longest length (a bound on the distance of either evaluation from the exact score): a probe
  // that is longer than the best one and scores below Fb - 4 e has an exact score below the best probe's, by
  // concavity the exact score cannot rise again beyond it, and every position at or before it computes (in the
  // ordered evaluation) below what the best probe's request computes; likewise for a shorter probe and every
  // position at or after it.  What lies strictly between the nearest such probes on both sides of the best one
  // (at most 64 positions, else the full scan below takes over) is scored in the ordered evaluation, and the best
  // request in question there, lowest position on equal scores, is the argmax over the whole waiting set:
  // everything left out computes strictly below a score that was kept.
  int span_fa = -1, span_la = -1;
  bool span_dirty = true;
  auto pick_single = [&](int room, int &pos, int &swin) -> bool {
    int bk, bp, km;
    {
      // first and last sorted position of a request in question: kept from search to search while the alive set
      // loses nothing at either end and no watermark narrows the set
      if (span_dirty || p.W > 0) {
        span_fa = -1, span_la = -1;
#pragma unroll
        for (int j = 0; j < E; ++j) {
          if (j * BR_WAVE < qn) {
            const unsigned long long bal = br_ballot(((alive >> j) & 1u) && sv[j] <= room);
            if (bal != 0ull) {
              if (span_fa < 0) span_fa = j * BR_WAVE + (int)__builtin_ctzll(bal);
              span_la = j * BR_WAVE + 63 - (int)__builtin_clzll(bal);
            }
          }
        }
        span_dirty = false;
      }
      const int fa = span_fa, la = span_la;
      if (fa < 0) return false;
      salive[lane] = (int)alive;
      br_wave_sync();
      const int p1 = lane * E;  // probe position
      const int e1 = skey[p1];
      const int s1 = e1 >> BR_IDX_BITS;
      const bool in1 = p1 < qn && p1 >= fa;  // (a probe before the first request in question brackets nothing that one does not)
      const bool q1 = in1 && (((unsigned)salive[p1 & 63] >> (p1 >> 6)) & 1u) && s1 <= room;
      const int top1 = br_uniform(skey[fa] >> BR_IDX_BITS);  // the longest request in question
      float pen1;
      if constexpr (NW > 1) {  // the probes' penalty sums are shared out by offset groups (the order is free here)
        mbox[2] = top1;
        mbox[0] = 2;
        __syncthreads();
        pen1 = br_long_penalty_part(smg, sd, HS, lane, top1, s1, SHARE);
        __syncthreads();
#pragma unroll
        for (int u = 1; u < NW; ++u) pen1 = __fadd_rn(pen1, __int_as_float(who[u * BR_WAVE + lane]));
      } else {
        pen1 = br_long_penalty_part(smg, sd, HS, lane, top1, s1, ~0ull);
      }
      const float F1 = br_scoreh_long_from(p.aD, p.beta, s1, pen1);
      const int k1 = q1 ? br_ord(F1) : BR_KEY_NONE;
      const int km1 = br_wave_max(k1);
      if (km1 != BR_KEY_NONE) {
        const int ls = (int)__builtin_ctzll(br_ballot(k1 == km1));
        const float thr = br_unord(km1) - 4.0f * err_unit * (float)top1;
        const unsigned long long ex = br_ballot(in1 && F1 < thr);
        const unsigned long long before = ex & ((1ull << ls) - 1ull);
        const unsigned long long after = ls < 63 ? ex >> (ls + 1) : 0ull;
        const int lo = before != 0ull ? (63 - (int)__builtin_clzll(before)) * E + 1 : fa;
        const int hi = after != 0ull ? min((ls + 1 + (int)__builtin_ctzll(after)) * E - 1, la) : la;
        const int nc = hi - lo + 1;
        if (nc <= BR_WAVE) {
          const int p2 = min(lo + lane, NP - 1);
          const int e2 = skey[p2];
          const int s2[1] = {e2 >> BR_IDX_BITS};
          const bool q2 = lane < nc && (((unsigned)salive[p2 & 63] >> (p2 >> 6)) & 1u) && s2[0] <= room;
          const int top2[1] = {__builtin_amdgcn_readfirstlane(s2[0])};
          float F2[1];
          br_scoreh_long_sel<1>(p.aD, p.beta, smg, sd, HS, lane, top2, s2, F2);
          const int k2 = q2 ? br_ord(F2[0]) : BR_KEY_NONE;
          const int km2 = br_wave_max(k2);
          const int l2 = (int)__builtin_ctzll(br_ballot(k2 == km2));  // positions rise with the lane: lowest first
          pos = lo + l2;
          swin = __builtin_amdgcn_readlane(s2[0], l2);
          br_wave_sync();
          return true;
        }
      }
      br_wave_sync();
    }
    if constexpr (NW > 1) {
      mbox[1] = room;
      salive[lane] = (int)alive;
      mbox[0] = 1;
      __syncthreads();
      br_long_slice_best<E, 0, EW>(p, smg, sd, HS, lane, qn, sv, alive, 0, room, bk, bp);
      km = br_wave_max(bk);
      pos = km == BR_KEY_NONE ? INT32_MAX : br_wave_min(bk == km ? bp : INT32_MAX);
      __syncthreads();
#pragma unroll
      for (int u = 1; u < NW; ++u) {
        const int ku = mbox[4 + 2 * u], pu = mbox[5 + 2 * u];
        if (ku > km) km = ku, pos = pu;  // positions of wave u lie above those of the waves before it
      }
      if (km == BR_KEY_NONE) return false;
    } else {
      if (p.W > 0) {  // under the watermark the longest alive requests may all be out of the question
        int smax = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) smax = max(smax, (((alive >> j) & 1u) && sv[j] <= room) ? sv[j] : 0);
        if (br_wave_max(smax) == 0) return false;
      }
      br_long_slice_best<E, 0, E>(p, smg, sd, HS, lane, qn, sv, alive, 0, room, bk, bp);
      km = br_wave_max(bk);
      if (km == BR_KEY_NONE) return false;
      pos = br_wave_min(bk == km ? bp : INT32_MAX);
    }
    swin = br_uniform(skey[pos] >> BR_IDX_BITS);
    return true;
  };

  // The same decided from four requests where that is certain: 1 (pos, swin set), 0 (no request is admissible), -1 (not
  // certain: pick_single).  Eq. (brh-Fscore) rises with the length while beta sum_{h: m_h < s} d_h stays below alpha D and
  // falls beyond, so with b the first sorted position on the rising side the best request is the first one in question at
  // or behind b or the last one before it (the first of its length).  b is searched with the lanes mapped to offsets, three
  // probes a step.  Those two and the next ones of other lengths beyond them are scored the same way (at most 12
  // roundings): the best of the four stands if it leads by more than 4 err_unit times the longest of them, what the two
  // evaluations of two requests can differ by; by concavity everything farther out is lower still.
  auto pick_quick = [&](int room, int &pos, int &swin) -> int {
    int b = 0;
#pragma unroll
    for (int step = 64; step > 0; step >>= 2) {  // (queues of up to 256)
      int e[3];
      float w[3];  // sum of the discounts whose margin the probe exceeds
#pragma unroll
      for (int k = 0; k < 3; ++k) e[k] = skey[min(b + (k + 1) * step, NP) - 1];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float fs = (float)(e[k] >> BR_IDX_BITS);
        w[k] = (mr[0] < fs ? dr[0] : 0.0f) + (mr[1] < fs ? dr[1] : 0.0f) + (mr[2] < fs ? dr[2] : 0.0f);
      }
      br_wave_fsums(w);
      int up = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) up += ((b + (k + 1) * step <= qn) & (p.beta * w[k] > p.aD)) ? step : 0;
      b += up;
    }
    b = br_uniform(b);
    // the requests in question as bits; neighbours are found on the scalar side
    unsigned long long qm[E];
#pragma unroll
    for (int j = 0; j < E; ++j) qm[j] = br_ballot(((alive >> j) & 1u) && sv[j] <= room);
    auto from_on = [&](int at) -> int {  // first one at or behind `at` / last one before it, or -1
      int r = -1;
#pragma unroll
      for (int j = E - 1; j >= 0; --j) {
        const int d = at - j * BR_WAVE;
        const unsigned long long m = d >= BR_WAVE ? 0ull : d > 0 ? qm[j] & (~0ull << d) : qm[j];
        r = m != 0ull ? j * BR_WAVE + (int)__builtin_ctzll(m) : r;
      }
      return r;
    };
    auto before = [&](int at) -> int {
      int r = -1;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int d = at - j * BR_WAVE;
        const unsigned long long m = d <= 0 ? 0ull : d < BR_WAVE ? qm[j] & ~(~0ull << d) : qm[j];
        r = m != 0ull ? j * BR_WAVE + 63 - (int)__builtin_clzll(m) : r;
      }
      return r;
    };
    auto length = [&](int at) -> int { return at >= 0 ? br_uniform(skey[at] >> BR_IDX_BITS) : 0; };
    const int lo = from_on(b);
    int hi = before(b);
    if (lo < 0 && hi < 0) return 0;
    const int s_lo = length(lo), s_hi = length(hi);
    int lo2 = -1, hi2 = -1;  // the next ones of other lengths; hi becomes the first of its length
    {
      int h1 = -1;
#pragma unroll
      for (int j = E - 1; j >= 0; --j) {
        const unsigned long long ml = qm[j] & br_ballot(sv[j] < s_lo), mh = qm[j] & br_ballot(sv[j] > s_hi);
        const unsigned long long me = qm[j] & br_ballot(sv[j] == s_hi);
        lo2 = ml != 0ull ? j * BR_WAVE + (int)__builtin_ctzll(ml) : lo2;
        hi2 = mh != 0ull && hi2 < 0 ? j * BR_WAVE + 63 - (int)__builtin_clzll(mh) : hi2;
        h1 = me != 0ull ? j * BR_WAVE + (int)__builtin_ctzll(me) : h1;
      }
      hi2 = hi >= 0 ? hi2 : -1;
      hi = hi >= 0 ? h1 : -1;
    }
    const int s_lo2 = length(lo2), s_hi2 = length(hi2);
    const int s[4] = {s_hi, s_lo, s_hi2, s_lo2};
    float F[4], pen[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      pen[v] = 0.0f;
#pragma unroll
      for (int u = 0; u < 3; ++u) pen[v] = __fmaf_rn(dr[u], fmaxf(__fsub_rn((float)s[v], mr[u]), 0.0f), pen[v]);
    }
    br_wave_fsums(pen);
#pragma unroll
    for (int v = 0; v < 4; ++v) F[v] = s[v] > 0 ? br_scoreh_long_from(p.aD, p.beta, s[v], pen[v]) : -INFINITY;
    const float e4 = 4.0f * err_unit * (float)max(max(s[0], s[1]), max(s[2], s[3]));
    const bool useh = br_ballot(F[0] > F[1]) != 0ull;
    const float lead = fmaxf(F[0], F[1]), other = fmaxf(fminf(F[0], F[1]), fmaxf(F[2], F[3]));
    if (br_ballot(lead - other > e4) != 0ull) {
      swin = useh ? s_hi : s_lo;
      pos = useh ? hi : lo;
      return 1;
    }
    return -1;
  };
  // Queues of up to 256 only (300 clusters, G = 16, queues of 500 in bursts, always bracketed / so: 279 / 352 us), and by what the
  // picks of the round have shown so far.
  // Starvation guard: while it decides at least two picks in three; among many waiting requests of nearly the same length the
  // leads are within the bounds pick after pick.  Whole pass, us, always bracketed / so, G = 8, H = 80, 2048 clusters,
  // overloaded, a decode step per call 78 / 67, 16 of them 208 / 191, 48: 424 / 400, 100: 748 / 705; a token watermark 82 / 84;
  // 128 admissions from a full queue 517 / 526 (a bracketing search skips the offsets that no request reaches, most of them there).
  int credit = 3;
  auto pick = [&](int room, int &pos, int &swin) -> bool {
    if constexpr (E == 4) {
      if (credit > 0) {
        const int r = pick_quick(room, pos, swin);
        if (r >= 0) {
          credit = min(credit + 1, 4);
          return r != 0;
        }
        credit -= 2;
      }
    }
    return pick_single(room, pos, swin);
  };

  // Stage 1, four waves a cluster (two: 2048 clusters in bursts of 200 arrivals 784 us bracketed, 800 so): many picks, at first with
  // wide margins, where bracketing skips most offsets and costs less than the quick pick's fixed work.  So a pick that reaches
  // the margins of fewer than eight offsets counts against it, and once out of credit it is tried again at every twelfth pick.
  // Whole pass, us, always bracketed / always tried / so: 8 clusters, G = 13, H = 56, 116 admissions (5 offsets a pick) 274 / 296 / 282;
  // the same with estimates (17 offsets) 372 / 351 / 363; G = 8, H = 80, one cluster in bursts of 60 169 / 152 / 155, 1000 in bursts of 200
  // (51 offsets) 695 / 656 / 556.
  int credit1 = 3, passed = 0;
  auto pick1 = [&](int room, int &pos, int &swin) -> bool {
    if constexpr (E == 4 && NW == 4) {
      if (credit1 > 0 || ++passed == 12) {
        passed = 0;
        const int r = pick_quick(room, pos, swin);
        if (r == 0) return false;
        if (r > 0) {
          int reach = 0;
#pragma unroll
          for (int u = 0; u < 3; ++u) reach += __builtin_popcountll(br_ballot(u * BR_WAVE + lane < H1 && mr[u] < (float)swin));
          credit1 = reach >= 8 ? min(credit1 + 1, 4) : max(credit1 - 1, 0);
          return true;
        }
        credit1 = max(credit1 - 2, 0);
      }
    }
    return pick_single(room, pos, swin);
  };

  // sticky binding of the request at sorted position pos to worker g
  auto bind = [&](int pos, int g, int slot) {
    adm[pos] = (g << 16) | slot;  // every lane stores the same word
    const int jw = pos >> 6, lw = pos & 63;
    alive = (lane == lw) ? (alive & ~(1u << jw)) : alive;
    span_dirty |= pos == span_fa || pos == span_la;
  };

  // load update: the admitted length enters every horizon offset of worker g; the envelope follows.  Worker g is
  // the one whose margins were formed last (margins_of(g)): its projections are still in Lg.
  auto add_load = [&](int g, int delta, int k) {
    add += (lane == g) ? delta : 0;
    Lcur += (lane == g) ? delta : 0;
    const int ag = __builtin_amdgcn_readlane(add, g);
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int h = u * BR_WAVE + lane;
      if (h < H1) {
        grew |= Lg[u] + ag > Mr[u];
        Mr[u] = max(Mr[u], Lg[u] + ag);
        sM[h] = Mr[u];
      }
    }
    br_wave_sync();
    cap -= (lane == g) ? k : 0;
    nn += (lane == g) ? k : 0;
    S_tot -= k;
    n_alive -= k;
    admitted += k;
  };

  auto drop_worker = [&](int g, int capg) {
    S_tot -= capg;
    cap = (lane == g) ? 0 : cap;
    ++wdrop;
  };

  if (run) {
    const int bound = qn + G + 1;  // every iteration admits a request or sets a worker aside

    // ---- Stage 1: greedy fill while free capacity is abundant.  Taken a level at a time: the workers that
    // share the largest free-slot count are picked once each in order of (load, index) before any other
    // worker can reach that count.  While the largest waiting request fits the next worker's horizon-min
    // margin (and the watermark), every penalty term of eq. (brh-Fscore) is zero for it, its score alpha D s
    // is the largest one, and the envelope does not move: the k-th lightest worker of the level takes the
    // k-th largest waiting request, all in one step.  The rest of the level goes one worker at a time.
    for (int it = 0; it < bound; ++it) {
      if (!(S_tot > p.S_greedy && n_alive > 0)) break;
      const int capmax = br_wave_max(cap);
      if (capmax <= 0) break;
      const bool member = cap == capmax;
      const int wkey = member ? (int)(((unsigned)Lcur << 6) | (unsigned)lane) : INT32_MAX;
      int rank = 0;
      for (int g0 = 0; g0 < G; g0 += 4) {  // lanes beyond G hold INT32_MAX and never count
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += (__builtin_amdgcn_readlane(wkey, g0 + u) < wkey) ? 1 : 0;
      }
      const int level = __builtin_popcountll(br_ballot(member));
      const int kmaxp = min(level, min(S_tot - p.S_greedy, n_alive));
      {  // the first kmaxp alive requests, by rank, through LDS
        int base = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
          if (base < kmaxp && j * BR_WAVE < qn) {
            const bool al = (alive >> j) & 1u;
            const unsigned long long bal = br_ballot(al);
            const int ar = base + br_rank_below(bal);
            if (al && ar < kmaxp) win[ar] = (sv[j] << BR_IDX_BITS) | (j * BR_WAVE + lane);
            base += __builtin_popcountll(bal);
          }
        }
      }
      br_wave_sync();
      const bool cand = member && rank < kmaxp;
      const int mine = cand ? win[rank] : 0;
      const int s_k = mine >> BR_IDX_BITS, pos_k = mine & IDX_MASK;
      int lim = lane_minm();
      if (p.W > 0) lim = min(lim, p.W - Lcur);
      const int k0 = br_wave_min((cand && s_k > lim) ? rank : kmaxp);
      if (k0 > 0) {
        const bool take = cand && rank < k0;
        if (take) adm[pos_k] = (lane << 16) | nn;
        add += take ? s_k : 0;
        Lcur += take ? s_k : 0;
        nn += take ? 1 : 0;
        cap -= take ? 1 : 0;
        const int pstar = br_uniform(win[k0 - 1] & IDX_MASK);  // last position taken; everything alive before it went too
        const int jf = pstar >> 6, lf = pstar & 63;
        const unsigned clear = ((1u << jf) - 1u) | ((lane <= lf) ? (1u << jf) : 0u);
        alive &= ~clear;
        span_dirty = true;
        S_tot -= k0;
        n_alive -= k0;
        admitted += k0;
        stage1 += k0;
      }
      br_wave_sync();
      for (int r = k0; r < level; ++r) {
        if (!(S_tot > p.S_greedy && n_alive > 0)) break;
        const int g = (int)__builtin_ctzll(br_ballot(member && rank == r));
        margins_of(g);
        const int room = p.W > 0 ? p.W - __builtin_amdgcn_readlane(Lcur, g) : INT32_MAX;
        int pos = 0, swin = 0;
        if (!pick1(room, pos, swin)) {
          drop_worker(g, capmax);
          continue;
        }
        bind(pos, g, __builtin_amdgcn_readlane(nn, g));
        add_load(g, swin, 1);
        ++stage1;
      }
    }

    // ---- Stage 2: refined allocation over the workers that still have free slots
    int lbit[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) lbit[b] = (lane >> b) & 1;
    const int lpop = __builtin_popcount(lane);
    for (int it = 0; it < bound; ++it) {
      if (n_alive <= 0) break;
      const int capmax = br_wave_max(cap);
      if (capmax <= 0) break;
      // priority (free slots, horizon-min margin), lowest index on ties
      const bool member = cap == capmax;
      const int mine_m = lane_minm();
      const int mm = br_wave_max(member ? mine_m : -1);
      const int g = (int)__builtin_ctzll(br_ballot(member && mine_m == mm));
      ++pops;
      margins_of(g);
      const int room = p.W > 0 ? p.W - __builtin_amdgcn_readlane(Lcur, g) : INT32_MAX;

      // candidate window: the first min(R_max, |R_wait|) alive requests in sorted order
      const int w = min(p.R_max, n_alive);
      {
        int base = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
          if (base < w && j * BR_WAVE < qn) {
            const bool al = (alive >> j) & 1u;
            const unsigned long long bal = br_ballot(al);
            const int ar = base + br_rank_below(bal);
            if (al && ar < w) win[ar] = (sv[j] << BR_IDX_BITS) | (j * BR_WAVE + lane);
            base += __builtin_popcountll(bal);
          }
        }
      }
      br_wave_sync();
      const int kmax = min(capmax, p.R_max);
      const int nmask = 1 << w;
      int bestmask = 0, bestkey = BR_KEY_NONE;
      int wv[8], ws[8];
      // Is the pop certain to end in the starvation guard?  eq. (brh-Fscore) is concave with F(0) = 0, so F(Delta) <=
      // F(s) Delta / s for every Delta >= s = the window's smallest entry.  If F(s), summed across the lanes in any order
      // (at most 12 roundings), is at or below -3 e(s), its exact value is at or below -2 e(s), every subset of the
      // window (all of them sum to at least s) has an exact score at or below -2 e(Delta) and computes below zero.
      // One value with the offsets on the lanes: 300 cycles, where the probes of a search that would decide it too take
      // 2000 to 6000.
      bool guard_sure;
      {
        const int s_last = br_uniform(win[w - 1] >> BR_IDX_BITS);
        const float fs = (float)s_last;
        float pen = 0.0f;
#pragma unroll
        for (int u = 0; u < 3; ++u) pen = __fmaf_rn(dr[u], fmaxf(__fsub_rn(fs, mr[u]), 0.0f), pen);  // (no discount beyond H)
        float pens[1] = {pen};
        br_wave_fsums(pens);
        pen = pens[0];
        guard_sure = br_ballot(br_scoreh_long_from(p.aD, p.beta, s_last, pen) <= -3.0f * err_unit * fs) != 0ull;
      }
      if (guard_sure) {
        br_wave_sync();  // the window has been read before a later pop rewrites it
      } else if (p.R_max > 8) {
        // Windows of up to 16 requests.  With at most half of the window per subset the admissible masks are taken
        // from a list (br_subset_list.h).  Otherwise lane l keeps the lower six mask bits, the upper bits run as passes
        // over a table of their partial sums (built here, 64 entries per step), four passes per trip; trips
        // whose upper bits alone exceed the cardinality limit are skipped; a lane sees its masks in ascending
        // order and keeps the first best.  Across lanes the lowest mask of the best score wins.
#pragma unroll
        for (int b = 0; b < 8; ++b) wv[b] = 0, ws[b] = 0;
        int top = 0;  // the largest sum any admissible subset can have (bound)
        for (int b = 0; b < min(kmax, w); ++b) top += win[b] >> BR_IDX_BITS;
        top = min(top, room);
        unsigned long long act[3];
        br_long_active(smg, HS, lane, top, act);
        int kw = min(kmax, w);
        {
          const int sums[1] = {br_min_sums(win, w, lane)};
          float F[1];
          br_scoreh_long_act<1>(p.aD, p.beta, smg, sd, act, sums, F);
          kw = br_useful_count(sums[0], F[0], 4.0f * err_unit * (float)top, room, kw, lane);
        }
        const bool listed = br_list_serves(w, kw);
        const int nhi = w > 6 ? 1 << (w - 6) : 1;
        if (!listed) {
          for (int c0 = 0; c0 < nhi; c0 += BR_WAVE) {
            const int c = c0 + lane;
            int sum = 0;
            for (int b = 6; b < w; ++b) sum += ((c >> (b - 6)) & 1) * (win[b] >> BR_IDX_BITS);
            if (c < nhi) hitab[c] = sum;
          }
        }
        int base = 0;
        for (int b = 0; b < min(w, 6); ++b) base += ((lane >> b) & 1) * (win[b] >> BR_IDX_BITS);
        br_wave_sync();
        auto score4 = [&](const int(&delta)[4], int(&key)[4]) {  // (sums beyond `top` score as anything: never admissible)
          float Fv[4];
          br_scoreh_long_act<4>(p.aD, p.beta, smg, sd, act, delta, Fv);
#pragma unroll
          for (int u = 0; u < 4; ++u) key[u] = br_ord(Fv[u]);
        };
        if (listed) {
          br_list_walk(win, hitab, w, kw, room, lane, 0, 1, true, score4, bestkey, bestmask);
          if (bestkey == BR_KEY_NONE) bestmask = 0;
        } else {
          int bk = BR_KEY_NONE, bm = INT32_MAX;
          const int klim = kw - lpop;
          const bool lane_ok = lane < nmask;
          for (int c0 = 0; c0 < nhi; c0 += 4) {
            if (__builtin_popcount(c0) > kw) continue;
            const int4 h4 = *reinterpret_cast<const int4 *>(hitab + c0);  // (entries beyond nhi: masks out of range)
            const int hd[4] = {h4.x, h4.y, h4.z, h4.w};
            int delta[4], key[4];
            bool okv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int c = c0 + u;
              delta[u] = base + hd[u];
              okv[u] = lane_ok && c < nhi && __builtin_popcount(c) <= klim && delta[u] <= room && (c != 0 || lane != 0);
            }
            score4(delta, key);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (okv[u] && key[u] > bk) {
                bk = key[u];
                bm = (c0 + u) * BR_WAVE + lane;
              }
            }
          }
          bestkey = br_wave_max(bk);
          bestmask = bestkey == BR_KEY_NONE ? 0 : br_wave_min(bk == bestkey ? bm : INT32_MAX);
        }
        br_wave_sync();
      } else {
      {
        const int4 lo = *reinterpret_cast<const int4 *>(win);
        const int4 hi = *reinterpret_cast<const int4 *>(win + 4);
        wv[0] = lo.x, wv[1] = lo.y, wv[2] = lo.z, wv[3] = lo.w;
        wv[4] = hi.x, wv[5] = hi.y, wv[6] = hi.z, wv[7] = hi.w;
      }
#pragma unroll
      for (int b = 0; b < 8; ++b) ws[b] = b < w ? (wv[b] >> BR_IDX_BITS) : 0;
      br_wave_sync();  // every lane holds the window before a later pop rewrites it

      // exhaustive subset search: lane l of pass c stands for mask c*64 + l (ascending masks, a later
      // one wins only if strictly better)
      int dv[4];
      bool okv[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        int delta = (c & 1) * ws[6] + (c >> 1) * ws[7];
#pragma unroll
        for (int b = 0; b < 6; ++b)
          if (b < w) delta += lbit[b] * ws[b];
        const int mask = c * BR_WAVE + lane;
        dv[c] = delta;
        okv[c] = mask != 0 && mask < nmask && lpop + __builtin_popcount(c) <= kmax && delta <= room;
      }
      float Fv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      int dmax = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) dmax = max(dmax, okv[c] ? dv[c] : 0);
      dmax = br_wave_max(dmax);
      if (dmax > 0) {  // else no subset is admissible
        if (nmask <= BR_WAVE) {
          const int d1[1] = {dv[0]}, top1[1] = {dmax};
          float F1[1];
          br_scoreh_long_sel<1>(p.aD, p.beta, smg, sd, HS, lane, top1, d1, F1);
          Fv[0] = F1[0];
        } else {
          const int top4[4] = {dmax, dmax, dmax, dmax};
          br_scoreh_long_sel<4>(p.aD, p.beta, smg, sd, HS, lane, top4, dv, Fv);
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c * BR_WAVE < nmask) {
          const int key = okv[c] ? br_ord(Fv[c]) : BR_KEY_NONE;
          const int km = br_wave_max(key);
          if (km > bestkey) {
            bestkey = km;
            bestmask = c * BR_WAVE + (int)__builtin_ctzll(br_ballot(key == km));
          }
        }
      }

      }

      if (bestmask == 0 || bestkey <= 0) {  // starvation guard: the single best request anyway
        ++guard;
        int pos = 0, swin = 0;
        if (!pick(room, pos, swin)) {
          drop_worker(g, capmax);
          continue;
        }
        bind(pos, g, __builtin_amdgcn_readlane(nn, g));
        add_load(g, swin, 1);
      } else {
        // lane b binds window entry b if chosen; slots follow the order of the window
        const int slot = __builtin_amdgcn_readlane(nn, g);
        int delta = 0;
        if (p.R_max > 8) {
          if (lane < 16 && ((bestmask >> lane) & 1))
            adm[win[lane] & IDX_MASK] = (g << 16) | (slot + __builtin_popcount(bestmask & ((1 << lane) - 1)));
          for (int b = 0; b < w; ++b)
            if ((bestmask >> b) & 1) {
              const int e = win[b];
              const int pb = e & IDX_MASK;
              alive = (lane == (pb & 63)) ? (alive & ~(1u << (pb >> 6))) : alive;
              span_dirty = true;
              delta += e >> BR_IDX_BITS;
            }
          br_wave_sync();  // the window has been read before a later pop rewrites it
        } else {
          const bool mine = lane < 8 && ((bestmask >> lane) & 1);
          if (mine) {
            const int me = lane == 0 ? wv[0] : lane == 1 ? wv[1] : lane == 2 ? wv[2] : lane == 3 ? wv[3]
                         : lane == 4 ? wv[4] : lane == 5 ? wv[5] : lane == 6 ? wv[6] : wv[7];
            adm[me & IDX_MASK] = (g << 16) | (slot + __builtin_popcount(bestmask & ((1 << lane) - 1)));
          }
#pragma unroll
          for (int b = 0; b < 8; ++b)
            if ((bestmask >> b) & 1) {
              const int pb = wv[b] & IDX_MASK;
              alive = (lane == (pb & 63)) ? (alive & ~(1u << (pb >> 6))) : alive;
              span_dirty = true;
              delta += ws[b];
            }
        }
        add_load(g, br_uniform(delta), __builtin_popcount(bestmask));
      }
    }
  }
  br_wave_sync();
  if constexpr (NW > 1) {
    mbox[0] = 0;  // the round is over: the helper waves leave
    __syncthreads();
    int32_t *best_i = br_late_out().best_i;
    if (best_i && lane < p.G) {  // lane g: the best of what the waves found for worker g
      int bk = BR_KEY_NONE, bs = 0, bi = -1;
#pragma unroll
      for (int u = 0; u <= RW; ++u) {
        const int *part = mbox + 16 + u * BR_LONG_RED_WORDS(HS, G) + BR_LONG_PART_AT(HS);
        const int k = part[lane], s = part[G + lane], i = part[2 * G + lane];
        const bool better = i >= 0 && (bi < 0 || k > bk || (k == bk && (s > bs || (s == bs && i < bi))));
        bk = better ? k : bk, bs = better ? s : bs, bi = better ? i : bi;
      }
      best_i[(int64_t)inst * p.G + lane] = bi;
    }
#pragma unroll
    for (int u = 1; u < NW; ++u) who[u * BR_WAVE + lane] = -1;  // (held the helpers' partial sums)
    br_wave_sync();
  }

#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int pos = j * BR_WAVE + lane;
    if (pos < qn && adm[pos] >= 0) who[IDX_MASK - (skey[pos] & IDX_MASK)] = adm[pos];
  }
  br_wave_sync();
  BrRoundCounts rc;
  rc.admitted = admitted;
  rc.stage1 = stage1;
  rc.pops = pops;
  rc.guard = guard;
  rc.wdrop = wdrop;
  rc.I_before = I_before;
  br_assign_epilogue<E, true>(inst, lane, q0, qn, cnt, who, Lcur, nn, rc, c0);
}

template <int E>
void br_launch_assign_long_one(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int HS = BR_HS(p.H);
  const int nw = br_long_waves(p);
  const bool best = o.best_g || o.best_i;
  const size_t words = (size_t)3 * E * BR_WAVE + 2 * BR_WAVE + 3 * (size_t)HS + (((size_t)HS * BR_LSTRIDE(p.G) + 3) & ~(size_t)3) +
                       (p.R_max > 8 ? 1024 : 0) + (nw > 1 ? 16 : 0);
  auto lds = [&](int waves) {
    const size_t round = words + (nw > 1 && best ? waves * BR_LONG_RED_WORDS(HS, p.G) : 0);
    return (p.project ? max(round, (size_t)BR_PROJECT_LONG_WORDS(p.G, HS, waves)) + 1 : round) * sizeof(int);
  };
  const dim3 grid((unsigned)p.N), block(BR_WAVE * nw);
  // A CU to each cluster: more waves for the reductions, where 60 KB of LDS hold them.  Three alone take up to 96 pairs of 1200
  // cycles where a token watermark keeps slots free everywhere, and the round waits for them.  One cluster, whole pass, us, a launch
  // of their own / three helper waves / so: such a watermark, H = 80: G = 8, Q = 256 43.9 / 44.6 / 36.7, G = 16, Q = 256 66 / 84 / 57, G = 4,
  // Q = 512 34 / 43 / 33, G = 12, Q = 512 50 / 83 / 56; H = 128: G = 8, Q = 256 46 / 56 / 41, G = 12, Q = 512 55 / 99 / 64; workers nearly
  // full, H = 80: 28.1 / 21.6 / 22.0, 36.0 / 27.3 / 26.5, 28.4 / 22.8 / 22.8, 35.7 / 28.1 / 28.9.  (Q = 256: twelve more 36.6 / 55.4 under the
  // watermark, and 3 % slower on a lightly loaded cluster.)
  auto with = [&](int waves) {  // the last word holds the estimate at age 0 when the blocks form the projections
    BrParams q = p;
    if (q.project) q.project = (int32_t)(lds(waves) / sizeof(int)) - 1;
    return q;
  };
  constexpr int XW = E == 8 ? 8 : E <= 16 ? 4 : 0;
  if (XW > 0 && best && p.N <= BR_LONG_EXTRA_MAX_N && lds(4 + XW) <= 60 * 1024)
    hipLaunchKernelGGL((br_k_assign_long<E, 4, XW>), grid, dim3(BR_WAVE * (4 + XW)), lds(4 + XW), st, with(4 + XW), a, o);
  else if (nw == 4)
    hipLaunchKernelGGL((br_k_assign_long<E, 4>), grid, block, lds(4), st, with(4), a, o);
  else if (nw == 2)
    hipLaunchKernelGGL((br_k_assign_long<E, 2>), grid, block, lds(2), st, with(2), a, o);
  else
    hipLaunchKernelGGL((br_k_assign_long<E, 1>), grid, block, lds(1), st, with(1), a, o);
}
