// Projected loads of short horizons (H <= BR_HP): what a prediction row means, and the pass over the lists that forms the
// projections and applies the decode steps to the entries as they stand.
#pragma once

#include "br_advance_seg.h"
#include "br_device.h"
#include "br_score_wave.h"

// c_hat of one active request (Appendix "Short-horizon prediction interface"): the survival sum
// of the hazards = E[min(r, H)] (eq. (two-stage)/(composite)) in sequential fp32, the p_fin gate and the floor
// of Appendix "Refresh logic", clip to [1, H]; or eq. (composite) on a supplied (p_fin, mu_rem) with the same gate;
// or the supplied / maintained value itself; all floored and clipped the same way.  A request counts kv + h at the offsets
// h <= floor(c_hat) (h is an integer, so that is (float)h <= c_hat; a NaN counts nowhere).
// PK, the kind of row: 0 a hazard per offset, 1 c_hat itself first in the row, 2 the pair (p_fin, mu_rem).  HB: 4 or 8 offsets
// beyond h = 0; EXACT: H == HB.
#define BR_ROW_FLOATS(HB, PK) ((PK) == 0 ? (HB) : (PK) == 2 ? 2 : 1)
// the last offset at which a request with this row counts, or -1
template <int HB, bool EXACT, int PK>
__device__ __forceinline__ int br_last_offset(const BrParams &p, const float (&row)[BR_ROW_FLOATS(HB, PK)]) {
  const float Hf = (float)p.H;
  float ch;
  if constexpr (PK == 0) {
    float S = 1.0f;
    ch = 0.0f;
#pragma unroll
    for (int q = 0; q < HB; ++q) {
      if (EXACT || q < p.H) {
        ch = __fadd_rn(ch, S);
        S = __fmul_rn(S, __fsub_rn(1.0f, row[q]));
      }
    }
    const float pfin = __fsub_rn(1.0f, S);
    if (p.gate > 0.0f && pfin < p.gate) ch = Hf;
  } else if constexpr (PK == 2) {
    const float pf = row[0], mu = row[1];
    ch = __fadd_rn(__fmul_rn(__fsub_rn(1.0f, pf), Hf), __fmul_rn(pf, mu));
    if (p.gate > 0.0f && pf < p.gate) ch = Hf;
  } else {
    ch = row[0];
  }
  ch = ch < 1.0f ? 1.0f : ch;
  ch = ch > Hf ? Hf : ch;
  return ch >= 1.0f ? (int)ch : -1;
}

// The projection and, in the same pass over the lists, the decode steps of their old entries (br_route_advance; br_project_advances): neither
// needs the round, which reads the projections and appends its admissions to the lists as they are left here
// (br_assign_epilogue_ahead).  LPL lanes hold a list as in br_k_advance_seg, four consecutive slots each; a request's row
// is read, and stored again where it moves, by the lane whose number follows that of the slot (contiguous memory).
// What a list lost and its load change go to the words of its margins (br_ahead_store); length and load stay until the
// round has read them.
// Bound by memory traffic (4096 clusters, G = 32, H = 4, lists of 96 slots, 40 steps: 448 MB in 107 us, 4.2 TB/s, both
// over passes on three states in turn; the projection by itself 73 us from cold memory).  Non-temporal stores, or two lists a lane group at a time, make no difference; non-temporal loads cost 7 us.
// row0: the first of `lists` lists (at most 64 / LPL); lds: BR_SEG_WORDS(1) of the wave's.
template <int LPL, int HB, bool EXACT, int PK>
__device__ __forceinline__ void br_project_lists(const BrParams &p, int64_t row0, int lists, int lane, int *lds) {
  constexpr int NF = BR_ROW_FLOATS(HB, PK);
  const int t = p.adv_t, P = EXACT && PK == 0 ? HB : p.P;
  const int lseg = lane & (LPL - 1), e0 = 4 * lseg, list = min(lane / LPL, lists - 1);
  const bool ok = lane / LPL < lists;
  const BrSegBase b = br_seg_base(p, row0);
  short *map = reinterpret_cast<short *>(lds + BR_SEG_LIST_WORDS);
  int n = ok ? br_seg_at<int>(b.n, 4u * (unsigned)list) : 0;
  BrSegSlots<1> v;
  br_seg_load<LPL, 1>(b, p.Bs, list, ok ? p.Bs : 0, lane, v);
  n = min(max(n, 0), p.B);
  auto row_at = [&](int slot) { return 4u * (unsigned)((list * p.Bs + slot) * P); };
  float q[4][NF];
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // (beyond the list: its last row again, without a branch)
    const unsigned at = row_at(min(lseg + k * LPL, max(n - 1, 0)));
    if constexpr (PK == 0 && EXACT) {
#pragma unroll
      for (int c = 0; c < HB; c += 4) {
        const float4 f = br_seg_at<float4>(b.pred, at + 4u * c);
        q[k][c] = f.x, q[k][c + 1] = f.y, q[k][c + 2] = f.z, q[k][c + 3] = f.w;
      }
    } else if constexpr (PK == 2) {
      const float2 f = br_seg_at<float2>(b.pred, at);
      q[k][0] = f.x, q[k][1] = f.y;
    } else {
#pragma unroll
      for (int c = 0; c < NF; ++c) q[k][c] = c < P ? br_seg_at<float>(b.pred, at + 4u * c) : 0.0f;
    }
  }
  short *last = reinterpret_cast<short *>(lds) + (lane - lseg) * 4;  // of the list's slots: last offset they count at
#pragma unroll
  for (int k = 0; k < 4; ++k) last[lseg + k * LPL] = (short)br_last_offset<HB, EXACT, PK>(p, q[k]);
  br_wave_sync();
  const short4 l4 = *reinterpret_cast<const short4 *>(last + e0);
  const int hm[4] = {l4.x, l4.y, l4.z, l4.w}, kv[4] = {v.kv4.x, v.kv4.y, v.kv4.z, v.kv4.w};
  int sum[HB + 1];
#pragma unroll
  for (int h = 0; h <= HB; ++h) sum[h] = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int upto = e0 + k < n ? hm[k] : -1;
#pragma unroll
    for (int h = 0; h <= HB; ++h) sum[h] += h <= upto ? kv[k] + h : 0;
  }
  br_seg_sums<LPL>(sum);
  br_wave_sync();  // the words are rewritten below
  BrSegPlan d;
  br_seg_decide<LPL, 1>(p, t, n, lane, v, lds, map, d);
  br_seg_store<LPL, 1>(b, p.Bs, list, lane, v, d, lds);
  if (ok && lseg == LPL - 1) {
    const int64_t row = row0 + list;
#pragma unroll
    for (int h = 0; h <= HB; ++h)
      if (EXACT || h <= p.H) p.Lh[row * (p.H + 1) + h] = sum[h];
    br_ahead_store(p, row, n - d.kept, d.kept * t - d.gone);
  }
  if (d.any) {  // rows follow their requests
    const short *to = map + (lane - lseg) * 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = lseg + k * LPL, s = to[j];
      if (j < n && s >= 0 && s != j) {
        const unsigned at = row_at(s);
        if constexpr (PK == 0 && EXACT) {
#pragma unroll
          for (int c = 0; c < HB; c += 4)
            br_seg_at<float4>(b.pred, at + 4u * c) = make_float4(q[k][c], q[k][c + 1], q[k][c + 2], q[k][c + 3]);
        } else if constexpr (PK == 2) {
          br_seg_at<float2>(b.pred, at) = make_float2(q[k][0], q[k][1]);
        } else {
#pragma unroll
          for (int c = 0; c < NF; ++c)
            if (c < P) br_seg_at<float>(b.pred, at + 4u * c) = q[k][c];
        }
      }
    }
  }
}

// Horizons beyond BR_HP (Appendix "Short-horizon prediction interface", eq. (wprofile-new)): a request counts
// kv + h at the offsets h <= c_hat, so one histogram of floor(c_hat) per worker (count and kv sum, in LDS) and
// its suffix sums give L_g(k+h) = sum_{c >= h} kvsum[c] + h * sum_{c >= h} count[c] without a register per
// offset.  Integer sums, so the order of accumulation does not matter.  One block per cluster: each wave takes
// every fourth worker list and leaves its row in an LDS tile as well; then, with threads mapped to offsets,
// the envelope M_h = max_g L_g(k+h) and the margins, and with threads mapped to workers the horizon-min
// margin (short horizons: by the round's wave, br_store_margins).
// The lists of a wave are taken in units of 64 slots with the next unit requested before the one in hand is used; suffix
// sums are wave-wide DPP scans with lanes mapped to offsets in descending order (a walk over all bins on every lane took
// 750 instructions per list).  2048 clusters, G = 8, B = 64, H = 80: 36 -> 10 us.  By NW waves of a block, each in its own part of
// LDS: in a launch of its own, or by those that go on with the cluster's round (br_k_assign_long).
#define BR_BINS 192  // offsets 0..BR_HL in whole waves
#define BR_PROJECT_LONG_WORDS(G, HS, NW) (((G) + 1) * (HS) + 2 * (NW) * BR_BINS)
template <int NW>
__device__ __forceinline__ void br_project_long(const BrParams &p, int inst, int tid, int *lds) {
  const int wave = br_uniform(tid >> 6), lane = br_lane();
  const int G = p.G, H = p.H, H1 = H + 1, HS = BR_HS(H);
  int *tile = lds;                                     // [G][HS] projections
  int *sM = lds + G * HS;                              // [HS] envelope
  int *cnt = sM + HS + wave * 2 * BR_BINS;             // this wave's histogram: requests whose last offset is c
  int *kvs = cnt + BR_BINS;                            // ... and the sum of their kv
  const float Hf = (float)H;
  const int64_t row0 = (int64_t)inst * G;
  const int mine = wave + NW * lane;                    // lane i: length of this wave's i-th list
  const int nn = mine < G ? min(max(p.n[row0 + mine], 0), p.B) : 0;
#pragma unroll
  for (int u = 0; u < BR_BINS / BR_WAVE; ++u) cnt[u * BR_WAVE + lane] = 0, kvs[u * BR_WAVE + lane] = 0;
  br_wave_sync();
  auto fetch = [&](int g, int j0, int &kv, float &c, float &c2) {  // (whole rows: no wait for the length)
    const int64_t at = (row0 + g) * p.Bs + min(j0 + lane, p.Bs - 1);
    kv = p.kv[at];
    c = p.pred[at * p.P];  // pred_mode 1 and 2 keep c_hat first
    c2 = p.pred_mode == 3 ? p.pred[at * p.P + 1] : 0.0f;
  };
  int kv_n = 0;
  float c_n = 0.0f, c2_n = 0.0f;
  if (wave < G) fetch(wave, 0, kv_n, c_n, c2_n);
  for (int g = wave; g < G; g += NW) {
    const int64_t row = row0 + g;
    const int n = __builtin_amdgcn_readlane(nn, (g - wave) / NW);
    int topc = 0, topk = 0;  // requests that reach the last offset (the gate's anchor: the common case)
    for (int j0 = 0; j0 < max(n, 1); j0 += BR_WAVE) {
      const int j = j0 + lane;
      const int kv = kv_n;
      float c = c_n;
      const float mu = c2_n;
      const int gn = j0 + BR_WAVE < n ? g : g + NW, jn = j0 + BR_WAVE < n ? j0 + BR_WAVE : 0;  // the next unit
      if (gn < G) fetch(gn, jn, kv_n, c_n, c2_n);
      if (p.pred_mode == 3) {              // the pair (p_fin, mu_rem): eq. (composite) and the gate
        const float pf = c;
        c = __fadd_rn(__fmul_rn(__fsub_rn(1.0f, pf), Hf), __fmul_rn(pf, mu));
        if (p.gate > 0.0f && pf < p.gate) c = Hf;
      }
      c = c < 1.0f ? 1.0f : c;
      c = c > Hf ? Hf : c;
      int hm = -1;
      if (j < n && c >= 0.0f) hm = min((int)c, H);  // offsets h with (float)h <= c_hat are 0..floor(c_hat); a NaN counts nowhere
      const bool top = hm == H;
      topc += __builtin_popcountll(br_ballot(top));
      topk += top ? kv : 0;
      if (hm >= 0 && !top) {
        atomicAdd(&cnt[hm], 1);
        atomicAdd(&kvs[hm], kv);
      }
    }
    topk = br_wave_sum(topk);
    br_wave_sync();
    // suffix sums: lane l of chunk u stands for offset 64 u + 63 - l; the chunks above are in the carry
    int Cc = topc, Kc = topk;
#pragma unroll
    for (int u = BR_BINS / BR_WAVE - 1; u >= 0; --u) {
      if (u * BR_WAVE < H1) {
        const int h = u * BR_WAVE + 63 - lane;
        const int C = br_scan_sum(cnt[h]) + Cc, K = br_scan_sum(kvs[h]) + Kc;
        cnt[h] = 0, kvs[h] = 0;
        Cc = __builtin_amdgcn_readlane(C, 63), Kc = __builtin_amdgcn_readlane(K, 63);
        if (h < H1) {
          const int v = K + h * C;
          p.Lh[row * H1 + h] = v;
          tile[g * HS + h] = v;
        }
      }
    }
    br_wave_sync();  // the histogram is filled again for this wave's next list
  }
  __syncthreads();
  for (int h = tid; h < H1; h += 64 * NW) {  // thread = offset
    int M = tile[h];
    for (int g = 1; g < G; ++g) M = max(M, tile[g * HS + h]);
    p.Mh[(int64_t)inst * H1 + h] = M;
    sM[h] = M;
  }
  __syncthreads();
  for (int g = wave; g < G; g += NW) {  // wave = worker, lane = offset
    int mn = INT32_MAX;
    for (int h = lane; h < H1; h += BR_WAVE) {
      const int m = max(sM[h] - tile[g * HS + h], 0);
      p.mh[(row0 + g) * H1 + h] = m;
      mn = min(mn, m);
    }
    mn = br_wave_min(mn);
    if (lane == 0) p.minm[row0 + g] = mn;
  }
}

// br_survival at age 0 by a whole wave: both ranks by 64 pivots a step, where a lane alone halves.
__device__ __forceinline__ float br_survival_start(const BrParams &p, int lane) {
  int step = p.hist_n > 0 ? 1 : 0, lo = 0, hi = 0;
  while (step > 0 && (long long)step * BR_WAVE < p.hist_n) step *= BR_WAVE;
  for (; step > 0; step /= BR_WAVE) {
    const int a = lo + (lane + 1) * step, b = hi + (lane + 1) * step;
    const int va = p.hist[min(a, p.hist_n) - 1], vb = p.hist[min(b, p.hist_n) - 1];
    lo += step * __builtin_popcountll(br_ballot(a <= p.hist_n && va <= 0));
    hi += step * __builtin_popcountll(br_ballot(b <= p.hist_n && vb <= p.H));
  }
  return br_survival_at(p, 0, lo, hi, p.hsum[lo], p.hsum[hi]);
}
