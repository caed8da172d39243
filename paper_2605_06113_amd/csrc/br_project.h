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

// The projection and, in the same pass over the lists, the decode steps of their old entries (br_route_advance): neither
// needs the round, which reads the projections and appends its admissions to the lists as they are left here
// (br_assign_epilogue_ahead).  LPL lanes hold a list as in br_k_advance_seg, four consecutive slots each; a request's row
// is read, and stored again where it moves, by the lane whose number follows that of the slot (contiguous memory).
// What a list lost and its load change go to the words of its margins (br_ahead_store); length and load stay until the
// round has read them.
// Bound by memory traffic (4096 clusters, G = 32, H = 4, lists of 96 slots, 40 steps: 432 MB in 106 us, 4.1 TB/s; the projection by itself 73 us
// from cold memory).  Non-temporal stores, or two lists a lane group at a time, make no difference; non-temporal loads cost 7 us.
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
