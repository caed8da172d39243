// Sorts of a waiting set beyond one list in registers (br_list.h): by the four waves of a block, and on one wave with the
// result across the lanes.
//
// Both are the bitonic sort of br_list.h, whose positions lie lane * E + j: partners up to E positions apart are two registers
// of one lane (a min and a max, or two med3), the others one DPP or permlane move and a med3.  With positions j * 64 + lane nearly
// every stage is a move between lanes, some of them through LDS.  Whole pass, us, so laid out / as lists of no more registers than
// hold the waiting set: one cluster, G = 64, H = 8, a queue of 2048 42.5 / 39.4, H = 0, 1500 27.0 / 24.4; H = 80 on one wave: a queue of
// 2048 70.2 / 50.7, of 1024 40.2 / 32.5; 300 clusters, 1000 64.5 / 54.6; 100 clusters, 2048, 30 admissions each 168 / 131.
#pragma once

#include <type_traits>

#include "br_list.h"

// Sort of up to 2048 keys (the first qn; the others are zero) by the four waves of a block, 512 per wave (8 registers per lane):
// position = w * 512 + lane * 8 + j, descending over the whole block.  Each wave sorts its own 512, then two merge levels follow
// (none where fewer wait).  A level starts by comparing the two sorted halves mirrored (element i of the first with element
// n-1-i of the second, through `buf` in LDS); after that every element of the first half is at least every element of the second
// and each half is bitonic, so halves are finished by plain half-cleaners: across waves at distance 512 (same position in the
// partner wave), inside a wave by the stages of a list.  Every wave of the block must call this with the same qn (block barriers).
__device__ __forceinline__ void br_sort_block4_exchange(unsigned (&x)[8], int *buf, int w, int lane, int partner,
                                                        bool mirrored, bool keep_max) {
  int4 *mine = reinterpret_cast<int4 *>(buf + w * 512 + lane * 8);
  mine[0] = make_int4((int)x[0], (int)x[1], (int)x[2], (int)x[3]);
  mine[1] = make_int4((int)x[4], (int)x[5], (int)x[6], (int)x[7]);
  __syncthreads();
  const int4 *other = reinterpret_cast<const int4 *>(buf + partner * 512 + (mirrored ? 63 - lane : lane) * 8);
  const int4 a = other[0], b = other[1];
  __syncthreads();
  const int z[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const unsigned y = (unsigned)(mirrored ? z[7 - j] : z[j]);
    x[j] = keep_max ? max(x[j], y) : min(x[j], y);
  }
}

__device__ __forceinline__ void br_sort_desc_block4(unsigned (&x)[8], int *buf, int w, int lane, int qn) {
  br_list_sort<8>(x, lane);
  if (qn > 512) {
    br_sort_block4_exchange(x, buf, w, lane, w ^ 1, true, (w & 1) == 0);   // pairs of waves: 1024 keys each
    br_list_stage<8, 512, 256>(x, lane);
  }
  if (qn > 1024) {
    br_sort_block4_exchange(x, buf, w, lane, 3 - w, true, w < 2);          // all four: 2048 keys
    br_sort_block4_exchange(x, buf, w, lane, w ^ 1, false, (w & 1) == 0);
    br_list_stage<8, 512, 256>(x, lane);
  }
}

// Sort of E * 64 keys on one wave, the first qn of them not zero, descending by position j * 64 + lane: as a list of as many
// registers as hold them, then through buf (E * 64 words of LDS).
template <int E>
__device__ __forceinline__ void br_sort_across(unsigned (&x)[E], int *buf, int lane, int qn) {
  auto as_list = [&](auto n) {
    constexpr int N = decltype(n)::value;
    unsigned y[N];
#pragma unroll
    for (int j = 0; j < N; ++j) y[j] = x[j];
    br_list_sort<N>(y, lane);
    if constexpr (N == 1) {
      x[0] = y[0];
    } else {
#pragma unroll
      for (int j = 0; j < N; j += 4)
        *reinterpret_cast<int4 *>(buf + lane * N + j) = make_int4((int)y[j], (int)y[j + 1], (int)y[j + 2], (int)y[j + 3]);
      br_wave_sync();
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = (unsigned)buf[j * BR_WAVE + lane];
    }
  };
  if (qn <= BR_WAVE)
    as_list(std::integral_constant<int, 1>{});
  else if (E == 4 || qn <= 4 * BR_WAVE)
    as_list(std::integral_constant<int, 4>{});
  else if (E == 8 || qn <= 8 * BR_WAVE)
    as_list(std::integral_constant<int, E < 8 ? E : 8>{});
  else if (E == 16 || qn <= 16 * BR_WAVE)
    as_list(std::integral_constant<int, E < 16 ? E : 16>{});
  else
    as_list(std::integral_constant<int, E>{});
}
