// The waiting set of a round as a sorted list in the registers of one wavefront.
//
// An entry is prefill length << 11 | 2047 - arrival position: all entries differ, and one unsigned order gives "longest
// first, earlier arrival first".  Position = lane * E + j (x[j] of the lane), descending, the list always dense: an
// entry that leaves is squeezed out, so neighbours in length are neighbours in position and no search has to look at
// who is still waiting.  Entries consumed from the front in bulk read as ~0 (above every key), positions beyond the end
// as 0.  The layout is what makes this cheap: squeezing out shifts registers within a lane (two instructions per
// register and one wave-wide DPP shift), a search by length is one compare and ballot over the lanes' first entries and
// a look at one lane.
#pragma once

#include "br_device.h"

#define BR_ENTRY_GONE 0xffffffffu  // consumed from the front

// median of three: max(a, b) where c is all ones, min(a, b) where c is zero (one instruction)
__device__ __forceinline__ unsigned br_med3(unsigned a, unsigned b, unsigned c) { return max(min(a, b), min(max(a, b), c)); }

// all ones on the lanes whose bit S (a power of two) is set
template <int S>
__device__ __forceinline__ unsigned br_lane_bit(int lane) {
  return S >= BR_WAVE ? 0u : (unsigned)__builtin_amdgcn_sbfe(lane, __builtin_ctz(S), 1);
}

// max or min (c: all ones or zero) of a lane's key and that of the lane S away (lane ^ S), on the VALU throughout
template <int S>
__device__ __forceinline__ unsigned br_exchange(unsigned x, unsigned c) {
  if constexpr (S == 1) {
    return br_med3(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true), c);  // quad_perm [1,0,3,2]
  } else if constexpr (S == 2) {
    return br_med3(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true), c);  // quad_perm [2,3,0,1]
  } else if constexpr (S == 4) {
    int y = __builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);  // row_half_mirror: lane ^ 7
    y = __builtin_amdgcn_update_dpp(0, y, 0x1B, 0xF, 0xF, true);            // quad_perm [3,2,1,0]: lane ^ 3
    return br_med3(x, (unsigned)y, c);
  } else if constexpr (S == 8) {
    return br_med3(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true), c);  // row_ror:8
  } else if constexpr (S == 16) {  // both keys of the pair on both of its lanes
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return br_med3(r[0], r[1], c);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return br_med3(r[0], r[1], c);
  }
}

// One stage (partner distance S in position) of the bitonic merge of blocks of K positions.
template <int E, int K, int S>
__device__ __forceinline__ void br_list_stage(unsigned (&x)[E], int lane) {
  if constexpr (S < E) {  // partners are two registers of one lane
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if ((j & S) == 0) {
        const unsigned a = x[j], b = x[j | S];
        if constexpr (K < E) {
          x[j] = (j & K) == 0 ? max(a, b) : min(a, b);
          x[j | S] = (j & K) == 0 ? min(a, b) : max(a, b);
        } else {
          const unsigned up = br_lane_bit<K / E>(lane);  // this block sorts upwards
          x[j] = br_med3(a, b, ~up);
          x[j | S] = br_med3(a, b, up);
        }
      }
    }
  } else {
    const unsigned c = ~(br_lane_bit<S / E>(lane) ^ br_lane_bit<K / E>(lane));
#pragma unroll
    for (int j = 0; j < E; ++j) x[j] = br_exchange<S / E>(x[j], c);
  }
  if constexpr (S > 1) br_list_stage<E, K, S / 2>(x, lane);
}

// Bitonic sort of all E * 64 positions, descending.  E = 4: 36 stages, 15 of them within a lane, about 220 instructions.
template <int E, int K = E * BR_WAVE>
__device__ __forceinline__ void br_list_sort(unsigned (&x)[E], int lane) {
  if constexpr (K > 2) br_list_sort<E, K / 2>(x, lane);
  br_list_stage<E, K, K / 2>(x, lane);
}

// The neighbours of threshold T (>= 1) within the registers [J, J + N) of lane l, given below = the first of them or
// an entry before it, above = what follows the last: narrowed by halves down to four, then by selects.
template <int J, int N, int E>
__device__ __forceinline__ void br_list_narrow(const unsigned (&x)[E], int l, unsigned T, unsigned &at_or_above, unsigned &below) {
  if constexpr (N > 4) {
    const unsigned mid = (unsigned)__builtin_amdgcn_readlane((int)x[J + N / 2], l);
    if (mid >= T) {
      at_or_above = mid;
      br_list_narrow<J + N / 2, N / 2>(x, l, T, at_or_above, below);
    } else {
      below = mid;
      br_list_narrow<J, N / 2>(x, l, T, at_or_above, below);
    }
  } else {
    unsigned r[N];
#pragma unroll
    for (int k = 1; k < N; ++k) r[k] = (unsigned)__builtin_amdgcn_readlane((int)x[J + k], l);
#pragma unroll
    for (int k = 1; k < N; ++k) at_or_above = r[k] >= T ? r[k] : at_or_above;
#pragma unroll
    for (int k = N - 1; k >= 1; --k) below = r[k] < T ? r[k] : below;
  }
}

// Last entry at or above T (0: none) and first entry below it (0: none), uniform.  1 <= T < BR_ENTRY_GONE.
// Lists of one or four registers: by selects throughout (a branch costs as much as four or more instructions).
template <int E>
__device__ __forceinline__ void br_list_around(const unsigned (&x)[E], unsigned T, unsigned &at_or_above, unsigned &below) {
  const int l = __builtin_popcountll(br_ballot(x[0] >= T)) - 1;  // the lane in which the list crosses T
  if constexpr (E <= 4) {
    unsigned r[E];
#pragma unroll
    for (int j = 0; j < E; ++j) r[j] = (unsigned)__builtin_amdgcn_readlane((int)x[j], max(l, 0));
    const unsigned next = (unsigned)__builtin_amdgcn_readlane((int)x[0], (l + 1) & 63);
    at_or_above = 0u, below = l < 63 ? next : 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) at_or_above = r[j] >= T ? r[j] : at_or_above;
#pragma unroll
    for (int j = E - 1; j >= 0; --j) below = r[j] < T ? r[j] : below;
  } else {
    const unsigned next = l < 63 ? (unsigned)__builtin_amdgcn_readlane((int)x[0], (l + 1) & 63) : 0u;
    at_or_above = 0u, below = next;
    if (l >= 0) {
      at_or_above = (unsigned)__builtin_amdgcn_readlane((int)x[0], l);
      br_list_narrow<0, E>(x, l, T, at_or_above, below);
    }
  }
}

// Squeezes entry K (a key of the list) out: what follows it moves up by one.
template <int E>
__device__ __forceinline__ void br_list_remove(unsigned (&x)[E], unsigned K) {
  const unsigned next = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x[0], 0x130, 0xF, 0xF, false);  // wave_shl:1
  unsigned y[E + 1];
#pragma unroll
  for (int j = 0; j < E; ++j) y[j] = x[j];
  y[E] = next;
#pragma unroll
  for (int j = 0; j < E; ++j) x[j] = y[j] <= K ? y[j + 1] : y[j];
}

// LDS copy of the list (E * 64 words, one spare word per 32 from E = 16 on, where a lane's entries would otherwise all
// start in the same bank).
template <int E>
__device__ __forceinline__ int br_list_at(int pos) {
  return E >= 16 ? pos + (pos >> 5) : pos;
}
#define BR_LIST_WORDS(E) ((E) >= 16 ? (E) * 66 : (E) * 64)

template <int E>
__device__ __forceinline__ void br_list_store(const unsigned (&x)[E], int *lst, int lane) {
  if constexpr (E == 4 || E == 8) {
#pragma unroll
    for (int j = 0; j < E; j += 4)
      *reinterpret_cast<int4 *>(lst + lane * E + j) = make_int4((int)x[j], (int)x[j + 1], (int)x[j + 2], (int)x[j + 3]);
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) lst[br_list_at<E>(lane * E + j)] = (int)x[j];
  }
}

// the n entries from position `by` of the LDS copy on, at the front of the list
template <int E>
__device__ __forceinline__ void br_list_load(unsigned (&x)[E], const int *lst, int lane, int by, int n) {
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int p = lane * E + j;
    const unsigned v = (unsigned)lst[br_list_at<E>(min(p + by, E * BR_WAVE - 1))];
    x[j] = p < n ? v : 0u;
  }
}
