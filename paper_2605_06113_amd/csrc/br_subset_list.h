// Stage-2 subsets of a window of 9..16 requests when a subset may hold at most half of them: the admissible subsets
// are enumerated themselves, from a constant list of all 16-bit masks ordered by (number of bits, value).
//
// Stage 2 runs where free slots are scarce, so the limit kmax = min(free slots of the worker, R_max) is usually a few:
// of the 65535 masks of a window of 16, 696 have at most three bits.  Within one bit count the masks below 2^w are the
// first C(w, c) of their section, so any window width reads a dense piece of the list.  A mask's sum is two reads of
// tables over its lower and upper byte that the wave builds per pop (256 words each, in LDS).  About 16 instructions
// per 64 masks against 11 of the scan over all masks (br_bigr_scan), which therefore stays for kmax > w / 2 (at 8 of 16
// the list still holds 39202 masks).  Sections up to three bits are 2.8 KB and stay in the L1 cache.
// 1024 clusters, G = 16, window 16, 46 admissions in 19 pops each: round 472 -> 140 us (with br_useful_count below).
#pragma once

#include "br_device.h"

#define BR_LIST_TABLE_WORDS 512  // LDS words of the two byte tables

// An entry holds the byte offsets of the two table reads, the upper byte's in the upper half: entries order as their
// masks do.
struct BrMaskList {
  unsigned v[65536];
};

constexpr BrMaskList br_make_mask_list() {
  BrMaskList t{};
  int at[17] = {};
  int count = 1;  // C(16, c)
  for (int c = 0; c < 16; ++c) {
    at[c + 1] = at[c] + count;
    count = count * (16 - c) / (c + 1);
  }
  for (int v = 0; v < 65536; ++v) {
    int b = v - ((v >> 1) & 0x5555);
    b = (b & 0x3333) + ((b >> 2) & 0x3333);
    b = (b + (b >> 4)) & 0x0f0f;
    b = (b + (b >> 8)) & 0x1f;
    t.v[at[b]++] = (unsigned)((256 + (v >> 8)) * 4) << 16 | (unsigned)((v & 255) * 4);
  }
  return t;
}

static __device__ constexpr BrMaskList br_mask_list = br_make_mask_list();

__device__ __forceinline__ int br_list_mask(unsigned v) { return (int)(((v >> 18) - 256u) << 8 | (v & 0xffffu) >> 2); }

// Which of the two exact searches of a window of up to 16 requests: the list, or the scan over all masks.
__device__ __forceinline__ bool br_list_serves(int w, int kmax) { return 2 * kmax <= w; }

// number of non-empty subsets of w requests with at most kmax of them
__device__ __forceinline__ int br_list_size(int w, int kmax) {
  int n = 0, c_w = 1;
  for (int c = 1; c <= kmax; ++c) {
    c_w = c_w * (w - c + 1) / c;
    n += c_w;
  }
  return n;
}

// Sum of the lane + 1 smallest entries of a window of up to 32 requests (sorted, longest first), for lanes below w.
__device__ __forceinline__ int br_min_sums(const int *win, int w, int lane) {
  int x = lane < w ? win[max(w - 1 - lane, 0)] >> BR_IDX_BITS : 0;
  x += br_dpp<0x111>(0, x);       // row_shr:1
  x += br_dpp<0x112>(0, x);       // row_shr:2
  x += br_dpp<0x114>(0, x);       // row_shr:4
  x += br_dpp<0x118>(0, x);       // row_shr:8
  x += br_dpp<0x142, 0x2>(0, x);  // row_bcast:15 into row 1
  return x;
}

// Most requests a subset of the window can usefully hold, at most kmax.  Lane c - 1 passes the sum of the c smallest
// entries and its score as computed; `slack` is four times the rounding bound of a score of any subset (0 for exact
// scores).  The score is concave in the sum: when the c smallest entries score below the c - 1 smallest (by more than
// the slack), the score falls from there on, and every subset of c or more requests, whose sum is no smaller, computes
// strictly below the c - 1 smallest entries, which are a candidate.  Sums beyond `room` end the row as well.
__device__ __forceinline__ int br_useful_count(int sum, float F, float slack, int room, int kmax, int lane) {
  const float prev = __int_as_float(__builtin_amdgcn_ds_bpermute(max(lane - 1, 0) << 2, __float_as_int(F)));
  const bool stop = lane >= 1 && (F < prev - slack || sum > room);
  const unsigned long long bal = br_ballot(stop);
  return bal != 0ull ? min(kmax, (int)__builtin_ctzll(bal)) : kmax;
}

// Sums of the window entries selected by the lower (tab[0..255]) and the upper byte (tab[256..511]) of a mask.
__device__ __forceinline__ void br_list_tables(const int *win, int w, int *tab, int lane) {
  int lo = 0, hi = 0;
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    lo += ((lane >> b) & 1) * (b < w ? win[b] >> BR_IDX_BITS : 0);
    hi += ((lane >> b) & 1) * (8 + b < w ? win[8 + b] >> BR_IDX_BITS : 0);
  }
  const int l6 = 6 < w ? win[6] >> BR_IDX_BITS : 0, l7 = 7 < w ? win[7] >> BR_IDX_BITS : 0;
  const int h6 = 14 < w ? win[14] >> BR_IDX_BITS : 0, h7 = 15 < w ? win[15] >> BR_IDX_BITS : 0;
  tab[lane] = lo, tab[64 + lane] = lo + l6, tab[128 + lane] = lo + l7, tab[192 + lane] = lo + l6 + l7;
  tab[256 + lane] = hi, tab[320 + lane] = hi + h6, tab[384 + lane] = hi + h7, tab[448 + lane] = hi + h6 + h7;
}

// Walks the admissible subsets of the window, NV per lane and trip; wave wv of nwv takes every nwv-th trip.
// score(delta[NV], key[NV]) gives the keys; the lane keeps its best key and, among equal ones, the lowest mask.
// In a window of 16 the sections follow each other without a gap and are walked as one; the last trip repeats the
// last entry on the lanes beyond it, which changes no maximum.
template <int NV, class Score>
__device__ __forceinline__ void br_list_walk(const int *tab, int w, int kmax, int room, int lane, int wv, int nwv, Score score,
                                             int &bk, int &bm) {
  bk = BR_KEY_NONE;
  unsigned bv = 0xffffffffu;
  auto walk = [&](int off, int n) {
    for (int i0 = wv * NV * BR_WAVE; i0 < n; i0 += nwv * NV * BR_WAVE) {
      unsigned e[NV];
      int delta[NV], key[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) e[v] = br_mask_list.v[off + min(i0 + v * BR_WAVE + lane, n - 1)];
#pragma unroll
      for (int v = 0; v < NV; ++v)
        delta[v] = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(tab) + (e[v] & 0xffffu)) +
                   *reinterpret_cast<const int *>(reinterpret_cast<const char *>(tab) + (e[v] >> 16));
      score(delta, key);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int k = delta[v] <= room ? key[v] : BR_KEY_NONE;
        if (k > bk || (k == bk && e[v] < bv)) bk = k, bv = e[v];
      }
    }
  };
  if (w == 16) {
    walk(1, br_list_size(w, kmax));
  } else {
    int off = 1, c_w = 1, c_16 = 1;
    for (int c = 1; c <= kmax; ++c) {
      c_w = c_w * (w - c + 1) / c;
      c_16 = c_16 * (17 - c) / c;
      walk(off, c_w);
      off += c_16;
    }
  }
  bm = bk == BR_KEY_NONE ? INT32_MAX : br_list_mask(bv);
}
