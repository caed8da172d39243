// BR-0, Stage 2: the best subset of a window of up to 16 requests with at most kmax of them, kmax = 3..5, every admissible
// sum formed.
//
// eq. (br0-Fscore) rises with the sum up to the margin and falls beyond it (G >= 2), so the largest sum up to T = min(margin,
// room) and the smallest one above it decide.  With d = T - sum as an unsigned word both are extremes of one order: the smallest d
// is the one, the largest the other, so a sum costs a subtraction, half a min3 and half a max3.  The upper byte of
// the mask rides in the low bits of d, so the smallest d names the lowest upper byte as well and four ballots find the lowest
// lower one; for a sum above the margin the walk is run again with T at that sum (one search in G or so).
// Sums of the window's lower half lie on the lanes in order of their number of requests (those of at most j are the first
// C(8, <= j)); each of the upper half's, read from LDS for the whole wave, meets the lanes' sums that its own number of
// requests leaves.  Where that leaves one request, seven upper subsets share a wave (9 lanes each), where it leaves none, 64.
// 15 wave-wide sums at kmax = 3, 57 at 4 and 151 at 5 (696, 2516 and 6884 subsets).  Loops with few sums a turn wait for LDS at
// every turn and are slower than what they replace, so this is straight code, one piece per kmax.
// 1024 clusters, G = 16, 46 admissions in 18 pops each (limits of 1 to 7), whole pass: window 16 71 -> 60 us (before: triples
// by a list at 3, the sums of the halves beyond), window 12 72 -> 64, window 9 (the list of masks) 69 -> 63.
#pragma once

#include <type_traits>

#include "br_subset_list.h"

#define BR_FEW_WORDS 515           // LDS words: lower sums, upper ones behind them (three words on: every section is aligned)
#define BR_FEW_ABSENT (1 << 21)    // length of a request the window does not hold: above every sum and every T (2^20)

// Limits it serves: 1 and 2 are fewer sums than its tables are words (window 16: 64 us without, 67 with them), and 6 takes 311
// wave-wide sums (66 us with it where limits of 3 stay by the list, 65 without).  Windows of up to 8 are one trip of the scan over
// all masks, except that triples there had a list of their own.
#define BR_FEW_MIN 3
#define BR_FEW_MAX 5
__device__ __forceinline__ bool br_few_serves(int w, int kmax) {
  return kmax >= BR_FEW_MIN && kmax <= BR_FEW_MAX && (w > 8 || kmax == BR_FEW_MIN);
}

// Byte values in order of (bits, value): their places, four to a word, by value & 63 with value >> 6 as the byte.
struct BrFewPlaces {
  unsigned v[64];
};
constexpr BrFewPlaces br_make_few_places() {
  BrFewPlaces t{};
  int at = 0;
  for (int c = 0; c <= 8; ++c)
    for (int v = 0; v < 256; ++v) {
      int b = 0;
      for (int k = 0; k < 8; ++k) b += (v >> k) & 1;
      if (b == c) t.v[v & 63] |= (unsigned)at++ << (8 * (v >> 6));
    }
  return t;
}
static __device__ constexpr BrFewPlaces br_few_places = br_make_few_places();

// byte values of fewer than c bits
constexpr int br_few_below(int c) {
  int n = 0, k = 1;
  for (int i = 0; i < c; ++i) n += k, k = k * (8 - i) / (i + 1);
  return n;
}

// Bit 31 is turned so that signed extremes are those of the unsigned words.  dn, dx: the lane's smallest and largest d.
// Straight code but for the long sections: a loop with a few sums a turn waits for LDS at each.
template <int KMAX>
__device__ __forceinline__ void br_few_walk(const int *lower, const int *upper, int lane, int &dn, int &dx) {
  auto take = [&](int a, int b) {
    dn = min(dn, min(a, b));
    dx = max(dx, max(a, b));
  };
  constexpr int REGS = (br_few_below(KMAX + 1) + BR_WAVE - 1) / BR_WAVE;
  int low[REGS];
#pragma unroll
  for (int r = 0; r < REGS; ++r) low[r] = lower[r * BR_WAVE + lane];
  auto section = [&](auto cc) {  // upper halves of c requests, two or more left for the lower one
    constexpr int C = decltype(cc)::value;
    if constexpr (C <= KMAX - 2) {
      constexpr int N = br_few_below(KMAX - C + 1), FIRST = br_few_below(C), LAST = br_few_below(C + 1);
      constexpr int BLOCK = C == 1 ? 8 : 28;
      static_assert(C == 0 || ((LAST - FIRST) % BLOCK == 0 && (FIRST + 3) % 4 == 0), "whole blocks of aligned pairs");
      int v[REGS];
#pragma unroll
      for (int r = 0; r < REGS; ++r) v[r] = (r + 1) * BR_WAVE <= N || r * BR_WAVE + lane < N ? low[r] : 0;  // (beyond: the empty subset)
      if constexpr (C == 0) {
        const int h = upper[0];
#pragma unroll
        for (int r = 0; r * BR_WAVE < N; ++r) take(h - v[r], h - v[r]);
      } else {
#pragma unroll 1
        for (int i = FIRST; i < LAST; i += BLOCK) {
          int h[BLOCK];
#pragma unroll
          for (int k = 0; k < BLOCK; k += 2) {
            const int2 two = *reinterpret_cast<const int2 *>(upper + i + k);
            h[k] = two.x, h[k + 1] = two.y;
          }
#pragma unroll
          for (int k = 0; k < BLOCK; k += 2)
#pragma unroll
            for (int r = 0; r * BR_WAVE < N; ++r) take(h[k] - v[r], h[k + 1] - v[r]);
        }
      }
    }
  };
  section(std::integral_constant<int, 0>{});
  section(std::integral_constant<int, 1>{});
  section(std::integral_constant<int, 2>{});
  section(std::integral_constant<int, 3>{});
  {  // one left
    constexpr int FIRST = br_few_below(KMAX - 1), N = br_few_below(KMAX) - FIRST, TURNS = (N + 6) / 7;
    static_assert(TURNS % 2 == 0, "in pairs");
    const int part = min((lane * 57) >> 9, 6), v = lower[min(lane - 9 * part, 8)];  // lane / 9, its remainder
#pragma unroll
    for (int i = 0; i < TURNS; i += 2)
      take(upper[FIRST + min(7 * i + part, N - 1)] - v, upper[FIRST + min(7 * i + 7 + part, N - 1)] - v);
  }
  {  // none left
    constexpr int FIRST = br_few_below(KMAX), N = br_few_below(KMAX + 1) - FIRST;
    take(upper[FIRST + min(lane, N - 1)], upper[FIRST + min(BR_WAVE + lane, N - 1)]);
  }
}

__device__ __forceinline__ void br_subset_few(int G, int m, int wl, int w, int kmax, int room, int lane, int *tab,
                                              int &bestkey, unsigned &bestmask) {
  bestkey = BR_KEY_NONE, bestmask = 0u;
  if (room < 0) return;
  br_stay(lane);
  const unsigned place = br_few_places.v[lane];
  int lo[4], hi[4];
  br_half_sums(wl, w, BR_FEW_ABSENT, lane, lo, hi);
  int *lower = tab, *upper = tab + 256 + 3;
#pragma unroll
  for (int u = 0; u < 4; ++u) lower[(place >> (8 * u)) & 255u] = min(lo[u], BR_FEW_ABSENT) << 8;
  const int pl = __builtin_popcount(lane);
  constexpr int pu[4] = {0, 1, 1, 2};
  unsigned mask = 0xffffffffu;
  for (int T = br_uniform(min(min(m, room), 1 << 20)), turn = 0;; ++turn) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      upper[(place >> (8 * u)) & 255u] =
          (int)(((unsigned)(T - min(hi[u], BR_FEW_ABSENT)) << 8 | (unsigned)(u * BR_WAVE + lane)) ^ 0x80000000u);
    br_wave_sync();
    int dn = INT32_MAX, dx = INT32_MIN;
    if (kmax == 3)
      br_few_walk<3>(lower, upper, lane, dn, dx);
    else if (kmax == 4)
      br_few_walk<4>(lower, upper, lane, dn, dx);
    else
      br_few_walk<5>(lower, upper, lane, dn, dx);
    const int best = br_uniform(br_wave_min(dn)) ^ (int)0x80000000u;  // (at least the empty subset does not exceed T)
    const int A = T - (best >> 8), h = best & 255;
    int FA = bestkey, FB = BR_KEY_NONE, B = 0;
    if (turn == 0) {
      const int above = br_uniform(br_wave_max(dx)) ^ (int)0x80000000u;
      B = above < 0 ? T - (above >> 8) : INT32_MAX;
      FA = A > 0 ? br_score0(G, m, A) : BR_KEY_NONE;
      FB = B <= room && B < BR_FEW_ABSENT ? br_score0(G, m, min(B, BR_FEW_ABSENT)) : BR_KEY_NONE;
      bestkey = max(FA, FB);
    }
    br_wave_sync();  // the sums have been read before they are written again
    if (bestkey <= 0) return;  // (the starvation guard's case: no mask is asked for)
    if (FA == bestkey) {
      const int reg = h < 128 ? (h < 64 ? hi[0] : hi[1]) : (h < 192 ? hi[2] : hi[3]);
      const int rest = A - __builtin_amdgcn_readlane(reg, h & 63), left = kmax - __builtin_popcount(h) - pl;
      int low = 0;
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        const unsigned long long at = br_ballot(lo[u] == rest && pu[u] <= left);
        low = at != 0ull ? u * BR_WAVE + (int)__builtin_ctzll(at) : low;
      }
      mask = min(mask, (unsigned)(h << 8 | low));
    }
    if (FB != bestkey) break;
    T = B;
  }
  bestmask = mask;
}
