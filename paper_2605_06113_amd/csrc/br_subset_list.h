// Stage-2 subsets of a window of 9..16 requests when a subset may hold at most half of them: the admissible subsets
// are enumerated themselves, from a constant list of the 16-bit masks of up to eight bits, ordered by (number of bits, value).
//
// Stage 2 runs where free slots are scarce, so the limit kmax = min(free slots of the worker, R_max) is usually a few:
// of the 65535 masks of a window of 16, 696 have at most three bits.  Those need neither masks nor tables
// (br_small_search); BR-0 forms every sum at limits of 3 to 5 (br_subset_few.h) and decides by the sums of the window's
// halves beyond (br_subset_halves.h), so the list serves BR-H and short walks.  Within one bit count the masks below 2^w are the
// first C(w, c) of their section, so any window width reads a dense piece of the list.  A mask's sum is two reads of
// tables over its lower and upper byte that the wave builds per pop (256 words each, in LDS).  About 16 instructions
// per 64 masks against 11 of the scan over all masks (br_bigr_scan), which therefore stays for kmax > w / 2 (at 8 of 16
// the list still holds 39202 masks).
// 1024 clusters, G = 16, window 16, 46 admissions in 19 pops each, whole pass: 505 us with the scan, 142 with the list
// alone, 75 with the searches named above, 60 with sums of three to five requests formed (br_subset_few.h), 57 since a pop reads the
// window from LDS once: what it looks up of it (smallest entry, sums, the requests it binds) waited for LDS each time.
#pragma once

#include "br_device.h"

#define BR_LIST_MASKS 39203  // masks of at most eight bits, the empty one among them (br_list_serves asks for no more)

// An entry holds the byte offsets of the two table reads, the upper byte's in the upper half: entries order as their
// masks do.  (157 KB; present in the code objects whose kernels search by it: br_assign_bigr and the br_assign_long ones.)
struct BrMaskList {
  unsigned v[BR_LIST_MASKS];
};

constexpr BrMaskList br_make_mask_list() {
  BrMaskList t{};
  int at[10] = {};
  int count = 1;  // C(16, c)
  for (int c = 0; c <= 8; ++c) {
    at[c + 1] = at[c] + count;
    count = count * (16 - c) / (c + 1);
  }
  for (int v = 0; v < 65536; ++v) {
    int b = v - ((v >> 1) & 0x5555);
    b = (b & 0x3333) + ((b >> 2) & 0x3333);
    b = (b + (b >> 4)) & 0x0f0f;
    b = (b + (b >> 8)) & 0x1f;
    if (b <= 8) t.v[at[b]++] = (unsigned)((256 + (v >> 8)) * 4) << 16 | (unsigned)((v & 255) * 4);
  }
  return t;
}

static __device__ constexpr BrMaskList br_mask_list = br_make_mask_list();
static_assert(br_mask_list.v[BR_LIST_MASKS - 1] == ((256u + 255u) * 4u << 16 | 0u), "eight bits: the largest mask is the last one");

__device__ __forceinline__ int br_list_mask(unsigned v) { return (int)(((v >> 18) - 256u) << 8 | (v & 0xffffu) >> 2); }

// Section sizes and their running sums: at[w][c] = C(w, c), upto[w][c] = sum of at[w][1..c] (c <= 8).
struct BrMaskCounts {
  int at[17][9], upto[17][9];
};

constexpr BrMaskCounts br_make_mask_counts() {
  BrMaskCounts t{};
  for (int w = 0; w <= 16; ++w) {
    int n = 1;
    for (int c = 0; c <= 8; ++c) {
      t.at[w][c] = n;
      t.upto[w][c] = c > 0 ? t.upto[w][c - 1] + n : 0;
      n = n * (w > c ? w - c : 0) / (c + 1);
    }
  }
  return t;
}

static __device__ constexpr BrMaskCounts br_mask_counts = br_make_mask_counts();

// Which of the two exact searches of a window of up to 16 requests: the list, or the scan over all masks (one trip
// up to a window of 8).
__device__ __forceinline__ bool br_list_serves(int w, int kmax) { return w > 8 && 2 * kmax <= w; }

// number of non-empty subsets of w requests with at most kmax of them (kmax <= 8)
__device__ __forceinline__ int br_list_size(int w, int kmax) { return br_mask_counts.upto[w][kmax]; }

// What a search computes from the lane alone (its tables' loads among it) stays in the search: taken out of the loop over the
// pops it holds registers throughout the round (BR-0, windows of up to 16, queues of up to 256: 220 of them, 153 so and with wider windows
// in a kernel of their own: three waves per SIMD instead of two; 3000 clusters, window 16, whole pass 143 -> 89 us).
__device__ __forceinline__ void br_stay(int &lane) { asm volatile("" : "+v"(lane)); }

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

// Sum of a window's entries from the lane's on, the w - lane smallest, for lanes below w; `wl`: the window, entry l on lane l (w <= 32).
__device__ __forceinline__ int br_rest_sums(int wl, int w, int lane) {
  const int s = lane < w ? wl >> BR_IDX_BITS : 0;
  int x = s;
  x += br_dpp<0x111>(0, x);       // row_shr:1
  x += br_dpp<0x112>(0, x);       // row_shr:2
  x += br_dpp<0x114>(0, x);       // row_shr:4
  x += br_dpp<0x118>(0, x);       // row_shr:8
  x += br_dpp<0x142, 0x2>(0, x);  // row_bcast:15 into row 1
  return __builtin_amdgcn_readlane(x, 31) - x + s;
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

// The same from br_rest_sums: lane w - c passes the sum of the c smallest entries.
__device__ __forceinline__ int br_useful_rest(int sum, float F, float slack, int room, int kmax, int w, int lane) {
  const float fewer = __int_as_float(br_dpp<0x130>(0, __float_as_int(F)));  // wave_shl:1
  const unsigned long long bal = br_ballot(lane < w - 1 && (F < fewer - slack || sum > room));
  return bal != 0ull ? min(kmax, w - 64 + (int)__builtin_clzll(bal)) : kmax;
}

// Sums of the window entries that the 256 values of a mask's lower (lo) and upper byte (hi) select, values lane, 64 +
// lane, ... per lane; `absent` stands for the entries beyond a window of fewer than 16 (w > 8).  wl: entry l on lane l < 16.
__device__ __forceinline__ void br_half_sums(int wl, int w, int absent, int lane, int (&lo)[4], int (&hi)[4]) {
  const int mine = lane < w ? wl >> BR_IDX_BITS : absent;
  auto length = [&](int b) { return __builtin_amdgcn_readlane(mine, b); };
  lo[0] = 0, hi[0] = 0;
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    lo[0] += (int)__umul24((lane >> b) & 1, length(b));
    hi[0] += (int)__umul24((lane >> b) & 1, length(8 + b));
  }
  const int l6 = length(6), l7 = length(7), h6 = length(14), h7 = length(15);
  lo[1] = lo[0] + l6, lo[2] = lo[0] + l7, lo[3] = lo[1] + l7;
  hi[1] = hi[0] + h6, hi[2] = hi[0] + h7, hi[3] = hi[1] + h7;
}

// The byte tables of a search: lower byte in tab[0..255], upper byte in tab[256..511].
__device__ __forceinline__ void br_list_tables(const int *win, int w, int *tab, int lane) {
  int lo[4], hi[4];
  br_half_sums(win[lane & 15], w, 0, lane, lo, hi);
#pragma unroll
  for (int u = 0; u < 4; ++u) tab[u * BR_WAVE + lane] = lo[u], tab[256 + u * BR_WAVE + lane] = hi[u];
}

// Takes four keys per lane into the best key and its lowest mask (both uniform); mask(u): the mask of a lane's u-th key.
// Keys that do not reach the best so far, nearly all of them, cost one maximum each and a ballot.
template <class Mask>
__device__ __forceinline__ void br_settle(const int (&key)[4], Mask mask, int &bk, int &bm) {
  const int t = max(max(key[0], key[1]), max(key[2], key[3]));
  if (br_ballot(t >= bk) == 0ull) return;
  const int km = br_wave_max(t);
  int v = INT32_MAX;
#pragma unroll
  for (int u = 0; u < 4; ++u) v = key[u] == km ? min(v, mask(u)) : v;
  v = br_wave_min(v);
  bm = km > bk && km != BR_KEY_NONE ? v : min(bm, v);
  bk = km;
}

// All triples of 16 requests, i > j > l, ordered by i: those of a window of w are the first C(w, 3).  An entry holds the
// three byte offsets 4i, 4j, 4l.
struct BrTriples {
  unsigned v[560];
};
constexpr BrTriples br_make_triples() {
  BrTriples t{};
  int n = 0;
  for (int i = 2; i < 16; ++i)
    for (int j = 1; j < i; ++j)
      for (int l = 0; l < j; ++l) t.v[n++] = (unsigned)(4 * i) << 16 | (unsigned)(4 * j) << 8 | (unsigned)(4 * l);
  return t;
}
static __device__ constexpr BrTriples br_triples = br_make_triples();

// The search at kmax <= 3, windows of up to 16: single requests, pairs and triples read the window itself, without tables.
// Lane (g, i) of 4 x 16 takes the pairs of i with 4g .. 4g + 3 (i with itself: the single request); triples come from
// a list, on its way meanwhile (TRIPLES: BR-H).  wl: entry lane & 15.  A search of up to 136 / 696 subsets took 2300 / 3500 cycles by tables
// and mask list.
template <bool TRIPLES, class Score>
__device__ __forceinline__ void br_small_search(int wl, const int *win, int w, int kmax, int room, int lane, Score score, int &bk, int &bm) {
  if constexpr (!TRIPLES) br_stay(lane);
  const int n3 = TRIPLES && kmax >= 3 ? br_mask_counts.at[w][3] : 0;
  unsigned e[3][4];
  if (n3 > 0) {
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) e[t][u] = br_triples.v[min((t * 4 + u) * BR_WAVE + lane, n3 - 1)];
  }
  auto length = [&](unsigned at) -> int {
    return *reinterpret_cast<const int *>(reinterpret_cast<const char *>(win) + at) >> BR_IDX_BITS;
  };
  int delta[4], key[4][4];
  const int i = lane & 15, j0 = (lane >> 4) * 4;
  {
    const int si = wl >> BR_IDX_BITS;
    int sj[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) sj[u] = win[j0 + u] >> BR_IDX_BITS;
#pragma unroll
    for (int u = 0; u < 4; ++u) delta[u] = si + (j0 + u == i ? 0 : sj[u]);
    score(delta, key[0]);
    const int jmax = kmax >= 2 ? w - 1 : i;  // pairs i <= j within the window
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = j0 + u >= i && j0 + u <= jmax && i < w && delta[u] <= room;
      key[0][u] = ok ? key[0][u] : BR_KEY_NONE;
    }
  }
  int best = max(max(key[0][0], key[0][1]), max(key[0][2], key[0][3]));
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t * 4 * BR_WAVE >= n3) break;
#pragma unroll
    for (int u = 0; u < 4; ++u) delta[u] = length(e[t][u] >> 16) + length((e[t][u] >> 8) & 0xffu) + length(e[t][u] & 0xffu);
    score(delta, key[t + 1]);
#pragma unroll
    for (int u = 0; u < 4; ++u) key[t + 1][u] = delta[u] <= room ? key[t + 1][u] : BR_KEY_NONE;
    best = max(best, max(max(key[t + 1][0], key[t + 1][1]), max(key[t + 1][2], key[t + 1][3])));
  }
  bk = br_wave_max(best);
  int v = INT32_MAX;
#pragma unroll
  for (int u = 0; u < 4; ++u) v = key[0][u] == bk ? min(v, 1 << i | 1 << (j0 + u)) : v;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t * 4 * BR_WAVE >= n3) break;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v = key[t + 1][u] == bk ? min(v, 1 << (e[t][u] >> 18) | 1 << ((e[t][u] >> 10) & 63u) | 1 << ((e[t][u] >> 2) & 63u)) : v;
  }
  bm = br_wave_min(v);
  if (bk == BR_KEY_NONE) bm = INT32_MAX;
}

// Walks the admissible subsets of the window (w > 8), four neighbours of the list per lane and trip, the next trip's on
// their way meanwhile; wave wv of nwv takes every nwv-th trip.  `build`: this wave makes the byte tables first (the first
// trip's entries are on their way).  score(delta[4], key[4]) gives the keys.  bk, bm (uniform): the best key and the
// lowest mask that has it.
// In a window of 16 the sections follow each other without a gap and are walked as one.  The last trip of a section
// takes its last four entries on the lanes beyond it, which changes no maximum.
template <class Score>
__device__ __forceinline__ void br_list_walk(const int *win, int *tab, int w, int kmax, int room, int lane, int wv, int nwv,
                                             bool build, Score score, int &bk, int &bm) {
  constexpr int TRIP = 4 * BR_WAVE;
  bk = BR_KEY_NONE, bm = INT32_MAX;
  int c = w == 16 ? kmax : 1, off = 1;
  int n = w == 16 ? br_list_size(16, kmax) : w;
  int i0 = wv * TRIP;
  auto fetch = [&](unsigned(&e)[4]) -> bool {  // this trip's entries; moves on to the next section where one is through
    while (i0 >= n) {
      if (c >= kmax) return false;
      off += br_mask_counts.at[16][c];
      ++c;
      n = br_mask_counts.at[w][c];
      i0 = wv * TRIP;
    }
    const unsigned *at = br_mask_list.v + off + min(i0 + 4 * lane, n - 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = at[u];
    i0 += nwv * TRIP;
    return true;
  };
  unsigned e[4] = {}, next[4] = {};
  bool more = fetch(e);
  if (build) {
    br_list_tables(win, w, tab, lane);
    br_wave_sync();
  }
  const bool check = room != INT32_MAX;
  while (more) {
    const bool another = fetch(next);
    int delta[4], key[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      delta[u] = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(tab) + (e[u] & 0xffffu)) +
                 *reinterpret_cast<const int *>(reinterpret_cast<const char *>(tab) + (e[u] >> 16));
    score(delta, key);
    if (check) {
#pragma unroll
      for (int u = 0; u < 4; ++u) key[u] = delta[u] <= room ? key[u] : BR_KEY_NONE;
    }
    br_settle(key, [&](int u) { return br_list_mask(e[u]); }, bk, bm);
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = next[u];
    more = another;
  }
  if (bk == BR_KEY_NONE) bm = INT32_MAX;
}
