// BR-0, Stage 2: the best subset of a window of 9..16 requests with at most kmax of them, from the sums of its two halves.
//
// eq. (br0-Fscore) rises with the sum up to the margin and falls beyond it (G >= 2), so two sums decide: the largest one
// up to the margin and the smallest one above it.  The 256 sums of the eight longest requests are sorted once in
// registers and written to LDS as one ascending list per cardinality limit j (those of at most j requests).  Each lane
// takes four of the 256 subsets of the others and looks up, in the list of what the limit leaves, the neighbours of
// what the margin leaves: 9 steps of one LDS read each, all four side by side.  The mask is the lowest one that has
// the chosen sum: lowest upper byte, then lowest lower byte.
// About 600 instructions on one wave at any limit, no memory beyond LDS: 6300 cycles at kmax = 6, a chain of
// LDS and DPP latencies (sort 1700, lists 900, search 1300).  The list of masks (br_subset_list.h) has 14892 of them at
// kmax = 6 (15000 cycles on four waves) and needs the scan of all 65536 beyond half of the window.  Limits of 3 to 5 form every
// sum (br_subset_few.h).
#pragma once

#include "br_list.h"
#include "br_subset_list.h"

#define BR_HALVES_LISTED 1279             // entries of the lists: C(8, <= j) for j = 1..8
#define BR_HALVES_WORDS (BR_HALVES_LISTED + BR_WAVE)  // LDS words
#define BR_HALVES_ABSENT (1 << 22)        // length of a request the window does not hold: above every sum that counts

// start << 16 | length of the list of at most j requests (j = 0: the empty subset, the first entry of any list)
struct BrHalvesLists {
  int v[16];
};
constexpr BrHalvesLists br_make_halves_lists() {
  BrHalvesLists t{};
  t.v[0] = 1;
  int c = 1, n = 1, off = 0;
  for (int j = 1; j <= 8; ++j) {
    c = c * (9 - j) / j;
    n += c;
    t.v[j] = off << 16 | n;
    off += n;
  }
  return t;
}
static __device__ constexpr BrHalvesLists br_halves_lists = br_make_halves_lists();

template <bool STAY>
__device__ __forceinline__ void br_subset_halves(int G, int m, int wl, int w, int kmax, int room, int lane, int *tab,
                                                 int &bestkey, unsigned &bestmask) {
  if constexpr (STAY) br_stay(lane);
  const int lists = br_halves_lists.v[lane & 15];
  int lo[4], hi[4];
  br_half_sums(wl, w, BR_HALVES_ABSENT, lane, lo, hi);
  const int pl = __builtin_popcount(lane);
  constexpr int pu[4] = {0, 1, 1, 2};

  unsigned x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) x[u] = (unsigned)(BR_HALVES_ABSENT - 1 - lo[u]) << 8 | (unsigned)(u * BR_WAVE + lane);
  br_list_sort<4>(x, lane);
  int sum[4], bits[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sum[j] = BR_HALVES_ABSENT - 1 - (int)(x[j] >> 8);
    bits[j] = __builtin_popcount(x[j] & 255u);
  }
  // places in the lists: one byte per limit j = 1..8 counts the lane's entries of at most j requests (the exclusive prefix
  // over the lanes stays below 256)
  unsigned own0 = 0u, own1 = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    own0 += bits[i] > 4 ? 0u : 0x01010101u << (8 * max(bits[i] - 1, 0));
    own1 += bits[i] < 5 ? 0x01010101u : 0x01010101u << (8 * (bits[i] - 5));
  }
  const unsigned pre0 = (unsigned)br_scan_sum((int)own0) - own0, pre1 = (unsigned)br_scan_sum((int)own1) - own1;
  const int spare = BR_HALVES_LISTED + lane;  // entries a list does not take are written here
#pragma unroll
  for (int j = 1; j <= 8; ++j) {
    if (j > kmax) break;
    int at = (br_halves_lists.v[j] >> 16) + (int)((j <= 4 ? pre0 >> (8 * (j - 1)) : pre1 >> (8 * (j - 5))) & 0xffu);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = bits[i] <= j;
      tab[in ? at : spare] = sum[i];
      at += in ? 1 : 0;
    }
  }
  br_wave_sync();

  const int T = min(m, room);
  int t[4], n[4], base[4], pos[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = kmax - pl - pu[u];
    const int l = __builtin_amdgcn_ds_bpermute(min(max(j, 0), 8) << 2, lists);
    n[u] = l & 0xffff, base[u] = (l >> 16) - 1;
    t[u] = j >= 0 ? T - hi[u] : INT32_MIN;
    pos[u] = t[u] >= 0 ? 1 : 0;
  }
#pragma unroll
  for (int step = 128; step >= 1; step >>= 1) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(pos[u] + step, n[u]);
      pos[u] = tab[base[u] + i] <= t[u] ? i : pos[u];
    }
  }
  int below[4], above[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    below[u] = hi[u] + tab[base[u] + max(pos[u], 1)];
    above[u] = hi[u] + tab[base[u] + min(pos[u] + 1, n[u])];
    below[u] = t[u] >= 0 ? below[u] : 0;
    above[u] = t[u] != INT32_MIN && pos[u] < n[u] ? above[u] : INT32_MAX;
  }
  const int A = br_wave_max(max(max(below[0], below[1]), max(below[2], below[3])));
  const int B = br_wave_min(min(min(above[0], above[1]), min(above[2], above[3])));
  // the lowest mask of a sum that `cand` holds
  auto mask_of = [&](const int(&cand)[4], int s) -> unsigned {
    int h = 0, rest = 0, left = 0;
    bool found = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned long long at = br_ballot(cand[u] == s);
      if (!found && at != 0ull) {
        const int l = (int)__builtin_ctzll(at);
        h = u * BR_WAVE + l;
        rest = s - __builtin_amdgcn_readlane(hi[u], l);
        found = true;
      }
    }
    left = kmax - __builtin_popcount(h);
    int low = 0;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const unsigned long long at = br_ballot(lo[u] == rest && pl + pu[u] <= left);
      low = at != 0ull ? u * BR_WAVE + (int)__builtin_ctzll(at) : low;
    }
    return (unsigned)(h << 8 | low);
  };
  const int FA = A > 0 ? br_score0(G, m, A) : BR_KEY_NONE;
  const int FB = B <= room && B < BR_HALVES_ABSENT ? br_score0(G, m, min(B, BR_HALVES_ABSENT)) : BR_KEY_NONE;
  bestkey = max(FA, FB);
  unsigned mask = 0xffffffffu;
  if (FA == bestkey) mask = mask_of(below, A);
  if (FB == bestkey) mask = min(mask, mask_of(above, B));
  bestmask = bestkey == BR_KEY_NONE ? 0u : mask;
  br_wave_sync();  // the lists have been read before a later search rewrites them
}
