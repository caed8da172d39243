// Decode steps on worker lists of up to 256 slots: LPL lanes hold a list of up to 4 * LPL slots, four consecutive slots each,
// so a wave holds 64 / LPL lists side by side.  Used by the decode kernel (br_k_advance_seg), by the waves that
// apply the decode steps to the lists of the cluster they have routed (br_advance_lists) and by the projection that applies them
// (br_project_lists).  PK as for br_adv_apply.
// A list is made dense again in LDS and goes back with 16-byte stores, whether or not it lost a request: one path without
// branches.  Bound by memory traffic, and before that by what a wave issues: storing word by word what had moved took
// eight masked stores of single words per list beside two of whole lines.  Kernel, us, before and now: 4096 clusters, G = 16,
// lists of 144 slots, 12 steps 28.8 and 22.6 (5.7 TB/s); 1531, G = 13, 101 slots, 3 steps 9.4 and 7.2; 1024, G = 16, 144 slots,
// 8 steps 10.3 and 7.9; 2048, G = 8, 64 slots with maintained estimates, one step 14.5 and 14.3.
#pragma once

#include <type_traits>

#include "br_device.h"

#define BR_SEG_LIST_WORDS 512   // LDS words of a wave: kv and remaining steps of 256 slots
#define BR_SEG_MAP_WORDS 128    // PK 1: and their new slots
#define BR_SEG_WORDS(PK) (BR_SEG_LIST_WORDS + ((PK) == 1 ? BR_SEG_MAP_WORDS : (PK) == 2 ? 768 : 0))

// The first of the lists a wave goes over (the same on every lane); what follows addresses a list by its 32-bit offset from
// there, which keeps 64-bit addresses per lane out of the registers.
struct BrSegBase {
  int32_t *kv, *rem, *L, *n;
  float *pred;
};
__device__ __forceinline__ BrSegBase br_seg_base(const BrParams &p, int64_t row0) {
  return BrSegBase{p.kv + row0 * p.Bs, p.rem + row0 * p.Bs, p.L + row0, p.n + row0, p.P ? p.pred + row0 * p.Bs * p.P : nullptr};
}
template <class T>
__device__ __forceinline__ T &br_seg_at(const void *base, unsigned bytes) {
  return *reinterpret_cast<T *>(reinterpret_cast<char *>(const_cast<void *>(base)) + bytes);
}

// Sums over the lanes of the lane's list up to and with it, two side by side, and the last lane's value on all of them.
template <int LPL>
__device__ __forceinline__ void br_seg_scans(int &x, int &y) {
  x += br_dpp<0x111>(0, x), y += br_dpp<0x111>(0, y);
  x += br_dpp<0x112>(0, x), y += br_dpp<0x112>(0, y);
  x += br_dpp<0x114>(0, x), y += br_dpp<0x114>(0, y);
  x += br_dpp<0x118>(0, x), y += br_dpp<0x118>(0, y);
  if constexpr (LPL >= 32) x += br_dpp<0x142, 0xA>(0, x), y += br_dpp<0x142, 0xA>(0, y);
  if constexpr (LPL == 64) x += br_dpp<0x143, 0xC>(0, x), y += br_dpp<0x143, 0xC>(0, y);
}
// Sums over the lanes of the list, on its last lane, N side by side.
template <int LPL, int N>
__device__ __forceinline__ void br_seg_sums(int (&x)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] += br_dpp<0x111>(0, x[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] += br_dpp<0x112>(0, x[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] += br_dpp<0x114>(0, x[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] += br_dpp<0x118>(0, x[k]);
  if constexpr (LPL >= 32) {
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] += br_dpp<0x142, 0xA>(0, x[k]);
  }
  if constexpr (LPL == 64) {
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] += br_dpp<0x143, 0xC>(0, x[k]);
  }
}
template <int LPL>
__device__ __forceinline__ int br_seg_last(int x, int lane) {
  if constexpr (LPL == 16) {
    return br_dpp<0x15F, 0xF, true>(0, x);  // row_newbcast:15
  } else {
    const int hi = __builtin_amdgcn_readlane(x, 63);
    return LPL == 64 ? hi : lane < 32 ? __builtin_amdgcn_readlane(x, 31) : hi;
  }
}

// The lane's four slots of its list.
template <int PK>
struct BrSegSlots {
  int4 kv4, rem4;
};
template <>
struct BrSegSlots<2> {
  int4 kv4, rem4;
  float ch[4], age[4], since[4];
};

// `list`: which one; `lim`: slots to fetch (0: no list on this lane); what lies beyond the list is ignored by br_seg_decide.
template <int LPL, int PK>
__device__ __forceinline__ void br_seg_load(const BrSegBase &b, int Bs, int list, int lim, int lane, BrSegSlots<PK> &v) {
  const int e0 = 4 * (lane & (LPL - 1));
  const unsigned at = 4u * (unsigned)(list * Bs + e0);
  v.kv4 = make_int4(0, 0, 0, 0), v.rem4 = make_int4(0, 0, 0, 0);
  if constexpr (PK == 2) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v.ch[k] = 0.0f, v.age[k] = 0.0f, v.since[k] = 0.0f;
  }
  if (e0 < lim) {
    v.kv4 = br_seg_at<int4>(b.kv, at);
    v.rem4 = br_seg_at<int4>(b.rem, at);
    if constexpr (PK == 2) br_rows3_load(&br_seg_at<float>(b.pred, 3u * at), v.ch, v.age, v.since);
  }
}

// What t decode steps do to the lane's list of n requests: its new length, the kv that left (complete on the last lane of the
// list), a new place for each slot (those who stay in order, then the others), and, PK 1, the first slot whose prediction row
// may move: that of the first leaver's lane (n: none).  `map` (PK 1): the new slots by lane * 4 + k, < 0 for one that left.
struct BrSegPlan {
  int to[4], kept, gone, from;
  bool any;  // (uniform, PK 1) some list of the wave lost a request
};

template <int LPL, int PK>
__device__ __forceinline__ void br_seg_decide(const BrParams &p, int t, int n, int lane, BrSegSlots<PK> &v, int *lds, short *map,
                                              BrSegPlan &d) {
  const int e0 = 4 * (lane & (LPL - 1));
  int kv[4] = {v.kv4.x, v.kv4.y, v.kv4.z, v.kv4.w}, rem[4] = {v.rem4.x, v.rem4.y, v.rem4.z, v.rem4.w};
  bool stay[4], leaves = false;
  int count = 0, lost = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bool used = e0 + k < n;
    stay[k] = used && rem[k] > t;
    leaves |= used && !stay[k];
    lost += used && !stay[k] ? kv[k] : 0;
    count += stay[k] ? 1 : 0;
    kv[k] += stay[k] ? t : 0;
    rem[k] -= stay[k] ? t : 0;
  }
  v.kv4 = make_int4(kv[0], kv[1], kv[2], kv[3]);
  v.rem4 = make_int4(rem[0], rem[1], rem[2], rem[3]);
  if constexpr (PK == 2) br_refresh_update4(p, t, stay, v.ch, v.age, v.since, lds, lane);
  int upto = count;
  br_seg_scans<LPL>(upto, lost);
  d.kept = br_seg_last<LPL>(upto, lane), d.gone = lost;
  int in = upto - count, out = d.kept + e0 - in;  // the next place of one who stays, of one who does not
  short to[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    d.to[k] = stay[k] ? in : out;
    if constexpr (PK == 1) to[k] = (short)(stay[k] ? in : -1);
    in += stay[k] ? 1 : 0;
    out += stay[k] ? 0 : 1;
  }
  if constexpr (PK == 1) {
    *reinterpret_cast<short4 *>(map + 4 * lane) = make_short4(to[0], to[1], to[2], to[3]);
    const unsigned long long bl = br_ballot(leaves);
    d.any = bl != 0ull;
    d.from = n;
    if constexpr (LPL == 64) {
      if (bl != 0ull) d.from = 4 * (int)__builtin_ctzll(bl);
    } else {
      unsigned mine = lane < 32 ? (unsigned)bl : (unsigned)(bl >> 32);
      if constexpr (LPL == 16) mine = (mine >> (lane & 16)) & 0xffffu;
      if (mine != 0u) d.from = 4 * __builtin_ctz(mine);
    }
  }
}

// The list as the plan leaves it.  lds: BR_SEG_WORDS(PK) less the map.
template <int LPL, int PK>
__device__ __forceinline__ void br_seg_store(const BrSegBase &b, int Bs, int list, int lane, const BrSegSlots<PK> &v,
                                             const BrSegPlan &d, int *lds) {
  const int lseg = lane & (LPL - 1), e0 = 4 * lseg;
  const int kv[4] = {v.kv4.x, v.kv4.y, v.kv4.z, v.kv4.w}, rem[4] = {v.rem4.x, v.rem4.y, v.rem4.z, v.rem4.w};
  int *mine = lds + 4 * (lane - lseg);
  float *rows = reinterpret_cast<float *>(lds + BR_SEG_LIST_WORDS);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    mine[d.to[k]] = kv[k], mine[d.to[k] + 256] = rem[k];
    if constexpr (PK == 2) {
      float *q = rows + 3 * (4 * (lane - lseg) + d.to[k]);
      q[0] = v.ch[k], q[1] = v.age[k], q[2] = v.since[k];
    }
  }
  br_wave_sync();
  if (e0 < d.kept) {
    const unsigned at = 4u * (unsigned)(list * Bs + e0);
    br_seg_at<int4>(b.kv, at) = *reinterpret_cast<const int4 *>(lds + 4 * lane);
    br_seg_at<int4>(b.rem, at) = *reinterpret_cast<const int4 *>(lds + 4 * lane + 256);
    if constexpr (PK == 2) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        br_seg_at<float4>(b.pred, 3u * at + 16u * c) = *reinterpret_cast<const float4 *>(rows + 12 * lane + 4 * c);
    }
  }
}

// Its load and its length.
template <int LPL>
__device__ __forceinline__ void br_seg_worker(const BrSegBase &b, int t, int list, bool ok, int L, int lane, const BrSegPlan &d) {
  if (ok && (lane & (LPL - 1)) == LPL - 1) {
    br_seg_at<int>(b.L, 4u * (unsigned)list) = L + d.kept * t - d.gone;  // survivors gain t tokens each
    br_seg_at<int>(b.n, 4u * (unsigned)list) = d.kept;
  }
}

// Prediction rows (PK 1) of the lists of a wave, from slot `from` of each on (from >= n: nothing moves), to the slots of
// `map`: the lanes of a list walk its rows as contiguous memory, a unit V at a time (UPR units per row; 0: as many as P says),
// four requested (br_seg_rows_ask) before the first is stored (br_seg_rows_place, which goes on with the rest of longer rows).
// Destinations lie at or below their sources, so no store reaches a source not yet read.
template <int LPL, class V>
__device__ __forceinline__ void br_seg_rows_fetch(const float *pred, unsigned first, int x, int end, V (&v)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k)  // (beyond the list: its last unit again, without a branch)
    v[k] = br_seg_at<V>(pred, first + (unsigned)sizeof(V) * (unsigned)min(x + k * LPL, max(end - 1, 0)));
}

template <int LPL, int UPR, class V>
__device__ __forceinline__ void br_seg_rows_ask(const float *pred, int Bs, int P, int list, int from, int n, int lane, V (&v)[4]) {
  const int upr = UPR > 0 ? UPR : P / (int)(sizeof(V) / sizeof(float));
  br_seg_rows_fetch<LPL>(pred, 4u * (unsigned)(list * Bs * P), from * upr + (lane & (LPL - 1)), n * upr, v);
}

template <int LPL, int UPR, class V>
__device__ __forceinline__ void br_seg_rows_place(float *pred, int Bs, int P, int list, int from, int n, const short *map, int lane,
                                                  V (&v)[4]) {
  const int upr = UPR > 0 ? UPR : P / (int)(sizeof(V) / sizeof(float));
  const unsigned inv = 65536u / (unsigned)upr + 1u;  // x / upr for x < 2048 by multiplication
  const unsigned first = 4u * (unsigned)(list * Bs * P);
  const short *mine = map + (lane & ~(LPL - 1)) * 4;
  const int end = n * upr;
  for (int x = from * upr + (lane & (LPL - 1)); br_ballot(x < end) != 0ull;) {
    int slot[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int y = min(x + k * LPL, end);
      slot[k] = mine[min(UPR == 1 ? y : (int)(((unsigned)y * inv) >> 16), 4 * LPL - 1)];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int y = x + k * LPL, j = UPR == 1 ? y : (int)(((unsigned)y * inv) >> 16);
      if (y < end && slot[k] >= 0 && slot[k] != j)
        br_seg_at<V>(pred, first + (unsigned)sizeof(V) * (unsigned)(slot[k] * upr + (y - j * upr))) = v[k];
    }
    x += 4 * LPL;
    if (UPR == 1 || br_ballot(x < end) == 0ull) break;
    br_seg_rows_fetch<LPL>(pred, first, x, end, v);
  }
}

// calls body(unit, units per row) with the unit that rows of P floats are moved in
typedef float br_float2 __attribute__((ext_vector_type(2)));
typedef float br_float4 __attribute__((ext_vector_type(4)));
template <class F>
__device__ __forceinline__ void br_with_row_unit(int P, F &&body) {
  if (P == 4)
    body(br_float4{}, std::integral_constant<int, 1>{});
  else if (P == 8)
    body(br_float4{}, std::integral_constant<int, 2>{});
  else if (P == 1)
    body(float{}, std::integral_constant<int, 1>{});
  else if ((P & 1) == 0)
    body(br_float2{}, std::integral_constant<int, 0>{});
  else
    body(float{}, std::integral_constant<int, 0>{});
}

// The decode steps of one cluster whose lists (of up to 4 * LPL slots, rows of UPR units V) are this wave's: lane g holds load
// and length of worker g.  What a wave alone moves per unit of time is what it has in flight over the memory's latency, and a
// wait for a load waits for the stores before it too, so RW groups of lists are loaded, decided and stored at a time, with as
// few waits as that takes: one where the rows are requested together with the slots, which is done while every list
// loses requests (`ahead`), else two.  Groups of lists that lose nothing have no rows to wait for (4096 clusters, G = 32, B = 96,
// H = 4, one step, lightly loaded: whole pass 98.1 us with that wait, 96.0 so); not with one list to a group, where the
// requests of two lists would no longer be on their way together (40 steps, B = 144: 221 us, 214 without).
// lds: RW * BR_SEG_WORDS(1) words of the wave's.
template <int LPL, int RW, int UPR, class V>
__device__ __forceinline__ void br_advance_lists(const BrParams &p, int t, int inst, int lane, int Lcur, int nn, int *lds) {
  constexpr int LPW = BR_WAVE / LPL;
  constexpr bool SKIP = LPL < BR_WAVE;
  const BrSegBase b = br_seg_base(p, (int64_t)br_uniform(inst) * p.G);
  auto batch = [&](int g0, auto ahead) -> bool {
    constexpr bool AHEAD = decltype(ahead)::value;
    BrSegSlots<1> v[RW];
    V q[RW][4];
    BrSegPlan d[RW];
    int n[RW], list[RW];
    bool ok[RW], all = true;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int g = g0 + r * LPW + lane / LPL;
      ok[r] = g < p.G;
      list[r] = ok[r] ? g : 0;
      n[r] = __builtin_amdgcn_ds_bpermute(list[r] << 2, nn);
      n[r] = ok[r] ? n[r] : 0;
      br_seg_load<LPL, 1>(b, p.Bs, list[r], n[r], lane, v[r]);
    }
    if constexpr (AHEAD) {
#pragma unroll
      for (int r = 0; r < RW; ++r) br_seg_rows_ask<LPL, UPR, V>(b.pred, p.Bs, p.P, list[r], 0, n[r], lane, q[r]);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      int *words = lds + r * BR_SEG_WORDS(1);
      br_seg_decide<LPL, 1>(p, t, n[r], lane, v[r], words, reinterpret_cast<short *>(words + BR_SEG_LIST_WORDS), d[r]);
      all = all && (d[r].kept < n[r] || n[r] == 0);
      if constexpr (AHEAD)
        d[r].from = 0;
      else if (!SKIP || d[r].any)
        br_seg_rows_ask<LPL, UPR, V>(b.pred, p.Bs, p.P, list[r], d[r].from, n[r], lane, q[r]);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int L = __builtin_amdgcn_ds_bpermute(list[r] << 2, Lcur);
      br_seg_store<LPL, 1>(b, p.Bs, list[r], lane, v[r], d[r], lds + r * BR_SEG_WORDS(1));
      br_seg_worker<LPL>(b, t, list[r], ok[r], L, lane, d[r]);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r)
      if (AHEAD || !SKIP || d[r].any)
        br_seg_rows_place<LPL, UPR, V>(b.pred, p.Bs, p.P, list[r], d[r].from, n[r],
                                       reinterpret_cast<const short *>(lds + r * BR_SEG_WORDS(1) + BR_SEG_LIST_WORDS), lane, q[r]);
    br_wave_sync();  // the words are rewritten by the next lists
    return br_ballot(!all) == 0ull;
  };
  bool ahead = false;
  for (int g0 = 0; g0 < p.G; g0 += RW * LPW)
    ahead = ahead ? batch(g0, std::true_type{}) : batch(g0, std::false_type{});
}

// The same for lists without prediction rows (BR-0; 4096 clusters, G = 16, B = 144, overloaded, a step per call: whole pass 46.9 us
// with lists one by one through masked single-word stores, 41.5 so; 48 steps and 250 admissions 111.5 and 105.9), workers [g0, g1): `done` gets each list's worker, plan and the lane that
// holds both whole.  lds: two turns of BR_SEG_WORDS(0) of the wave's.
template <int LPL, int RW, class F>
__device__ __forceinline__ void br_advance_lists_plain(const BrParams &p, int t, const BrSegBase &b, int lane, int g0, int g1,
                                                       int nn, int *lds, F &&done) {
  constexpr int LPW = BR_WAVE / LPL;
  // a list per wave, four at a time: number and length of the list are the wave's, not the lanes' (one cluster, G = 64, lists of 144
  // slots: whole pass 28.3 us, 29.0 without; eight at a time the kernel would get by with five waves per SIMD instead of four,
  // which batches of several times that size are slower with: 8192 clusters 94.1 us, 91.8 without)
  constexpr bool WHOLE = LPL == BR_WAVE && RW <= 4;
  for (; g0 < g1; g0 += RW * LPW) {
    BrSegSlots<0> v[RW];
    int n[RW], list[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int g = g0 + r * LPW + (WHOLE ? 0 : lane / LPL);
      list[r] = min(g, g1 - 1);
      n[r] = WHOLE ? __builtin_amdgcn_readlane(nn, list[r]) : __builtin_amdgcn_ds_bpermute(list[r] << 2, nn);
      n[r] = g < g1 ? n[r] : 0;
      br_seg_load<LPL, 0>(b, p.Bs, list[r], n[r], lane, v[r]);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      int *words = lds + (r & 1) * BR_SEG_WORDS(0);
      BrSegPlan d;
      br_seg_decide<LPL, 0>(p, t, n[r], lane, v[r], words, nullptr, d);
      br_seg_store<LPL, 0>(b, p.Bs, list[r], lane, v[r], d, words);
      done(list[r], d, g0 + r * LPW + lane / LPL < g1 && (lane & (LPL - 1)) == LPL - 1);
    }
    br_wave_sync();
  }
}
// LONG: lists beyond 128 slots taken at a time: 8 for what one cluster alone takes, 4 where the registers that eight hold (some
// 20) would cost waves that a batch needs (br_k_route_split, br_k_route).
template <int LONG, class F>
__device__ __forceinline__ void br_advance_lists_any(const BrParams &p, int t, const BrSegBase &b, int lane, int g0, int g1, int nn,
                                                     int *lds, F &&done) {
  if (p.Bs <= 64)
    br_advance_lists_plain<16, 2>(p, t, b, lane, g0, g1, nn, lds, done);
  else if (p.Bs <= 128)
    br_advance_lists_plain<32, 4>(p, t, b, lane, g0, g1, nn, lds, done);
  else if (LONG <= 4 || g1 - g0 <= 4)
    br_advance_lists_plain<64, 4>(p, t, b, lane, g0, g1, nn, lds, done);
  else
    br_advance_lists_plain<64, LONG>(p, t, b, lane, g0, g1, nn, lds, done);
}
