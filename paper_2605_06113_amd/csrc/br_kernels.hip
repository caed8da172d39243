// gfx950 kernels of the BalanceRoute route step, except the sequential assignment
// (br_assign_kernel.h): state initialisation, decode step, horizon projection, and the
// F-score matrix with its stage-one reductions.
#include "br.h"
#include "br_device.h"
#include "br_advance_seg.h"
#include "br_launch.h"
#include "br_project.h"
#include "br_score_wave.h"

// ------------------------------------------------------------------ initialisation

__global__ void br_k_clear(BrParams p, int *pol) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t rows = (int64_t)p.N * p.G;
  if (tid < rows) {
    p.L[tid] = 0;
    p.n[tid] = 0;
  }
  if (tid < p.N) {
    p.qlen[tid] = 0;
    pol[2 * tid] = 0;
    pol[2 * tid + 1] = 0;
  }
}

// One wave per (cluster, worker): copy the caller's dense active list into the workspace
// layout and derive L_g = sum of kv (Sec. 2.2).
__global__ __launch_bounds__(256) void br_k_load_init(BrParams p, const int32_t *n_in, const int32_t *kv_in,
                                                     const int32_t *rem_in, const float *pred_in) {
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= (int64_t)p.N * p.G) return;  // whole wave leaves together
  const int lane = br_lane();
  int n_g = n_in[row];
  n_g = min(max(n_g, 0), p.B);
  int acc = 0;
  for (int j = lane; j < n_g; j += BR_WAVE) {
    const int kv = kv_in[row * p.B + j];
    p.kv[row * p.Bs + j] = kv;
    p.rem[row * p.Bs + j] = max(rem_in[row * p.B + j], 1);
    for (int q = 0; q < p.P; ++q) p.pred[(row * p.Bs + j) * p.P + q] = pred_in[(row * p.B + j) * p.P + q];
    acc += kv;
  }
  const int tot = br_wave_sum(acc);
  if (lane == 0) {
    p.L[row] = tot;
    p.n[row] = n_g;
  }
}

// ------------------------------------------------------------------ decode step
// Sec. 2.2: each active request advances one decode iteration per step: its KV length and
// the load of its worker grow by one token; after its last step it leaves and its whole KV
// footprint goes with it.  t steps are applied in closed form: a request with rem <= t
// leaves (net load change -kv), the others gain t tokens.  Dense lists are compacted
// in place, order preserved (writes never run ahead of reads).  PK as for br_adv_apply.

// Lists of up to 4 * LPL slots (LPL = 16, 32, 64): RW x 64 / LPL lists per wave, everything requested before the first
// result is needed.  Short lists side by side keep the lanes busy and their chains (the list, the rows that move, the
// estimator's look-ups) in step: lists of 64 slots with maintained estimates (2048 clusters, G = 8) 36 -> 14.5 us, of
// 96 with hazards (4096 clusters, G = 32, 40 steps) 113 -> 93 us, against one list per wave.
template <int LPL, int RW, int PK>
__global__ __launch_bounds__(256) void br_k_advance_seg(BrParams p, int t) {
  constexpr int LPW = BR_WAVE / LPL;  // lists of a wave side by side
  const int wave = br_uniform((int)(threadIdx.x >> 6));
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * (RW * LPW);
  const int64_t rows = (int64_t)p.N * p.G;
  if (row0 >= rows) return;
  const int lane = br_lane(), lists = (int)min(rows - row0, (int64_t)(RW * LPW));
  const BrSegBase b = br_seg_base(p, row0);
  __shared__ __align__(16) int lds_all[4 * BR_SEG_WORDS(PK)];
  int *lds = lds_all + wave * BR_SEG_WORDS(PK);
  int n_g[RW], L_g[RW];
  BrSegSlots<PK> v[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int at = r * LPW + lane / LPL, list = min(at, lists - 1);
    const bool ok = at < lists;
    n_g[r] = ok ? br_seg_at<int>(b.n, 4u * (unsigned)list) : 0;
    L_g[r] = ok ? br_seg_at<int>(b.L, 4u * (unsigned)list) : 0;
    br_seg_load<LPL, PK>(b, p.Bs, list, ok ? p.Bs : 0, lane, v[r]);
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int at = r * LPW + lane / LPL, list = min(at, lists - 1);
    const bool ok = at < lists;
    short *map = reinterpret_cast<short *>(lds + BR_SEG_LIST_WORDS);
    BrSegPlan d;
    br_seg_decide<LPL, PK>(p, t, n_g[r], lane, v[r], lds, map, d);
    if (PK == 1 && d.any) {
      br_with_row_unit(p.P, [&](auto unit, auto upr) {  // the rows are requested before anything is stored
        using V = decltype(unit);
        V q[4];
        br_seg_rows_ask<LPL, decltype(upr)::value, V>(b.pred, p.Bs, p.P, list, d.from, n_g[r], lane, q);
        br_seg_store<LPL, PK>(b, p.Bs, list, lane, v[r], d, lds);
        br_seg_rows_place<LPL, decltype(upr)::value, V>(b.pred, p.Bs, p.P, list, d.from, n_g[r], map, lane, q);
      });
    } else {
      br_seg_store<LPL, PK>(b, p.Bs, list, lane, v[r], d, lds);
    }
    br_seg_worker<LPL>(b, t, list, ok, L_g[r], lane, d);
    br_wave_sync();  // the words are rewritten by the next lists
  }
}

// Lists of more than 256 slots: one wave per list (RW of them), NC chunks of 256 slots, four slots per lane.
template <int NC, int RW, int PK>
__global__ __launch_bounds__(256) void br_k_advance(BrParams p, int t) {
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * RW;
  const int64_t rows = (int64_t)p.N * p.G;
  if (row0 >= rows) return;
  const int lane = br_lane();
  __shared__ __align__(16) int lds_all[PK > 0 ? 4 * 256 : 4];
  short *map = PK > 0 ? reinterpret_cast<short *>(lds_all + (threadIdx.x >> 6) * 256) : nullptr;
  int n_g[RW];
  int4 kv[RW][NC], rem[RW][NC];
#pragma unroll
  for (int r = 0; r < RW; ++r) n_g[r] = row0 + r < rows ? p.n[row0 + r] : 0;
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int64_t base = (row0 + r) * p.Bs;
#pragma unroll
    for (int c = 0; c < NC; ++c) br_adv_load(p.kv + base, p.rem + base, c * 256 + 4 * lane, row0 + r < rows ? p.Bs : 0, kv[r][c], rem[r][c]);
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    if (row0 + r >= rows) break;
    const int64_t base = (row0 + r) * p.Bs;
    int kept = 0, gone = 0;  // uniform
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (c * 256 < n_g[r]) {
        int from;
        br_adv_apply<PK>(p, t, c * 256 + 4 * lane, n_g[r], c * 256, kv[r][c], rem[r][c], p.kv + base, p.rem + base,
                           PK > 0 ? p.pred + base * p.P : nullptr, kept, gone, map, from);
        if (PK == 1 && from >= 0) {
          br_wave_sync();
          br_rows_move(p.pred + base * p.P, p.P, map, c * 256, from, min(n_g[r], c * 256 + 256), lane);
          br_wave_sync();  // the map is rewritten by the next chunk
        }
      }
    }
    if (lane == 0) {
      p.L[row0 + r] += kept * t - gone;  // survivors gain t tokens each
      p.n[row0 + r] = kept;
    }
  }
}
// The kernel is VALU-bound before it is HBM-bound (rocprofv3: ~500 vector instructions per wave with every
// loop written for 8 offsets and run-time widths), so HB, EXACT and PK (br_project.h) are compile-time.  Per offset the kv
// part is summed in a register and over the wave, the count comes from a ballot.
template <int NC, int RW, int HB, bool EXACT, int PK>
__global__ __launch_bounds__(256) void br_k_project_rows(BrParams p) {
  constexpr bool HAZ = PK == 0;
  if constexpr (PK == 1) {
    if (p.pred_mode == 2 && blockIdx.x == gridDim.x - 1) {  // a last block: the estimate at age 0, for this round's admissions
      if (threadIdx.x < BR_WAVE) {
        const float c = br_survival(p, 0);
        if (threadIdx.x == 0) *p.c0 = c;
      }
      return;
    }
  }
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * RW;
  const int64_t rows = (int64_t)p.N * p.G;
  if (row0 >= rows) return;
  const int lane = br_lane();
  const int H1 = p.H + 1;
  int n_g[RW], kv[RW][NC];
  float pr[RW][NC][BR_ROW_FLOATS(HB, PK)];
#pragma unroll
  for (int r = 0; r < RW; ++r) n_g[r] = row0 + r < rows ? p.n[row0 + r] : 0;
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int64_t base = (row0 + r) * p.Bs;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = c * BR_WAVE + lane;
      const bool used = j < n_g[r];
      kv[r][c] = used ? p.kv[base + j] : 0;
      const float *src = p.pred + (base + j) * p.P;
      if constexpr (PK == 2) {
        const float2 v = used ? *reinterpret_cast<const float2 *>(src) : make_float2(0.0f, 0.0f);
        pr[r][c][0] = v.x, pr[r][c][1] = v.y;
      } else if constexpr (!HAZ) {
        pr[r][c][0] = used ? src[0] : 0.0f;
      } else if constexpr (EXACT) {  // rows of HB floats: 16-byte loads
#pragma unroll
        for (int q = 0; q < HB; q += 4) {
          const float4 v = used ? *reinterpret_cast<const float4 *>(src + q) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          pr[r][c][q] = v.x, pr[r][c][q + 1] = v.y, pr[r][c][q + 2] = v.z, pr[r][c][q + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int q = 0; q < HB; ++q) pr[r][c][q] = (used && q < p.H) ? src[q] : 0.0f;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    if (row0 + r >= rows) break;
    int acc[HB + 1], cnt[HB + 1];
#pragma unroll
    for (int h = 0; h <= HB; ++h) acc[h] = 0, cnt[h] = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = c * BR_WAVE + lane;
      const int hm = j < n_g[r] ? br_last_offset<HB, EXACT, PK>(p, pr[r][c]) : -1;
#pragma unroll
      for (int h = 0; h <= HB; ++h) {
        if (EXACT || h <= p.H) {
          const bool in = h <= hm;
          acc[h] += in ? kv[r][c] : 0;
          cnt[h] += __builtin_popcountll(br_ballot(in));
        }
      }
    }
#pragma unroll
    for (int h = 0; h <= HB; ++h) {
      if (EXACT || h <= p.H) {
        const int v = br_wave_sum(acc[h]) + h * cnt[h];
        if (lane == 0) p.Lh[(row0 + r) * H1 + h] = v;
      }
    }
  }
}

// The same with p.adv_t decode steps applied to the lists as they stand, in one pass over them (br_project_lists).
template <int LPL, int HB, bool EXACT, int PK>
__global__ __launch_bounds__(256) void br_k_project_advance(BrParams p) {
  constexpr int LPW = BR_WAVE / LPL;
  const int wave = br_uniform((int)(threadIdx.x >> 6));
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * LPW;
  const int64_t rows = (int64_t)p.N * p.G;
  if (row0 >= rows) return;
  __shared__ __align__(16) int lds_all[4 * BR_SEG_WORDS(1)];
  br_project_lists<LPL, HB, EXACT, PK>(p, row0, (int)min(rows - row0, (int64_t)LPW), br_lane(), lds_all + wave * BR_SEG_WORDS(1));
}

__global__ __launch_bounds__(256) void br_k_project_long(BrParams p) {
  extern __shared__ int lds[];
  if ((int)blockIdx.x == p.N) {  // the estimate at age 0 that newly admitted requests get (pred_mode 2)
    if (threadIdx.x < BR_WAVE) {
      const float c = br_survival(p, 0);
      if (threadIdx.x == 0) *p.c0 = c;
    }
    return;
  }
  br_project_long<4>(p, (int)blockIdx.x, (int)threadIdx.x, lds);
}

// d = (1, gamma, ..., gamma^H) by repeated fp32 product (Sec. 4.1), zeros up to the padded length
__global__ void br_k_discounts(BrParams p, float gamma) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  float *d = const_cast<float *>(p.dl);
  float dh = 1.0f;
  for (int h = 0; h < BR_HS(p.H); ++h) {
    if (h > 0) dh = __fmul_rn(dh, gamma);
    d[h] = h <= p.H ? dh : 0.0f;
  }
}

// Step-start margins m_{g,h} = (M_h - L_g(k+h))_+ of the workers [g0, g0 + gn) of a cluster with a short horizon, from the
// projections, into sm (stride words per worker, zeros beyond offset H), by one wave: lane = worker.
__device__ __forceinline__ void br_margins_to_lds(const BrParams &p, int inst, int lane, int g0, int gn, int *sm, int stride) {
  const int64_t wrow = (int64_t)inst * p.G + min(lane, p.G - 1);
  int l[BR_HP + 1];
#pragma unroll
  for (int h = 0; h <= BR_HP; ++h) l[h] = p.Lh[wrow * (p.H + 1) + min(h, p.H)];  // (lanes beyond G repeat the last worker)
#pragma unroll
  for (int h = 0; h <= BR_HP; ++h) {
    const int m = br_wave_max(l[h]) - l[h];
    if (lane >= g0 && lane < g0 + gn) sm[(lane - g0) * stride + h] = h <= p.H ? m : 0;
  }
}

// ------------------------------------------------------------------ F-score matrix + reductions
// Scores every (waiting request, worker) pair on the step-start snapshot, eq. (brh-Fscore) in fp32.  Pass A maps lanes to requests (coalesced request-major
// reads, worker margins broadcast from LDS) and reduces over workers in registers (best worker per
// request).  Pass B maps lanes to (request sub-slot, worker) and keeps a running best
// request per worker, combined across lanes and waves at the end.
// LONG (horizons beyond BR_HP): the margins keep BR_HS(H) entries per worker, the discounts sit in LDS next
// to them and a score loops over the offsets (br_scoreh_long), skipping the four-offset groups whose margins no
// request of the tile reaches (clusters too large for br_k_score_long).
template <bool LONG>
__global__ __launch_bounds__(512) void br_k_score(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds[];
  const int G = p.G;
  const int HS = LONG ? BR_HS(p.H) : BR_HP + 1;  // margins per worker
  int *sm = lds;                         // [G][HS] margins
  float *sd = (float *)(sm + G * HS);    // LONG: [HS] discounts
  int *sL = sm + G * HS + (LONG ? HS : 0);  // [G]
  int *scap = sL + G;                    // [G]
  int *ss = scap + G;                    // [Q] prefill lengths of the waiting set
  int *cand = ss + p.Q;                  // [3][blockDim] candidates of pass B
  // a cluster may be spread over gridDim.y blocks: block `split` scores its share of the requests
  // against all workers (pass A) and all requests against its share of the workers (pass B), so no
  // result needs combining across blocks
  const int inst = blockIdx.x, split = blockIdx.y, nsplit = gridDim.y;
  const int tid = threadIdx.x, lane = br_lane(), wave = tid >> 6, nw = blockDim.x >> 6;

  const int q0 = min(max(p.qlen[inst], 0), p.Q);
  int cnt = a.count ? a.count[inst] : 0;
  cnt = min(max(cnt, 0), a.arr_cap);
  const int qn = q0 + min(cnt, p.Q - q0);

  if (tid < G) {
    sL[tid] = p.L[(int64_t)inst * G + tid];
    scap[tid] = p.B - p.n[(int64_t)inst * G + tid];
  }
  if constexpr (LONG) {  // br_scoreh_long takes the margins as floats
    for (int e = tid; e < G * HS; e += blockDim.x) {
      const int g = e / HS, h = e - g * HS;
      sm[e] = __float_as_int(h <= p.H ? (float)p.mh[((int64_t)inst * G + g) * (p.H + 1) + h] : 0.0f);
    }
  } else {
    if (wave == 0) br_margins_to_lds(p, inst, lane, 0, G, sm, HS);
  }
  if constexpr (LONG)
    for (int h = tid; h < HS; h += blockDim.x) sd[h] = p.dl[h];
  for (int i = tid; i < qn; i += blockDim.x) {
    int s = i < q0 ? p.qs[(int64_t)inst * p.Q + i] : a.s[(int64_t)inst * a.arr_cap + (i - q0)];
    ss[i] = min(max(s, 1), BR_MAX_S_DEV);
  }
  __syncthreads();
  // pass A: one request per lane, loop over workers
  for (int t0 = (split * nw + wave) * BR_WAVE; t0 < qn; t0 += nsplit * nw * BR_WAVE) {
    const int i = t0 + lane;
    const bool valid = i < qn;
    const int s = valid ? ss[i] : 1;
    int bk = BR_KEY_NONE, bg = -1;
    int tile_top[1] = {0};
    if constexpr (LONG) tile_top[0] = br_wave_max(valid ? s : 0);  // the longest request of the tile
    for (int g = 0; g < G; ++g) {
      if (scap[g] <= 0) continue;  // (no candidate)
      int key;
      if constexpr (LONG) {
        const int dv[1] = {s};
        float Fv[1];
        br_scoreh_long_sel<1>(p.aD, p.beta, (const float *)(sm + g * HS), sd, HS, lane, tile_top, dv, Fv);
        key = br_ord(Fv[0]);
      } else {
        int m[BR_HP + 1];
#pragma unroll
        for (int h = 0; h <= BR_HP; ++h) m[h] = sm[g * (BR_HP + 1) + h];
        key = br_score_key<true>(p, m, s);
      }
      const bool ok = p.W <= 0 || sL[g] + s <= p.W;
      if (ok && key > bk) {
        bk = key;
        bg = g;
      }
    }
    if (valid && o.best_g) o.best_g[(int64_t)inst * p.Q + i] = bg;
  }
  if (o.best_g && split == 0)
    for (int i = qn + tid; i < p.Q; i += blockDim.x) o.best_g[(int64_t)inst * p.Q + i] = -1;

  // pass B: lane = (sub-slot, worker of this block's share); running best request per worker
  if (o.best_i) {
    const int Gs = (G + nsplit - 1) / nsplit, gbase = split * Gs;  // workers [gbase, gbase + Gs)
    int Gp = 1;
    while (Gp < Gs) Gp <<= 1;
    const int nsub = BR_WAVE / Gp;
    const int sub = lane / Gp, gl = lane - sub * Gp, g = gbase + gl;
    const bool act = gl < Gs && g < G;
    int m[BR_HP + 1];
#pragma unroll
    for (int h = 0; h <= BR_HP; ++h) m[h] = (!LONG && act) ? sm[g * (BR_HP + 1) + h] : 0;
    const int Lg = act ? sL[g] : 0;
    const bool free_slot = act && scap[g] > 0;
    int bk = BR_KEY_NONE, bs = 0, bi = -1;
    for (int i = wave * nsub + sub; i < qn; i += nw * nsub) {
      const int s = ss[i];
      int key;
      if constexpr (LONG) {  // lanes hold different workers: each reads its own row of margins
        const int dv[1] = {s};
        float Fv[1];
        br_scoreh_long<1>(p.aD, p.beta, (const float *)(sm + (act ? g : 0) * HS), sd, HS, dv, Fv);
        key = br_ord(Fv[0]);
      } else {
        key = br_score_key<true>(p, m, s);
      }
      const bool ok = free_slot && (p.W <= 0 || Lg + s <= p.W);
      if (ok && (key > bk || (key == bk && s > bs))) {
        bk = key;
        bs = s;
        bi = i;
      }
    }
    cand[tid] = bk;
    cand[blockDim.x + tid] = bs;
    cand[2 * blockDim.x + tid] = bi;
    __syncthreads();
    if (tid < Gs && gbase + tid < G) {
      bk = BR_KEY_NONE, bs = 0, bi = -1;
      for (int w = 0; w < nw; ++w)
        for (int sb = 0; sb < nsub; ++sb) {
          const int c = w * BR_WAVE + sb * Gp + tid;
          const int k = cand[c], s = cand[blockDim.x + c], i = cand[2 * blockDim.x + c];
          if (i < 0) continue;
          if (bi < 0 || k > bk || (k == bk && (s > bs || (s == bs && i < bi)))) {
            bk = k;
            bs = s;
            bi = i;
          }
        }
      o.best_i[(int64_t)inst * G + gbase + tid] = bi;
    }
  }
}

// K2 + K3 for long horizons, a cluster per block: a score costs 3 (H + 1) operations here, so every pair is scored once,
// pairs of a worker without a free slot (no candidate on either side) not at all, and the (tile of 64 requests, worker)
// pairs left are dealt out to the block's waves whatever the queue length.  The keys meet in LDS, a column per worker
// with a free slot; best worker per request with threads mapped to requests, best request per worker with a wave per
// worker (the tie rules of br_k_score).  Groups of four offsets whose margins no request of the tile reaches are skipped.
// Overloaded clusters are nearly full most of the time: 2048 clusters, G = 8, H = 80, 135 waiting, 1.2 free slots each:
// whole pass 89.6 us with every worker scored, 75.1 so.
__global__ __launch_bounds__(1024) void br_k_score_long(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds[];
  const int G = p.G, HS = BR_HS(p.H), KS = G | 1;
  float *sm = (float *)lds;              // [G][HS] margins
  float *sd = sm + G * HS;               // [HS] discounts
  int *sL = (int *)(sd + HS);            // [G] loads
  int *sf = sL + G;                      // [G] the workers with a free slot, ascending
  int *ss = sf + G;                      // [Q] prefill lengths, then zeros to whole tiles
  int *keys = ss + ((p.Q + 63) & ~63);   // [Q'][KS] by position in sf
  const int inst = blockIdx.x, tid = threadIdx.x, lane = br_lane(), wave = tid >> 6, nw = blockDim.x >> 6;
  const int64_t wrow = (int64_t)inst * G;
  const int q0 = min(max(p.qlen[inst], 0), p.Q);
  int cnt = a.count ? a.count[inst] : 0;
  cnt = min(max(cnt, 0), a.arr_cap);
  const int qn = q0 + min(cnt, p.Q - q0);
  // (every wave reads the counts: what is free decides what it does next)
  const int n_raw = p.n[wrow + min(lane, G - 1)];
  const unsigned long long freem = br_ballot(lane < G && n_raw < p.B);
  const int nf = __builtin_popcountll(freem);
  if (nf == 0 || qn == 0) {
    if (o.best_g)
      for (int i = tid; i < p.Q; i += blockDim.x) o.best_g[(int64_t)inst * p.Q + i] = -1;
    if (o.best_i && tid < G) o.best_i[wrow + tid] = -1;
    return;
  }
  if (tid < G) {
    sL[tid] = p.L[wrow + tid];
    if ((freem >> tid) & 1ull) sf[br_rank_below(freem)] = tid;
  }
  for (int g = wave; g < G; g += nw) {
    if (!((freem >> g) & 1ull)) continue;
    for (int h = lane; h < HS; h += BR_WAVE) sm[g * HS + h] = h <= p.H ? (float)p.mh[(wrow + g) * (p.H + 1) + h] : 0.0f;
  }
  for (int h = tid; h < HS; h += blockDim.x) sd[h] = p.dl[h];
  for (int i = tid; i < ((qn + 63) & ~63); i += blockDim.x) {
    const int64_t qrow = (int64_t)inst * p.Q, arow = (int64_t)inst * a.arr_cap;
    ss[i] = i < qn ? min(max(i < q0 ? p.qs[qrow + i] : a.s[arow + (i - q0)], 1), BR_MAX_S_DEV) : 0;
  }
  __syncthreads();
  const int items = ((qn + 63) >> 6) * nf;
  for (int it = wave; it < items; it += nw) {
    const int t = it / nf, c = it - t * nf, g = br_uniform(sf[c]);
    const int s[1] = {ss[t * BR_WAVE + lane]};
    const int top[1] = {br_wave_max(s[0])};
    float F[1];
    br_scoreh_long_sel<1>(p.aD, p.beta, sm + g * HS, sd, HS, lane, top, s, F);
    keys[(t * BR_WAVE + lane) * KS + c] = br_ord(F[0]);
  }
  __syncthreads();
  if (o.best_g) {
    for (int i = tid; i < p.Q; i += blockDim.x) {
      int bk = BR_KEY_NONE, bg = -1;
      if (i < qn) {
        const int s = ss[i];
        for (int c = 0; c < nf; ++c) {
          const int key = keys[i * KS + c], g = sf[c];
          if ((p.W <= 0 || sL[g] + s <= p.W) && key > bk) bk = key, bg = g;
        }
      }
      o.best_g[(int64_t)inst * p.Q + i] = bg;
    }
  }
  if (o.best_i) {
    if (tid < G && !((freem >> tid) & 1ull)) o.best_i[wrow + tid] = -1;
    for (int c = wave; c < nf; c += nw) {
      const int g = br_uniform(sf[c]);
      int bk = BR_KEY_NONE, bs = 0, bi = INT32_MAX;
      const int room = p.W > 0 ? p.W - sL[g] : INT32_MAX;
      for (int i = lane; i < qn; i += BR_WAVE) {
        const int s = ss[i], key = keys[i * KS + c];
        if (s <= room && (key > bk || (key == bk && s > bs))) bk = key, bs = s, bi = i;
      }
      const int km = br_wave_max(bk);
      int best = -1;
      if (km != BR_KEY_NONE) {
        const int sb = br_wave_max(bk == km ? bs : -1);
        best = br_wave_min(bk == km && bs == sb ? bi : INT32_MAX);
      }
      if (lane == 0) o.best_i[wrow + g] = best;
    }
  }
}

// K2 with the matrix materialised: every (waiting request, worker) score of the step-start snapshot written to
// HBM, request-major (F[inst][i][g]), and nothing else: the reductions run as their own launch without it.
// An HBM-write stream: one block per cluster; margins and prefill lengths are staged in LDS once, then every
// thread computes the four scores of one 16-byte store straight in the output's layout (element e of the
// cluster's rows is request e / G, worker e % G, by a multiply-high with the rounded-up reciprocal of G, exact for
// e < 2^17), so the matrix leaves in full-width contiguous stores and no tile is staged.  Rows at or beyond the
// queue length are left untouched.
template <bool BRH, bool LONG>
__global__ __launch_bounds__(256) void br_k_score_matrix(BrParams p, BrArr a, BrOut o, unsigned recip_g) {
  extern __shared__ int lds[];
  const int G = p.G;
  const int HS = LONG ? BR_HS(p.H) : BR_HP + 1;
  int *sm = lds;                                   // [G][HS] margins (LONG: as floats)
  float *sd = (float *)(sm + G * HS);              // LONG: [HS + 4] discounts
  int *ss = sm + G * HS + (LONG ? HS + 4 : 0);     // [Q] prefill lengths
  int *sL = ss + p.Q;                              // [G] loads (BR-0)
  const int inst = blockIdx.x, tid = threadIdx.x;
  const int q0 = min(max(p.qlen[inst], 0), p.Q);
  int cnt = a.count ? a.count[inst] : 0;
  cnt = min(max(cnt, 0), a.arr_cap);
  const int qn = q0 + min(cnt, p.Q - q0);
  if (!BRH && tid < G) sL[tid] = p.L[(int64_t)inst * G + tid];
  if constexpr (LONG) {
    for (int e = tid; e < G * HS; e += blockDim.x) {
      const int g = e / HS, h = e - g * HS;
      sm[e] = __float_as_int(h <= p.H ? (float)p.mh[((int64_t)inst * G + g) * (p.H + 1) + h] : 0.0f);
    }
  } else if constexpr (BRH) {
    if (tid < BR_WAVE) br_margins_to_lds(p, inst, tid, 0, G, sm, HS);
  }
  if constexpr (LONG)
    for (int h = tid; h < HS + 4; h += blockDim.x) sd[h] = h < HS ? p.dl[h] : 0.0f;
  for (int i = tid; i < qn; i += blockDim.x) {
    const int s = i < q0 ? p.qs[(int64_t)inst * p.Q + i] : a.s[(int64_t)inst * a.arr_cap + (i - q0)];
    ss[i] = min(max(s, 1), BR_MAX_S_DEV);
  }
  __syncthreads();
  if (!BRH) {  // M(k) = max_g L_g, m_g = M - L_g
    if (tid < G) {
      int M = sL[0];
      for (int g = 1; g < G; ++g) M = max(M, sL[g]);
      sm[tid * HS] = M - sL[tid];
    }
    __syncthreads();
  }
  int *Fi = (int *)o.F + (int64_t)inst * p.Q * G;   // 16-byte aligned: Q * G * 4 bytes per cluster with Q * G % 4 == 0 or a scalar tail
  const int total = qn * G;
  auto score_at = [&](int e) -> int {
    const int i = G == 1 ? e : (int)__umulhi((unsigned)e, recip_g), g = e - i * G;
    int key;
    if constexpr (LONG) {
      const int dv[1] = {ss[i]};
      float Fv[1];
      br_scoreh_long<1>(p.aD, p.beta, (const float *)(sm + g * HS), sd, HS, dv, Fv);
      return __float_as_int(Fv[0]);
    } else {
      int m[BR_HP + 1];
#pragma unroll
      for (int h = 0; h <= BR_HP; ++h) m[h] = (BRH || h == 0) ? sm[g * (BR_HP + 1) + h] : 0;
      key = br_score_key<BRH>(p, m, ss[i]);
      return BRH ? __float_as_int(br_unord(key)) : key;
    }
  };
  const bool vec = (((int64_t)inst * p.Q * G) & 3) == 0;   // the cluster's rows start on a 16-byte boundary
  if (vec) {
    for (int e = 4 * tid; e < total; e += 4 * blockDim.x) {
      if (e + 3 < total) {
        *reinterpret_cast<int4 *>(Fi + e) = make_int4(score_at(e), score_at(e + 1), score_at(e + 2), score_at(e + 3));
      } else {
        for (int k = e; k < total; ++k) Fi[k] = score_at(k);
      }
    }
  } else {
    for (int e = tid; e < total; e += blockDim.x) Fi[e] = score_at(e);
  }
}

// K2 + K3 for a few clusters with long queues (single-instance serving): the block-per-cluster kernel above
// leaves most of the chip idle and its two passes score every pair twice.  Here one wave takes a tile of 64
// requests against a quarter of the workers (grid: tiles x 4 worker groups x clusters), scores each pair
// once, keeps the best worker of its group per request in registers and finds the best request of its tile per
// worker by three wave reductions (score, then length, then arrival position: the tie rule of br_k_score).
// The partial results go to a scratch area of the workspace; br_k_score_combine folds them (groups in
// ascending worker order, tiles in ascending request order, so ties resolve as in the one-block kernel).
// Scratch per cluster: pg_key, pg_g [WGN][Q]; pi_key, pi_s, pi_i [T][G].
#define BR_TILE_WORKERS 16  // most workers in a group (64 workers in 4 groups)
#define BR_TILE_GROUPS 4
__host__ __device__ inline size_t br_score_scratch_words(int Q, int G) {
  const size_t T = (size_t)(Q + BR_WAVE - 1) / BR_WAVE;
  return 2 * BR_TILE_GROUPS * (size_t)Q + 3 * T * (size_t)G;
}

template <bool BRH, bool LONG>
__global__ __launch_bounds__(64) void br_k_score_tiles(BrParams p, BrArr a, int *partials, int wpg) {
  extern __shared__ int lds[];
  const int tile = blockIdx.x, wg = blockIdx.y, inst = blockIdx.z;
  const int T = gridDim.x, WGN = gridDim.y;
  const int lane = br_lane(), G = p.G;
  const int g0 = wg * wpg, gn = min(wpg, G - g0);  // wpg <= BR_TILE_WORKERS workers per group
  const int HS = LONG ? BR_HS(p.H) : BR_HP + 1;
  int *sm = lds;                                      // [16][HS] margins of the group's workers (LONG: as floats)
  float *sd = (float *)(sm + BR_TILE_WORKERS * HS);   // LONG: [HS] discounts (+ 4 words read ahead)
  int *sL = sm + BR_TILE_WORKERS * HS + (LONG ? HS + 4 : 0);  // [16] loads, then [16] free slots
  int *scap = sL + BR_TILE_WORKERS;
  int *sc = partials + (size_t)inst * br_score_scratch_words(p.Q, G);
  int *pg_key = sc, *pg_g = sc + (size_t)WGN * p.Q;
  int *pi_key = sc + 2 * (size_t)WGN * p.Q, *pi_s = pi_key + (size_t)T * G, *pi_i = pi_s + (size_t)T * G;

  const int q0 = min(max(p.qlen[inst], 0), p.Q);
  int cnt = a.count ? a.count[inst] : 0;
  cnt = min(max(cnt, 0), a.arr_cap);
  const int qn = q0 + min(cnt, p.Q - q0);

  // worker state of the group
  if (lane < gn) {
    sL[lane] = p.L[(int64_t)inst * G + g0 + lane];
    scap[lane] = p.B - p.n[(int64_t)inst * G + g0 + lane];
  }
  if constexpr (!BRH) {  // (a score reads the first margin only)
    const int L = p.L[(int64_t)inst * G + min(lane, G - 1)], m = br_wave_max(L) - L;
    if (lane >= g0 && lane < g0 + gn) sm[(lane - g0) * HS] = m;
  } else if constexpr (!LONG) {
    br_margins_to_lds(p, inst, lane, g0, gn, sm, HS);
  } else {
    for (int e = lane; e < gn * HS; e += BR_WAVE) {
      const int gl = e / HS, h = e - gl * HS;
      sm[e] = __float_as_int(h <= p.H ? (float)p.mh[((int64_t)inst * G + g0 + gl) * (p.H + 1) + h] : 0.0f);
    }
  }
  if constexpr (LONG)
    for (int h = lane; h < HS + 4; h += BR_WAVE) sd[h] = h < HS ? p.dl[h] : 0.0f;
  br_wave_sync();

  const int i = tile * BR_WAVE + lane;
  const bool valid = i < qn;
  int s = 1;
  if (valid) s = i < q0 ? p.qs[(int64_t)inst * p.Q + i] : a.s[(int64_t)inst * a.arr_cap + (i - q0)];
  s = min(max(s, 1), BR_MAX_S_DEV);
  int bk = BR_KEY_NONE, bg = -1;
  for (int gl = 0; gl < gn; ++gl) {
    const size_t at = (size_t)tile * G + g0 + gl;
    if (scap[gl] <= 0) {  // no candidate
      if (lane == 0) pi_key[at] = BR_KEY_NONE, pi_s[at] = 0, pi_i[at] = -1;
      continue;
    }
    int key;
    if constexpr (LONG) {
      const int dv[1] = {s};
      float Fv[1];
      br_scoreh_long<1>(p.aD, p.beta, (const float *)(sm + gl * HS), sd, HS, dv, Fv);
      key = br_ord(Fv[0]);
    } else {
      int m[BR_HP + 1];
#pragma unroll
      for (int h = 0; h <= BR_HP; ++h) m[h] = BRH || h == 0 ? sm[gl * HS + h] : 0;
      key = br_score_key<BRH>(p, m, s);
    }
    const bool ok = valid && (p.W <= 0 || sL[gl] + s <= p.W);
    if (ok && key > bk) {  // workers in ascending order: the first best stays
      bk = key;
      bg = g0 + gl;
    }
    // best request of this tile for worker g: score, then the longer request, then the earlier arrival
    const int kk = ok ? key : BR_KEY_NONE;
    const int km = br_wave_max(kk);
    int sbest = 0, ibest = -1;
    if (km != BR_KEY_NONE) {
      sbest = br_wave_max(kk == km ? s : -1);
      ibest = br_wave_min((kk == km && s == sbest) ? i : INT32_MAX);
    }
    if (lane == 0) pi_key[at] = km, pi_s[at] = sbest, pi_i[at] = ibest;
  }
  if (i < p.Q) {
    pg_key[(size_t)wg * p.Q + i] = bk;
    pg_g[(size_t)wg * p.Q + i] = bg;
  }
}

// Blocks [0, QB) fold the per-group best workers of 256 requests each; the others take four workers each, one
// wave per worker with lanes mapped to tiles (at most 32), and fold the per-tile best requests by the same three
// reductions.  All partial results are requested at once: nothing here waits on a load more than once.
__global__ __launch_bounds__(256) void br_k_score_combine(BrParams p, BrOut o, const int *partials, int T, int WGN, int QB) {
  const int inst = blockIdx.y, tid = threadIdx.x, G = p.G;
  const int *sc = partials + (size_t)inst * br_score_scratch_words(p.Q, G);
  const int *pg_key = sc, *pg_g = sc + (size_t)WGN * p.Q;
  const int *pi_key = sc + 2 * (size_t)WGN * p.Q, *pi_s = pi_key + (size_t)T * G, *pi_i = pi_s + (size_t)T * G;
  if ((int)blockIdx.x < QB) {
    const int i = blockIdx.x * 256 + tid;
    if (!o.best_g || i >= p.Q) return;
    int k[4], gg[4];
#pragma unroll
    for (int wg = 0; wg < 4; ++wg) {
      k[wg] = wg < WGN ? pg_key[(size_t)wg * p.Q + i] : BR_KEY_NONE;
      gg[wg] = wg < WGN ? pg_g[(size_t)wg * p.Q + i] : -1;
    }
    int bk = BR_KEY_NONE, bg = -1;
#pragma unroll
    for (int wg = 0; wg < 4; ++wg)
      if (k[wg] > bk) bk = k[wg], bg = gg[wg];
    o.best_g[(int64_t)inst * p.Q + i] = bg;
  } else {
    const int g = ((int)blockIdx.x - QB) * 4 + (tid >> 6), lane = br_lane();
    if (!o.best_i || g >= G) return;  // whole waves leave
    const bool in = lane < T;
    const int i = in ? pi_i[(size_t)lane * G + g] : -1;
    const int k = in ? pi_key[(size_t)lane * G + g] : BR_KEY_NONE;
    const int s = in ? pi_s[(size_t)lane * G + g] : 0;
    const int kk = i >= 0 ? k : BR_KEY_NONE;
    const int km = br_wave_max(kk);
    int bi = -1;
    if (km != BR_KEY_NONE) {
      const int sbest = br_wave_max(kk == km ? s : -1);
      bi = br_wave_min((kk == km && s == sbest) ? i : INT32_MAX);
    }
    if (lane == 0) o.best_i[(int64_t)inst * G + g] = bi;
  }
}

// K2 + K3, one wave per cluster (br_score_wave.h)
template <int EM, int HB>
__global__ __launch_bounds__(256) void br_k_score_wave(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds[];
  const int w = threadIdx.x >> 6, inst = (int)(blockIdx.x * (blockDim.x >> 6)) + w;
  if (inst >= p.N) return;
  br_snapshot_helper<EM, HB>(p, a, o, inst, br_lane(), 0, 1, 0u, lds + w * (BR_LIST_WORDS(EM) + 2 * BR_WAVE));
}

// ------------------------------------------------------------------ launchers

void br_launch_clear(const BrParams &p, int *pol, hipStream_t st) {
  const int64_t n = (int64_t)p.N * p.G;
  hipLaunchKernelGGL(br_k_clear, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, pol);
}

void br_launch_load_init(const BrParams &p, const int32_t *n, const int32_t *kv, const int32_t *rem, const float *pred,
                         hipStream_t st) {
  const int64_t rows = (int64_t)p.N * p.G;
  hipLaunchKernelGGL(br_k_load_init, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, p, n, kv, rem, pred);
}

template <int NC, int RW>
static void launch_advance(const BrParams &p, int t, hipStream_t st) {
  const int64_t rows = (int64_t)p.N * p.G;
  const int rw = p.P ? 1 : RW;
  const dim3 grid((unsigned)(((rows + rw - 1) / rw + 3) / 4)), block(256);
  if (!p.P)
    hipLaunchKernelGGL((br_k_advance<NC, RW, 0>), grid, block, 0, st, p, t);
  else if (p.pred_mode == 2)
    hipLaunchKernelGGL((br_k_advance<NC, 1, 2>), grid, block, 0, st, p, t);
  else
    hipLaunchKernelGGL((br_k_advance<NC, 1, 1>), grid, block, 0, st, p, t);
}

template <int LPL>
static void launch_advance_seg(const BrParams &p, int t, hipStream_t st) {
  const int64_t rows = (int64_t)p.N * p.G;
  const int rw = p.P ? 1 : 2, per = rw * (BR_WAVE / LPL);
  const dim3 grid((unsigned)(((rows + per - 1) / per + 3) / 4)), block(256);
  if (!p.P)
    hipLaunchKernelGGL((br_k_advance_seg<LPL, 2, 0>), grid, block, 0, st, p, t);
  else if (p.pred_mode == 2)
    hipLaunchKernelGGL((br_k_advance_seg<LPL, 1, 2>), grid, block, 0, st, p, t);
  else
    hipLaunchKernelGGL((br_k_advance_seg<LPL, 1, 1>), grid, block, 0, st, p, t);
}

void br_launch_advance(const BrParams &p, int t, hipStream_t st) {
  if (p.Bs <= 64)
    launch_advance_seg<16>(p, t, st);
  else if (p.Bs <= 128)
    launch_advance_seg<32>(p, t, st);
  else if (p.Bs <= 256)
    launch_advance_seg<64>(p, t, st);
  else if (p.Bs <= 512)
    launch_advance<2, 4>(p, t, st);
  else
    launch_advance<4, 2>(p, t, st);
}

template <int NC, int RW, int HB, bool EXACT>
static void launch_project_rows_h(const BrParams &p, hipStream_t st) {
  const int64_t waves = ((int64_t)p.N * p.G + RW - 1) / RW;
  const dim3 grid((unsigned)((waves + 3) / 4) + (p.pred_mode == 2 ? 1u : 0u)), block(256);
  if (p.pred_mode == 0)
    hipLaunchKernelGGL((br_k_project_rows<NC, RW, HB, EXACT, 0>), grid, block, 0, st, p);
  else if (p.pred_mode == 3)
    hipLaunchKernelGGL((br_k_project_rows<NC, RW, HB, EXACT, 2>), grid, block, 0, st, p);
  else
    hipLaunchKernelGGL((br_k_project_rows<NC, RW, HB, EXACT, 1>), grid, block, 0, st, p);
}

template <int NC, int RW>
static void launch_project_rows(const BrParams &p, hipStream_t st) {
  if (p.H == 4)
    launch_project_rows_h<NC, RW, 4, true>(p, st);
  else if (p.H == 8)
    launch_project_rows_h<NC, RW, 8, true>(p, st);
  else if (p.H < 4)
    launch_project_rows_h<NC, RW, 4, false>(p, st);
  else
    launch_project_rows_h<NC, RW, 8, false>(p, st);
}

template <int LPL, int HB, bool EXACT>
static void launch_project_advance_h(const BrParams &p, hipStream_t st) {
  const int64_t rows = (int64_t)p.N * p.G, per = 4 * (BR_WAVE / LPL);
  const dim3 grid((unsigned)((rows + per - 1) / per)), block(256);
  if (p.pred_mode == 0)
    hipLaunchKernelGGL((br_k_project_advance<LPL, HB, EXACT, 0>), grid, block, 0, st, p);
  else if (p.pred_mode == 3)
    hipLaunchKernelGGL((br_k_project_advance<LPL, HB, EXACT, 2>), grid, block, 0, st, p);
  else
    hipLaunchKernelGGL((br_k_project_advance<LPL, HB, EXACT, 1>), grid, block, 0, st, p);
}

template <int LPL>
static void launch_project_advance(const BrParams &p, hipStream_t st) {
  if (p.H == 4)
    launch_project_advance_h<LPL, 4, true>(p, st);
  else if (p.H == 8)
    launch_project_advance_h<LPL, 8, true>(p, st);
  else if (p.H < 4)
    launch_project_advance_h<LPL, 4, false>(p, st);
  else
    launch_project_advance_h<LPL, 8, false>(p, st);
}

// BR-H, H <= 8: decode steps in the projection's pass over the lists, where the rows are supplied (maintained estimates query the
// history), lists fit br_project_lists and the round's kernel has the epilogue for it (queues of up to 512, windows of up to 8); some batches have them
// in the round's launch instead (br_route_h_advances).  Whole pass, us, the same round, a launch of their own behind it / so, B = 96, gate on, reductions asked for,
// offered load in brackets:
//   one step    1 cluster, G = 16, H = 4 (0.8) 15.1 / 10.1    H = 8 (1.3) 19.9 / 15.3    256: 17.2 / 13.4, 28.1 / 24.0    1500: 30.0 / 24.9, 57.6 / 50.1
//               2400, G = 48, H = 4 (0.7) 101 / 94.6    4096, G = 16, H = 4 (0.7, 1.3) 62.3 / 57.8, 85.6 / 78.1    G = 32, H = 4, pairs (1.3) 132 / 120    4500 (0.9) 148 / 139
//   8 steps     1500, G = 32, H = 4 (1.3) 120 / 112, no gate 191 / 183    4096, G = 32, H = 4 (0.7, 1.3) 141 / 129, 238 / 210    3000, G = 32, B = 144, H = 8 (1.3) 405 / 327
//   20 to 40    1500, G = 32, H = 4 (0.8) 90.3 / 79.1    4096 (0.7) 211 / 187    2048, G = 64, H = 8 (0.9) 423 / 353    G = 32 (0.7, 1.3) 180 / 158, 203 / 179
// (42 batches at loads of 0.7 and 1.3, gate on and off, 1, 8 and 40 steps: nowhere slower, 2 to 28 %.)
bool br_project_advances(const BrParams &p) {
  return p.H > 0 && p.H <= BR_HP && p.pred_mode != 2 && p.Bs <= 256 && p.Q <= 512 && p.R_max <= 8;
}

void br_launch_project_advance(const BrParams &p, hipStream_t st) {
  if (p.Bs <= 64)
    launch_project_advance<16>(p, st);
  else if (p.Bs <= 128)
    launch_project_advance<32>(p, st);
  else
    launch_project_advance<64>(p, st);
}

void br_launch_discounts(const BrParams &p, float gamma, hipStream_t st) {
  hipLaunchKernelGGL(br_k_discounts, dim3(1), dim3(64), 0, st, p, gamma);
}

void br_launch_project(const BrParams &p, hipStream_t st) {
  if (p.H > BR_HP) {  // projection, envelope and margins in one launch
    const size_t lds = (size_t)BR_PROJECT_LONG_WORDS(p.G, BR_HS(p.H), 4) * sizeof(int);
    hipLaunchKernelGGL(br_k_project_long, dim3((unsigned)p.N + (p.pred_mode == 2 ? 1u : 0u)), dim3(256), lds, st, p);
    return;
  }
  if (p.B <= 64)
    launch_project_rows<1, 4>(p, st);
  else if (p.B <= 128)
    launch_project_rows<2, 2>(p, st);
  else if (p.B <= 192)
    launch_project_rows<3, 2>(p, st);
  else if (p.B <= 256)
    launch_project_rows<4, 2>(p, st);
  else if (p.B <= 512)
    launch_project_rows<8, 1>(p, st);
  else
    launch_project_rows<16, 1>(p, st);
}

size_t br_score_scratch_bytes(int N, int Q, int G) {
  return N <= BR_SCORE_TILES_MAX_N ? (size_t)N * br_score_scratch_words(Q, G) * sizeof(int) : 0;
}

// The same partial results for callers that cannot allocate (br_route_step_static): a fixed device array in
// place of the workspace area, large enough for the most the tiled path ever needs (BR_SCORE_TILES_MAX_N
// clusters with the longest queue and the most workers: 1.4 MB).  Every GPU holds its own copy until the
// process ends.  Host code never uses the array by name: its address on a device comes from
// hipGetSymbolAddress, once per device, and the kernels get that pointer as an argument like any other buffer.
// Both kernels write every entry they later read, so nothing has to be cleared between calls; calls that
// overlap on one GPU (two streams) would race on it.
#define BR_STATIC_SCRATCH_WORDS (BR_SCORE_TILES_MAX_N * (2 * BR_TILE_GROUPS * 2048 + 3 * 32 * 64))
static __device__ __align__(256) int scratch[BR_STATIC_SCRATCH_WORDS];
static_assert(BR_STATIC_SCRATCH_WORDS * sizeof(int) == BR_STATIC_SCRATCH_BYTES && BR_SCORE_TILES_MAX_N == BR_STATIC_MAX_INST &&
                  BR_MAX_WAIT == 2048 && BR_MAX_G == 64,
              "the fixed scratch array covers the largest tiled score launch");

#define BR_MAX_DEVICES 64
static int *g_static_scratch[BR_MAX_DEVICES];  // device address of `scratch` per device, once resolved

size_t br_static_scratch_bytes() { return (size_t)BR_STATIC_SCRATCH_WORDS * sizeof(int); }

// Address of this library's static scratch array on the CURRENT device (resolved once per device).
hipError_t br_static_scratch_resolve(int **out) {
  *out = nullptr;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= BR_MAX_DEVICES) return hipErrorInvalidDevice;
  if (!g_static_scratch[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_static_scratch[dev] = (int *)ptr;
  }
  *out = g_static_scratch[dev];
  return hipSuccess;
}

static void br_launch_reductions(const BrParams &p, const BrArr &a, const BrOut &o, int *partials, hipStream_t st);

void br_launch_score(const BrParams &p, const BrArr &a, const BrOut &o, int *partials, hipStream_t st) {
  if (o.F) {  // the matrix as a stream of its own; the reductions, if asked for, by whichever kernel serves the shape
    const bool longh = p.H > BR_HP;
    const size_t HS = longh ? BR_HS(p.H) : BR_HP + 1;
    const size_t lds = ((size_t)p.G * HS + (longh ? HS + 4 : 0) + (size_t)p.Q + (size_t)p.G) * sizeof(int);
    const unsigned recip = (unsigned)((0x100000000ull + (unsigned)p.G - 1u) / (unsigned)p.G);  // ceil(2^32 / G)
    if (longh)
      hipLaunchKernelGGL((br_k_score_matrix<true, true>), dim3((unsigned)p.N), dim3(256), lds, st, p, a, o, recip);
    else if (p.H > 0)
      hipLaunchKernelGGL((br_k_score_matrix<true, false>), dim3((unsigned)p.N), dim3(256), lds, st, p, a, o, recip);
    else
      hipLaunchKernelGGL((br_k_score_matrix<false, false>), dim3((unsigned)p.N), dim3(256), lds, st, p, a, o, recip);
    if (!o.best_g && !o.best_i) return;
    BrOut o2 = o;
    o2.F = nullptr;
    br_launch_reductions(p, a, o2, partials, st);
    return;
  }
  br_launch_reductions(p, a, o, partials, st);
}

template <int HB>
static void launch_score_wave(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_waves_per_block(p.N);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  if (p.Q <= 256)
    hipLaunchKernelGGL((br_k_score_wave<4, HB>), grid, block, wpb * (BR_LIST_WORDS(4) + 2 * BR_WAVE) * sizeof(int), st, p, a, o);
  else if (p.Q <= 512)
    hipLaunchKernelGGL((br_k_score_wave<8, HB>), grid, block, wpb * (BR_LIST_WORDS(8) + 2 * BR_WAVE) * sizeof(int), st, p, a, o);
  else
    hipLaunchKernelGGL((br_k_score_wave<16, HB>), grid, block, wpb * (BR_LIST_WORDS(16) + 2 * BR_WAVE) * sizeof(int), st, p, a, o);
}

// The size of a BR-H cluster's reductions: units of 64 requests x worker x offset (and two more for a score's frame).
static int br_pair_units(const BrParams &p) {
  return ((p.Q + BR_WAVE - 1) / BR_WAVE) * p.G * ((p.H <= BR_HP / 2 ? BR_HP / 2 : BR_HP) + 2);
}

// Which kernel takes the reductions.  BR-0 needs no score per pair (br_score_wave.h): one wave up to queues of 1024, except
// where few clusters with queues of 513..1024 have windows beyond 8 and so a launch of their own (whole pass, us, one wave / tiles,
// Q = 1024: one cluster, G = 4 21.8 / 21.1, G = 16 29.4 / 26.8, G = 64 46.0 / 44.0; 16 clusters 30.5 / 26.6, 36.4 / 32.8, 55.2 / 53.7).
// BR-H, queues of up to 512 and windows of up to 8: on other waves of the round's block (br_k_route_h_helped) or its own.  Else more
// waves per cluster cost launches of their own, so what is faster depends on how many workers have a free slot and how many
// requests wait, which is not known here.  Whole pass (round and one decode step), us: workers full / a token watermark that
// keeps slots free everywhere and the queue full (between them: a queue nearly empty).
//   few clusters, Q <= 512             round's block       tiles
//     N =  1  G = 16  H = 8  Q = 512   21.5 / 21.1 / 41.1  27.8 / 27.5 / 48.2
//     N = 16  G = 32  H = 4  Q = 512   24.5 / 24.2 / 48.0  32.8 / 33.2 / 56.5
//     N =  1  G = 64  H = 8  Q = 256   26.3 / 25.8 / 73.6  35.1 / 34.6 / 85.5
//     N = 16  G = 64  H = 8  Q = 512   35.5 / 35.1 / 86.8  45.5 / 47.7 / 94.8
//   windows beyond 8                   one wave            tiles
//     N =  1  G = 16  H = 8  Q = 256   26.9 / 47.7         28.7 / 39.4
//     N =  1  G = 64  H = 8  Q = 512   52.8 / 90.3         54.3 / 81.3
//     N = 16  G = 64  H = 4  Q = 256   55.1 / 96.4         58.7 / 80.6
//   few clusters, Q = 1024             one wave            tiles
//     N =  1  G =  8  H = 4            30.7 / 48.4         28.9 / 37.8
//     N = 16  G = 16  H = 8            45.0 / 126          40.9 / 81
//     N =  1  G = 64  H = 8            50.7 / 112          48.6 / 98
//   more clusters, Q = 1024            one wave            block of eight waves
//     N =  64  G =  8  H = 4           40 / 57             55 / 64        (768 units)
//     N = 256  G = 16  H = 4           49 / 80             57 / 74        (1536)
//     N = 256  G = 16  H = 8           58 / 142            65 / 111       (2560)
//     N =  64  G = 64  H = 8           66 / 172            80 / 139       (10240)
//     N = 256  G = 64  H = 8           82 / 226            101 / 161
//     N = 512  G = 64  H = 8           109 / 246           151 / 214
//   hence the block from 2048 units on, where the watermark's side is the larger one, for up to a block per CU.
#define BR_UNITS_ONE_WAVE 2048
#define BR_BLOCK_MAX_N 256

// Long horizons, up to 16 clusters, more pairs of (tile of 64 requests, worker) than the round's waves take (96): one launch of
// a block per cluster (br_k_score_long) or the tiles and their combine.  The block scores the pairs of workers with a free slot
// only, and without a watermark a long queue leaves few of those; under a watermark all pairs may be scored.  97 to 128 pairs,
// whole pass, us, block / tiles:
//   overloaded     G = 13, H = 80, Q = 512 32.7 / 37.4 (16 clusters 45.4 / 49.2)   G = 32, H = 80, Q = 256 41.1 / 48.6
//                  G = 25, H = 30, Q = 256 34.7 / 38.8 (44.8 / 48.7)               G = 7, H = 80, Q = 1024, 16 clusters 68.6 / 67.3
//   watermark that keeps slots free everywhere, queue full: 64 / 55 (76 / 66), 121 / 113, 89 / 86 (102 / 98), 96 / 81
static size_t br_long_block_bytes(const BrParams &p) {  // LDS of br_k_score_long
  const size_t HS = BR_HS(p.H), Qp = ((size_t)p.Q + 63) & ~(size_t)63;
  return (((size_t)p.G + 1) * HS + 2 * (size_t)p.G + Qp + Qp * (size_t)(p.G | 1)) * sizeof(int);
}
#define BR_LONG_BLOCK_LDS (60 * 1024)

static bool br_long_in_block(const BrParams &p, int T) {
  return br_long_block_bytes(p) <= BR_LONG_BLOCK_LDS && p.W <= 0 && T * p.G <= 128;
}

bool br_score_in_tiles(const BrParams &p) {
  const int T = (p.Q + BR_WAVE - 1) / BR_WAVE, wpg = (p.G + BR_TILE_GROUPS - 1) / BR_TILE_GROUPS, WGN = (p.G + wpg - 1) / wpg;
  if (p.N > BR_SCORE_TILES_MAX_N || T * WGN < 8) return false;
  if (p.H == 0) return p.R_max > 8 && p.Q > 512;  // (narrower windows: in the round's launch)
  if (p.H > BR_HP && br_long_in_block(p, T)) return false;
  return p.H > BR_HP || p.Q > 512 || p.R_max > 8;  // (elsewhere in the round's launch)
}

static void br_launch_reductions(const BrParams &p, const BrArr &a, const BrOut &o, int *partials, hipStream_t st) {
  int waves = (p.Q + 63) / 64;  // one wave per tile of 64 requests, at most 8 waves
  waves = waves < 1 ? 1 : (waves > 8 ? 8 : waves);
  const bool longh = p.H > BR_HP;
  {  // a wave per (tile of requests, group of workers), then a combine
    const int T = (p.Q + BR_WAVE - 1) / BR_WAVE;
    const int wpg = (p.G + BR_TILE_GROUPS - 1) / BR_TILE_GROUPS, WGN = (p.G + wpg - 1) / wpg;  // at most 4 groups
    if (partials && br_score_in_tiles(p)) {
      const dim3 grid((unsigned)T, (unsigned)WGN, (unsigned)p.N), block(BR_WAVE);
      const int HS = longh ? BR_HS(p.H) : BR_HP + 1;
      const size_t lds = ((size_t)BR_TILE_WORKERS * HS + (longh ? HS + 4 : 0) + 2 * BR_TILE_WORKERS) * sizeof(int);
      if (longh)
        hipLaunchKernelGGL((br_k_score_tiles<true, true>), grid, block, lds, st, p, a, partials, wpg);
      else if (p.H > 0)
        hipLaunchKernelGGL((br_k_score_tiles<true, false>), grid, block, lds, st, p, a, partials, wpg);
      else
        hipLaunchKernelGGL((br_k_score_tiles<false, false>), grid, block, lds, st, p, a, partials, wpg);
      const int QB = (p.Q + 255) / 256;
      hipLaunchKernelGGL(br_k_score_combine, dim3((unsigned)(QB + (p.G + 3) / 4), (unsigned)p.N), dim3(256), 0, st, p, o,
                         (const int *)partials, T, WGN, QB);
      return;
    }
  }
  const bool block = p.H > 0 && p.Q > 512 && p.N <= BR_BLOCK_MAX_N && br_pair_units(p) >= BR_UNITS_ONE_WAVE;
  if (!longh && !block) {  // one wave per cluster (queues of up to 1024: longer ones do not come here)
    if (p.H == 0)
      launch_score_wave<0>(p, a, o, st);
    else if (p.H <= BR_HP / 2)
      launch_score_wave<BR_HP / 2>(p, a, o, st);
    else
      launch_score_wave<BR_HP>(p, a, o, st);
    return;
  }
  // LDS: 48 KiB at most (64 workers at a horizon of 128, queues of 2048), within the default 64 KiB per block
  const size_t HS = longh ? BR_HS(p.H) : BR_HP + 1;
  const size_t lds = ((size_t)p.G * HS + (longh ? HS : 0) + 2 * (size_t)p.G + (size_t)p.Q + 3 * 64 * (size_t)waves) * sizeof(int);
  // few clusters: spread each over several blocks (at most 8, at most one per worker) to fill more CUs
  int nsplit = 1;
  while (nsplit < 8 && nsplit * 2 <= p.G && (int64_t)p.N * nsplit * 2 <= 512 && p.Q > 64 * waves * nsplit) nsplit *= 2;
  const dim3 grid((unsigned)p.N, (unsigned)nsplit);
  if (longh && br_long_block_bytes(p) <= BR_LONG_BLOCK_LDS) {  // room for all keys of a cluster: every pair is scored once
    // sixteen waves per cluster for a few of them, eight while that leaves the batch resident at once
    const int threads = p.N <= BR_SCORE_TILES_MAX_N ? 1024 : p.N <= 1024 ? 512 : 256;
    hipLaunchKernelGGL(br_k_score_long, dim3((unsigned)p.N), dim3(threads), br_long_block_bytes(p), st, p, a, o);
    return;
  }
  if (longh)
    hipLaunchKernelGGL(br_k_score<true>, grid, dim3(64 * waves), lds, st, p, a, o);
  else
    hipLaunchKernelGGL(br_k_score<false>, grid, dim3(64 * waves), lds, st, p, a, o);
}
