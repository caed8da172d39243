// BR-H counterpart of br_k_route: for clusters with queues of up to 512 entries the wave that
// owns a cluster first computes the snapshot reductions (K2 + K3, on the step-start margins of the projection
// kernels), then runs the two-stage assignment (K4) and, ADV, applies the decode steps, in one launch.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

// LDS words of a cluster
static constexpr int br_route_h_words(int E, bool adv) {
  return adv && BR_TAIL_WORDS > BR_ROUND_WORDS(E, false) ? BR_TAIL_WORDS : BR_ROUND_WORDS(E, false);
}

template <int E, int HB, bool ADV>
__global__ __launch_bounds__(256, E == 8 || ADV ? 4 : 1) void br_k_route_h(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6;
  br_assign_body<E, HB, ADV, false, false, true>(p, a, o, lds_all + w * br_route_h_words(E, ADV),
                                               (int)(blockIdx.x * (blockDim.x >> 6)) + w);
}

template <int E, int HB>
static void launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_clusters_per_block(p.N, E);
  const size_t lds = (size_t)wpb * br_route_h_words(E, p.adv_t > 0) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  if (p.adv_t > 0)
    hipLaunchKernelGGL((br_k_route_h<E, HB, true>), grid, block, lds, st, p, a, o);
  else
    hipLaunchKernelGGL((br_k_route_h<E, HB, false>), grid, block, lds, st, p, a, o);
}

// Decode steps in the round's launch, for batches that fill the chip.  A wave streams its cluster's lists with fewer loads in flight
// than the decode kernel has, while other waves still route.  That pays while the latency is that of the last-level cache, or the
// lists lose enough for the round to be uneven from cluster to cluster; else the streaming only lengthens the tail of the launch.
// Whole pass, us, as two launches / in one, offered load 0.7 and 1.3 times what the workers serve (one figure: 0.9):
//   lists and rows of the batch within 240 MiB
//     4096 clusters, G = 16, B = 96, H = 4     1 step 54.4 / 49.0, 69.3 / 60.7    8: 75.0 / 62.6, 110 / 91
//     2400 clusters, G = 16, B = 144, H = 8    1 step 77.0 / 75.9                 4: 106 / 99
//     2048 clusters, G = 32, B = 96, H = 8     1 step 68.2 / 66.8, 95.3 / 96.3    8: 95.1 / 92.3, 163 / 163    40: 168 / 155, 195 / 180
//   beyond
//     2400 clusters, G = 48, B = 96, H = 4     1 step 93.8 / 100.5                4: 124 / 126
//     2400 clusters, G = 32, B = 96, H = 8     1 step 94.3 / 99.2                 4: 123 / 126
//     4500 clusters, G = 32, B = 96, H = 4     1 step 128 / 137
//     4096 clusters, G = 32, B = 96, H = 4     1 step 95.6 / 96.0, 133 / 131      8: 126 / 127, 204 / 199      (no gate 150 / 141, 317 / 280)
//       256 admissions to each of the 4096 from cold memory, no gate              1 step 176 / 179             8: 193 / 194   40: 224 / 229
//     2500 clusters, G = 32, B = 144, H = 4    1 step 81 / 87, 112 / 124          8: 116 / 119, 189 / 192     16: 140 / 140, 260 / 239
//   from 480 MiB on
//     3000 clusters, G = 32, B = 144, H = 8    1 step 141 / 151, 219 / 228        8: 222 / 229, 387 / 390     16: 275 / 272, 498 / 451
//     2048 clusters, G = 64, B = 96, H = 8     1 step 131 / 145, 189 / 199        8: 181 / 200, 344 / 338     24: 242 / 251, 252 / 257   40: 184 / 187
//     4096 clusters, G = 64, B = 96, H = 4     8 steps 272 / 275, 410 / 421       16: 315 / 329, 507 / 492    40: 243 / 237
//   a wave goes over its lists in more than 12 turns
//     2048 clusters, G = 32, B = 144, c_hat supplied    1 step 99 / 102           8: 229 / 229                40: 360 / 360
//   5 waves of the round without decode steps share a SIMD, 4 with (H <= 4, queues of up to 256)
//     4200 clusters, G = 16, B = 96, H = 4     1 step 55.9 / 58.7, 70.7 / 73.1    12: 85.9 / 86.0, 135 / 129
//     5120 clusters                            1 step 63.0 / 64.7, 81.4 / 82.1    12: 96.0 / 96.8, 155 / 157
// Maintained estimates look up the history per request, which the decode kernel's waves, twice as many, hide better.
bool br_route_h_advances(const BrParams &p, int t) {
  if (!(p.H > 0 && p.H <= BR_HP && p.pred_mode != 2 && p.R_max <= 8 && p.Q <= 512 && p.Bs <= 256 && p.N >= BR_FULL_BATCH_N)) return false;
  const int64_t bytes = (int64_t)p.N * p.G * p.Bs * (2 + p.P) * 4;
  const int lists = p.Bs <= 64 ? 8 : p.Bs <= 128 ? 4 : 2;  // of a turn
  if (bytes >= (480ll << 20)) return t > 16;
  if (p.H <= BR_HP / 2 && p.Q <= 256 && p.N > 4 * 1024 && p.N <= 5 * 1024) return t > 8;
  return t > 4 || (bytes <= (240ll << 20) && p.G <= 12 * lists);
}

void br_launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.H <= BR_HP / 2) {
    if (p.Q <= 256)
      launch_route_h<4, BR_HP / 2>(p, a, o, st);
    else
      launch_route_h<8, BR_HP / 2>(p, a, o, st);
  } else if (p.Q <= 256) {
    launch_route_h<4, BR_HP>(p, a, o, st);
  } else {
    launch_route_h<8, BR_HP>(p, a, o, st);
  }
}

void br_launch_route_h_helped(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.H <= BR_HP / 2) {
    if (p.Q <= 256)
      br_launch_helped_one<4, BR_HP / 2>(p, a, o, st);
    else
      br_launch_helped_one<8, BR_HP / 2>(p, a, o, st);
  } else if (p.Q <= 256) {
    br_launch_helped_one<4, BR_HP>(p, a, o, st);
  } else {
    br_launch_helped_one<8, BR_HP>(p, a, o, st);
  }
}
