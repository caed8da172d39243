// BR-H counterpart of br_k_route: for clusters with queues of up to 512 entries the wave that
// owns a cluster first computes the snapshot reductions (K2 + K3, on the step-start margins of the projection
// kernels), then runs the two-stage assignment (K4) and, ADV, applies the decode steps (br_route_h_advances), in one launch.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

// LDS words of a cluster
static constexpr int br_route_h_words(int E, bool adv) {
  return adv && BR_TAIL_WORDS > BR_ROUND_WORDS(E, BR_HP, false) ? BR_TAIL_WORDS : BR_ROUND_WORDS(E, BR_HP, false);
}

template <int E, int HB, bool ADV>
__global__ __launch_bounds__(256, E == 8 || ADV ? 4 : 1) void br_k_route_h(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6;
  br_assign_body<E, HB, ADV, false, false, true>(p, a, o, lds_all + w * br_route_h_words(E, ADV),
                                               (int)(blockIdx.x * (blockDim.x >> 6)) + w);
}

template <int E, int HB>
static void launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, bool steps, hipStream_t st) {
  const int wpb = br_clusters_per_block(p.N, E);
  const size_t lds = (size_t)wpb * br_route_h_words(E, steps) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  if (steps)
    hipLaunchKernelGGL((br_k_route_h<E, HB, true>), grid, block, lds, st, p, a, o);
  else
    hipLaunchKernelGGL((br_k_route_h<E, HB, false>), grid, block, lds, st, p, a, o);
}

// Where br_project_advances: the decode steps by the wave that has routed the cluster.  A wave streams its cluster's lists and rows, a
// second time, while other waves still route; in the projection's pass they are streamed once, beside nothing.  That pays where rounds are
// long and end unevenly and every wave is resident at once, four to a SIMD: 3073 to 4096 clusters, hazard rows of 16 bytes and more, many steps.  The gate, which
// keeps c_hat at H for most requests, makes rounds short: there only while lists and rows come from the last-level cache, and up to 16 lists a wave.
// Whole pass, us, the same round, in the projection's pass / in the round's launch, B = 96 and 4096 clusters unless given, offered load 0.7 and 1.3 times what the workers serve:
//   no gate    G = 16, H = 4 (144 MiB)           1 step 62.0 / 61.4, 84.7 / 83.6    8: 94.1 / 90.1, 154 / 144    40: 164 / 153, 273 / 256
//                (0.4 times: 8 steps 63.6 / 66.9; the load is not known here)
//              G = 32, queues of 512             1 step 112 / 116, 160 / 159        8: 174 / 171, 314 / 299      40: 309 / 290, 570 / 543
//              G = 64, B = 64                    8: 236 / 227, 353 / 329            32: 422 / 392, 443 / 414
//              G = 16, B = 200, queues of 512    8: 172 / 170, 306 / 298            32: 244 / 228, 405 / 378
//              G = 16, H = 6                     1 step 70.3 / 76.3, 94.3 / 103     8: 114 / 115, 196 / 179      40: 210 / 193, 358 / 330
//              G = 12, B = 64, H = 8 (120 MiB)   8: 61.1 / 64.7, 97.7 / 97.6        40: 138 / 137, 227 / 220
//              G = 16, B = 40 (60 MiB)           16: 62.8 / 65.1, 109 / 109
//              3000 clusters, G = 16             8: 67.9 / 72.3, 128 / 120          40: 128 / 126, 223 / 214     3500: 8: 82.7 / 81.1, 145 / 136
//              5000                              8: 110 / 123, 179 / 185            40: 188 / 199, 319 / 321     7000: 40: 253 / 249, 427 / 417
//              2048, G = 32, H = 8               8: 149 / 155, 257 / 256            40: 282 / 282, 304 / 303
//   H < 4      H = 1, G = 32 (gate or not)       8: 89.9 / 103, 140 / 147           32: 129 / 138, 267 / 257
//              H = 3, G = 16, no gate            8: 86.8 / 92.6, 149 / 148          32: 150 / 150, 256 / 254
//   gate       G = 16, H = 4                     8: 77.2 / 76.5, 114 / 116          16: 103 / 99 (0.8), 152 / 142     40: 127 / 118, 222 / 206
//              H = 8 (240 MiB)                   4: 96.3 / 97.4, 140 / 142          16: 133 / 130, 224 / 215
//              H = 6                             1 step 66.9 / 73.8, 90.3 / 100     8: 96.7 / 101, 155 / 151     40: 165 / 152, 309 / 279
//              H = 5, B = 64 (112 MiB)           8: 70.2 / 74.2, 110 / 109          16: 85.9 / 85.1, 143 / 136
//              G = 8, H = 8                      8: 64.3 / 64.2, 107 / 105          32: 116 / 111, 204 / 197
//              G = 16, B = 40                    16: 47.5 / 49.1, 73.4 / 73.5
//              G = 24, queues of 512             4: 91.3 / 97.4, 141 / 147          16: 118 / 124, 220 / 210
//              G = 32, queues of 512 (288 MiB)   8: 129 / 140, 210 / 233            40: 187 / 204, 393 / 368
//              3500, G = 16                      8: 64.8 / 67.6, 105 / 105          40: 114 / 108, 212 / 199     5000: 144 / 161, 259 / 267
//              2048, G = 32, H = 8               8: 101 / 119, 167 / 182            40: 158 / 173, 179 / 196
//   c_hat or pairs supplied, G = 16, H = 4       8: 71.7 / 75.1, 106 / 108 and 70.1 / 75.4, 110 / 106    40: 164 / 164, 248 / 247 and 163 / 164, 256 / 248
bool br_route_h_advances(const BrParams &p, int t) {
  const int64_t mib = ((int64_t)p.N * p.G * p.Bs * (2 + p.P) * 4) >> 20;  // lists and rows
  if (p.pred_mode != 0 || p.H < 4 || p.N <= 3 * 1024 || p.N > 4 * 1024) return false;
  return p.gate > 0.0f ? t >= 16 && p.G <= 16 && mib >= 110 && mib <= 256 : t >= 8 && mib >= 140;
}

void br_launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, bool steps, hipStream_t st) {
  if (p.H <= BR_HP / 2) {
    if (p.Q <= 256)
      launch_route_h<4, BR_HP / 2>(p, a, o, steps, st);
    else
      launch_route_h<8, BR_HP / 2>(p, a, o, steps, st);
  } else if (p.Q <= 256) {
    launch_route_h<4, BR_HP>(p, a, o, steps, st);
  } else {
    launch_route_h<8, BR_HP>(p, a, o, steps, st);
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
