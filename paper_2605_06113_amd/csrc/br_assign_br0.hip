// BR-0 instantiations of the assignment kernel (Alg. BR-0); the BR-H ones are a translation unit
// of their own so that the two compile side by side.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

// The whole round of a cluster on one wave, in one launch: the snapshot
// reductions (per-request best worker, per-worker best request: K2 + K3) on the step-start state, then the two-stage
// assignment on the same sorted list (K4, and the decode step with ADV).
// ADV: for a few decode steps, half of the waves apply them to their lists as they stand before the round (and append
// what they admit already advanced), the other half after it.  With one order for all, the memory idles while every wave
// routes and the issue slots idle while every wave streams.  After many steps rounds are long (many admissions) and the
// streaming hides in their tail anyway.  Both orders / one order, us, offered load 0.7 and 1.3 times what the workers serve:
//   4096 clusters, G = 16, B = 144    1 step 29.2 / 32.3, 38.6 / 40.3    4: 32.9 / 34.8, 51.1 / 50.0    8: 39.3 / 38.5, 66.9 / 65.5    16: - , 84.6 / 83.3
//   4096 clusters, G = 32, B = 96     1 step 34.2 / 39.9, 44.2 / 49.2    4: 37.0 / 42.0, 55.7 / 59.9    8: 39.5 / 44.6, 72.4 / 71.2    16: - , 101 / 100
//   4096 clusters, G =  8, B = 64     1 step 14.7 / 14.8, 18.5 / 18.5    4: 18.3 / 18.2, 26.3 / 26.0    8: 21.1 / 21.1, 32.1 / 32.0    16: - , 42.4 / 42.2
//   2300 clusters, G = 64, B = 60     1 step 29.5 / 37.9, 36.4 / 40.7    4: 33.6 / 39.3, 54.4 / 55.5    8: 37.2 / 41.0, 70.4 / 70.8
//   8192 clusters, G =  8, B = 96     1 step 28.9 / 28.8, 36.6 / 35.9    4: 34.7 / 34.2, 51.2 / 50.3    8: 40.4 / 39.8, 64.4 / 63.9
// 48 steps: 112 / 110, 86 / 85 and 60.6 / 60.0 on the first three.
// Batches of 4097..6144 clusters (5120 with queues beyond 256) are resident at once where the decode steps take four long lists
// at a time (ADV = 4: 80 and 83 registers, six and five waves per SIMD); with eight, 102 registers leave four.  Batches that fit four,
// or are several times that, are faster with eight.  Eight / four at a time, us (and with the masked single-word stores before either):
//   4100 clusters, G = 16, B = 144, one step 52.5 / 45.1 (49.2)    5120: 67.1 / 58.7 (61.4), 48 steps 145 / 121 (126)    6000: 73.4 / 68.6 (86.5)
//   queues of 500                            5120: 81.7 / 70.3 (72.0), 48 steps 167 / 136 (140)                         6000: 89.0 / 93.0 (99.6)
//   4096 clusters, one step 43.2 / 44.2, 48 steps 105.8 / 107.5    8192: 91.8 / 96.2    16000: 172 / 176
// (80 registers leave three words per lane in scratch memory, outside the loops: five instructions in all.)
template <int E, int ADV>
__global__ __launch_bounds__(256, ADV == 4 ? (E == 4 ? 6 : 5) : 1) void br_k_route(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  constexpr bool MIX = ADV > 0 && E <= 8;
  constexpr int ROUND = ADV ? BR_ROUND_ADV_WORDS(E) : BR_ROUND_WORDS(E, 0, false), WORDS = ROUND + (MIX ? BR_SPLIT_WORDS : 0);
  const int w = threadIdx.x >> 6, b = (int)blockIdx.x, inst = b * (int)(blockDim.x >> 6) + w;
  int *lds = lds_all + w * WORDS, *split = nullptr;
  if constexpr (MIX) {
    if (p.adv_t <= 8 && ((b + (b >> 8) + w) & 1) && inst < p.N) {  // (blocks 256 apart share a CU: both orders on every SIMD)
      split = lds + ROUND;
      if (br_lane() == 0) split[1] = 1;  // (no other wave reads this cluster)
      br_split_advance<ADV>(p, inst, br_lane(), split, lds);
    }
  }
  br_assign_body<E, 0, ADV, false, false, true>(p, a, o, lds, inst, 0, split);
}

template <int E>
static void launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_clusters_per_block(p.N, E);
  const bool adv = p.adv_t > 0;
  const size_t lds = (size_t)wpb * (adv ? BR_ROUND_ADV_WORDS(E) + (E <= 8 ? BR_SPLIT_WORDS : 0) : BR_ROUND_WORDS(E, 0, false)) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  if (adv && E <= 8 && p.N > 4 * 1024 && p.N <= (E == 4 ? 6 : 5) * 1024)
    hipLaunchKernelGGL((br_k_route<E, E <= 8 ? 4 : 8>), grid, block, lds, st, p, a, o);
  else if (adv)
    hipLaunchKernelGGL((br_k_route<E, 8>), grid, block, lds, st, p, a, o);
  else
    hipLaunchKernelGGL((br_k_route<E, 0>), grid, block, lds, st, p, a, o);
}

void br_launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    launch_route<4>(p, a, o, st);
  else if (p.Q <= 512)
    launch_route<8>(p, a, o, st);
  else
    launch_route<16>(p, a, o, st);
}

void br_launch_route_helped(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    br_launch_helped_one<4, 0>(p, a, o, st);
  else if (p.Q <= 512)
    br_launch_helped_one<8, 0>(p, a, o, st);
  else
    br_launch_helped_one<16, 0>(p, a, o, st);
}

void br_launch_assign_br0(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  br_launch_assign_sized<0>(p, a, o, st);
}
