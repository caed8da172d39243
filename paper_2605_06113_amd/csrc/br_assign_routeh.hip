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

// Decode steps in the round's launch, for batches that fill the chip.  Whole pass, us, as two launches / in one (lists losing
// requests all the time from about 20 steps on):
//   4096 clusters, G = 32, B = 96, H = 4, Q = 512    1 step 137 / 134    8: 215 / 186    40: 264 / 235
//   4096 clusters, G = 16, B = 96, Q = 256           H = 4, 1 step 79 / 75    H = 8, 12 steps 147 / 124
//   2048 clusters, G = 16, B = 144, H = 8, Q = 256   1 step 95 / 96
//   2048 clusters, G = 32, B = 144, c_hat supplied   40 steps 411 / 399    2300, G = 24, B = 48, the pair supplied 30: 125 / 118
// Maintained estimates look up the history per request, which the decode kernel's waves, twice as many, hide better.
bool br_route_h_advances(const BrParams &p) {
  return p.H > 0 && p.H <= BR_HP && p.pred_mode != 2 && p.R_max <= 8 && p.Q <= 512 && p.Bs <= 256 && p.N >= BR_FULL_BATCH_N;
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
