// BR-H counterpart of br_k_route: for clusters with queues of up to 512 entries the wave that
// owns a cluster first computes the snapshot reductions (K2 + K3, on the step-start margins of the projection
// kernels), then runs the two-stage assignment (K4) and, ADV, applies the decode steps, in one launch.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

template <int E, int HB>
__global__ __launch_bounds__(256, E == 8 ? 4 : 1) void br_k_route_h(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6;
  br_assign_body<E, HB, 0, false, false, true>(p, a, o, lds_all + w * BR_ROUND_WORDS(E, false),
                                               (int)(blockIdx.x * (blockDim.x >> 6)) + w);
}

template <int E, int HB>
static void launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_clusters_per_block(p.N, E);
  const size_t lds = (size_t)wpb * BR_ROUND_WORDS(E, false) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  hipLaunchKernelGGL((br_k_route_h<E, HB>), grid, block, lds, st, p, a, o);
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
