// BR-0 instantiations of the assignment kernel (Alg. BR-0); the BR-H ones are a translation unit
// of their own so that the two compile side by side.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

// The whole round of a cluster on one wave, in one launch: the snapshot
// reductions (per-request best worker, per-worker best request: K2 + K3) on the step-start state, then the two-stage
// assignment on the same sorted list (K4, and the decode step with ADV).
template <int E, bool ADV>
__global__ __launch_bounds__(256) void br_k_route(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6;
  br_assign_body<E, 0, ADV, false, false, true>(p, a, o, lds_all + w * BR_ROUND_WORDS(E, false),
                                                (int)(blockIdx.x * (blockDim.x >> 6)) + w);
}

template <int E>
static void launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_clusters_per_block(p.N, E);
  const size_t lds = (size_t)wpb * BR_ROUND_WORDS(E, false) * sizeof(int);
  const dim3 grid((unsigned)((p.N + wpb - 1) / wpb)), block(BR_WAVE * wpb);
  if (p.adv_t > 0)
    hipLaunchKernelGGL((br_k_route<E, true>), grid, block, lds, st, p, a, o);
  else
    hipLaunchKernelGGL((br_k_route<E, false>), grid, block, lds, st, p, a, o);
}

void br_launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    launch_route<4>(p, a, o, st);
  else if (p.Q <= 512)
    launch_route<8>(p, a, o, st);
  else
    launch_route<16>(p, a, o, st);
}

void br_launch_assign_br0(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  br_launch_assign_sized<0>(p, a, o, st);
}
