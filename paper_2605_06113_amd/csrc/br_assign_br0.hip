// BR-0 instantiations of the assignment kernel (Alg. BR-0); the BR-H ones are a translation unit
// of their own so that the two compile side by side.
#include "br_assign_kernel.h"
#include "br_score_wave.h"

// The whole round of a cluster with a short queue on one wave, in one launch: the snapshot
// reductions (per-request best worker, per-worker best request: K2 + K3) on the step-start state, then the two-stage
// assignment on the same sorted list (K4, and the decode step with ADV).
template <bool ADV>
__global__ __launch_bounds__(256) void br_k_route4(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  constexpr int E = 4;
  const int w = threadIdx.x >> 6;
  br_assign_body<E, 0, ADV, false, false, true>(p, a, o, lds_all + w * BR_ROUND_WORDS(E, false), (int)blockIdx.x * 4 + w);
}

void br_launch_route4(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const size_t lds = (size_t)4 * BR_ROUND_WORDS(4, false) * sizeof(int);
  const dim3 grid((unsigned)((p.N + 3) / 4)), block(256);
  if (p.adv_t > 0)
    hipLaunchKernelGGL(br_k_route4<true>, grid, block, lds, st, p, a, o);
  else
    hipLaunchKernelGGL(br_k_route4<false>, grid, block, lds, st, p, a, o);
}

void br_launch_assign_br0(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  br_launch_assign_sized<0>(p, a, o, st);
}
