// Round and decode steps of a BR-0 cluster on two or three waves (br_route_advance for queues of up to 512 entries, windows
// of up to 8 requests, small batches), a block per cluster: the first wave runs the round (Alg. BR-0); meanwhile the second
// applies the decode steps (Sec. 2.2) to the lists as they stand at the start of the step, and a third, where the snapshot
// reductions or the score matrix are asked for, computes those (br_snapshot_helper).  The first wave appends its
// admissions behind the old survivors, already advanced (br_assign_epilogue_split).  The decode step streams the lists
// from HBM while the round, a dependent chain that leaves the memory system idle, is still running: the first wave waits
// at one LDS flag for each of the others before its epilogue, and those always come.
#include "br_assign_kernel.h"

// The decode steps take four long lists at a time: with eight the kernel holds 100 registers instead of 79 (queues of up to 256) and 94,
// and two fifths of the waves that were resident are not.  Whole pass with reductions, us, eight / four at a time (and with the masked
// single-word stores before either), G = 16, B = 144:
//   one step              1024 clusters 19.1 / 18.6 (19.2)    1600: 24.3 / 22.4 (23.2)    2047: 27.7 / 23.7 (24.4)    with the matrix 31.1 / 26.7 (27.0)
//   48 steps              2047 clusters 85.0 / 75.3 (76.9)
//   queues of 500         2047 clusters 33.1 / 30.9 (32.1)    without reductions 30.5 / 29.1 (29.1)
// (The bound on the block's size is that of four waves: with the true one the compiler reserves scratch memory that nothing uses.)
template <int E, bool THIRD>
__global__ __launch_bounds__(256, E == 4 ? 6 : 5) void br_k_route_split(BrParams p, BrArr a, BrOut o, unsigned recip_g) {
  extern __shared__ int lds_all[];
  const int w = threadIdx.x >> 6, lane = br_lane(), inst = (int)blockIdx.x;
  int *split = lds_all + BR_ROUND_WORDS(E, 0, false);
  // flags down before any wave looks: the lists, and what a third wave reads of the step-start state
  if (threadIdx.x == 0) split[0] = 0, split[1] = THIRD ? 0 : 1;
  __syncthreads();
  if (w == 0) {
    br_assign_body<E, 0, 0, false, false, false, false, true>(p, a, o, lds_all, inst, 0, split);
  } else if (!THIRD || w == 1) {
    br_split_advance<4>(p, inst, lane, split, split + BR_SPLIT_WORDS);
  } else if constexpr (THIRD) {
    br_snapshot_helper<E, 0>(p, a, o, inst, lane, 0, 1, recip_g, split + BR_SPLIT_WORDS + BR_PLAIN_WORDS);
    __builtin_amdgcn_s_waitcnt(0);  // every read has returned before the flag is seen
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) split[1] = 1;
  }
}

template <int E, bool THIRD>
static void launch_split_waves(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const size_t lds = (BR_ROUND_WORDS(E, 0, false) + BR_SPLIT_WORDS + BR_PLAIN_WORDS + (THIRD ? BR_LIST_WORDS(E) + 2 * BR_WAVE : 0)) * sizeof(int);
  hipLaunchKernelGGL((br_k_route_split<E, THIRD>), dim3((unsigned)p.N), dim3(BR_WAVE * (THIRD ? 3 : 2)), lds, st, p, a, o, br_recip(p.G));
}

template <int E>
static void launch_split(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (o.F || o.best_g || o.best_i)
    launch_split_waves<E, true>(p, a, o, st);
  else
    launch_split_waves<E, false>(p, a, o, st);
}

// For batches below two one-wave clusters per SIMD: one round and one helper per block.  Beyond, with four or more waves
// per SIMD, the decode step overlaps other clusters' rounds on the one-wave kernels as well.  Whole pass with reductions,
// us, two waves / one wave per cluster (G = 16):
//   B = 96, overloaded, one step       1024 clusters 15.4 / 20.2   2047: 19.8 / 23.5   3072: 25.4 / 26.1
//   B = 144, 250 admitted, 48 steps    1024 clusters 60.8 / 67.9   2047: 75.2 / 79.9   3072: 98.7 / 91.2
//   B = 144, overloaded                2048 clusters, 1 step 24.8 / 30.6   4: 35.0 / 41.0   8: 46.9 / 52.8   16: 59.8 / 64.7   48: 78.8 / 83.3
// (at 2048 two waves are ahead still: the line is on the safe side).
bool br_split_shape(const BrParams &p) {
  return p.H == 0 && p.R_max <= 8 && p.Q <= 512 && p.N < BR_FULL_BATCH_N;
}

bool br_split_serves(const BrParams &p) { return p.adv_t > 0 && br_split_shape(p); }

void br_launch_route_split(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    launch_split<4>(p, a, o, st);
  else
    launch_split<8>(p, a, o, st);
}
