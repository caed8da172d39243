// Round and decode steps of a BR-0 cluster on two waves (br_route_advance for queues of up to 512 entries,
// windows of up to 8 requests, small batches): a block holds RPB waves that each run the round of one cluster
// (Alg. BR-0) and NH helper waves that, meanwhile, compute the snapshot reductions of those clusters (if asked for) and apply the
// decode steps (Sec. 2.2) to their lists as they stand at the start of the step.  The wave that ran the round
// appends its admissions behind the old survivors, already advanced (br_assign_epilogue_split).  The decode step
// streams the lists from HBM while the rounds, dependent chains that leave the memory system idle, are still
// running: neither waits for the other except at one LDS flag per cluster, which the helper always sets.
#include "br_assign_kernel.h"

template <int E, int RPB, int NH>
__global__ __launch_bounds__((RPB + NH) * BR_WAVE) void br_k_route_split(BrParams p, BrArr a, BrOut o) {
  extern __shared__ int lds_all[];
  constexpr int WORDS = BR_ROUND_WORDS(E, false) + BR_SPLIT_WORDS;
  constexpr int HELP = BR_LIST_WORDS(E);  // the helper's list (snapshot reductions), after the clusters' areas
  constexpr int SPLIT_AT = WORDS - BR_SPLIT_WORDS;
  const int w = threadIdx.x >> 6, lane = br_lane();
  const int first = (int)blockIdx.x * RPB;
  if (w == RPB && lane < RPB) lds_all[lane * WORDS + SPLIT_AT] = 0;  // flags down before any wave looks
  __syncthreads();
  if (w < RPB) {
    const int inst = first + w;
    if (inst >= p.N) return;
    int *lds = lds_all + w * WORDS;
    br_assign_body<E, 0, false>(p, a, o, lds, inst, 0, lds + SPLIT_AT);
  } else {
    for (int c = w - RPB; c < RPB; c += NH) {  // helper h takes clusters h, h + NH, ...
      const int inst = first + c;
      if (inst >= p.N) break;
      br_split_helper<E, 8>(p, a, o, inst, lane, lds_all + c * WORDS + SPLIT_AT, lds_all + RPB * WORDS + (w - RPB) * HELP);
    }
  }
}

template <int E, int RPB, int NH>
static void launch_split(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const size_t lds = ((size_t)RPB * (BR_ROUND_WORDS(E, false) + BR_SPLIT_WORDS) + (size_t)NH * BR_LIST_WORDS(E)) * sizeof(int);
  const dim3 grid((unsigned)((p.N + RPB - 1) / RPB)), block((RPB + NH) * BR_WAVE);
  hipLaunchKernelGGL((br_k_route_split<E, RPB, NH>), grid, block, lds, st, p, a, o);
}

// For batches below two one-wave clusters per SIMD: one round and one helper per block.  Beyond, with four or more waves
// per SIMD, the decode step overlaps other clusters' rounds on the one-wave kernels as well.  Whole pass with reductions,
// us, two waves / one wave per cluster (G = 16):
//   B = 96, 256 waiting, one step      1024 clusters 19 / 27   2047: 24 / 31   3072: 29 / 35   4096: 39 / 38
//   B = 144, 246 admitted, 48 steps    1024 clusters 66 / 76   2047: 80 / 88   3072: 95 / 98   4096: 116 / 111
// (two waves are ahead up to about 3500 clusters: the line is on the safe side).
bool br_split_shape(const BrParams &p) {
  return p.H == 0 && p.R_max <= 8 && p.Q <= 512 && p.N < BR_FULL_BATCH_N;
}

bool br_split_serves(const BrParams &p) { return p.adv_t > 0 && br_split_shape(p); }

void br_launch_route_split(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    launch_split<4, 1, 1>(p, a, o, st);
  else
    launch_split<8, 1, 1>(p, a, o, st);
}
