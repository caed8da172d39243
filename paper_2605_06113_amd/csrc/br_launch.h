// Host-side launchers of the gfx950 kernels (one per kernel; each only enqueues).
#pragma once

#include <hip/hip_runtime.h>

#include "br_device.h"

// One wave per cluster: waves per block.  768..4096 clusters take the same time either way (BR-0 and BR-H rounds,
// pool-bypass, reductions: within 1 us of 14..80); four keep larger batches within the chip's block slots.
static inline int br_waves_per_block(int N) { return N > BR_FULL_BATCH_N ? 4 : 1; }

// `pol`: per-cluster state of the comparison policies (round-robin cursor, draws made), [N][2]
void br_launch_clear(const BrParams &p, int *pol, hipStream_t st);
void br_launch_load_init(const BrParams &p, const int32_t *n, const int32_t *kv, const int32_t *rem, const float *pred,
                         hipStream_t st);
void br_launch_advance(const BrParams &p, int t, hipStream_t st);
void br_launch_project(const BrParams &p, hipStream_t st);
// the same with p.adv_t decode steps applied to the lists as they stand, where br_project_advances
bool br_project_advances(const BrParams &p);
void br_launch_project_advance(const BrParams &p, hipStream_t st);
// horizons beyond BR_HP: fills the discount table p.dl (once per context)
void br_launch_discounts(const BrParams &p, float gamma, hipStream_t st);
// `partials`: br_score_scratch_bytes() of device memory for the partial results of the tiled path, or null
void br_launch_score(const BrParams &p, const BrArr &a, const BrOut &o, int *partials, hipStream_t st);
size_t br_score_scratch_bytes(int N, int Q, int G);
// the snapshot reductions of these shapes go to a wave per (tile of requests, group of workers)
bool br_score_in_tiles(const BrParams &p);
// the library's fixed scratch array (for the entry point that may not use workspace scratch): its size, and its
// device address on the current device
size_t br_static_scratch_bytes();
hipError_t br_static_scratch_resolve(int **out);
void br_launch_assign(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// horizons beyond BR_HP: per-offset state in LDS, one wave per cluster
void br_launch_assign_long(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// waves per cluster of that kernel (1, 2 or 4)
int br_long_waves(const BrParams &p);
// that kernel's blocks form the projections first, where nothing else needs them before it
bool br_long_projects(const BrParams &p);
// the snapshot reductions of these shapes ride on that kernel's helper waves (where o.best_g / o.best_i are set)
bool br_long_helped(const BrParams &p);
// candidate windows of 9..32 requests (H <= BR_HP); no fused decode steps
void br_launch_assign_bigr(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
void br_launch_assign_br0(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// BR-H, H <= 4
void br_launch_assign_brh4(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// Queues of 513..1024, windows of up to 8: the round on a block of four waves per cluster, as beyond 1024 (sort and epilogue
// shared; BR-0 reductions on the waves that wait), while every block is resident at once: registers leave three of these waves per
// SIMD for BR-0, two for H > 4.  Whole pass, us, one wave and its helpers / so, G = 16, a queue of 1000, reductions asked for,
// overloaded / under a watermark that keeps slots free everywhere / lightly loaded:
//   H = 0   one cluster 17.7 / 11.5, 27.2 / 20.9    256: 25.6 / 19.0, 30.4 / 24.6    600: - , - , 22.3 / 15.1    768: 32.6 / 25.7, 38.7 / 31.0
//           1024: 34.8 / 32.6, 41.9 / 48.0          2047: 47.4 / 51.0, 59.5 / 72.3
//   H = 4   16 clusters 36.5 / 29.4, 45.2 / 39.0, 25.7 / 22.2    768: 59.3 / 51.9, 77.8 / 74.7, 30.5 / 27.1, with 700 arrivals 209 / 211
//   H = 8   one cluster 33.4 / 28.1, 48.7 / 41.9, 24.0 / 22.1    512: 65.7 / 57.5, 128 / 118, 35.4 / 32.4, with 700 arrivals 394 / 363
//           1024 without reductions: 62.2 / 66.4
// Neither reductions nor matrix, overloaded, a queue of 520 | 1000, whole pass with a decode step:
//   H = 0   one cluster 16.0 / 12.7 | 18.8 / 12.9    64: 20.8 / 17.5 | 23.8 / 17.6    768: 26.3 / 25.3 | 31.0 / 27.1
//   H = 8   one cluster 25.8 / 22.5 | 29.1 / 22.3    512: 43.3 / 40.1 | 50.4 / 43.9
// `matrix` (BR-0): the helpers of one wave take the score matrix beside the round, with the block it is a launch before it; under 640 the
// sort that the block shares is worth less than that launch once a few clusters overlap.  Overloaded, lightly loaded, G = 16 (and overloaded G = 64, 64 clusters; G = 48, 300 clusters):
//   queue of 520     4 clusters 20.4 / 20.3, 14.5 / 13.6    64: 21.6 / 22.6, 14.8 / 14.2 (35.7 / 37.9)    300: 25.5 / 27.2, 16.0 / 15.8 (38.3 / 41.8)
//                    768: 32.9 / 34.4, 18.2 / 18.5
//            600     16: 22.1 / 22.0, 14.9 / 13.9           64: 22.6 / 23.0, 15.1 / 14.2                  300: 26.4 / 28.0, 16.2 / 15.8
//            700     64: 23.6 / 23.4, 16.4 / 15.0 (45.2 / 40.8)    300: 27.8 / 28.3, 17.6 / 16.7 (46.7 / 45.3)    768: 35.4 / 36.4, 20.0 / 19.2
//           1000     64: 29.4 / 25.0, 20.0 / 15.1 (58.9 / 45.7)    768: 41.2 / 39.8, 24.1 / 20.0
inline bool br_block_serves(const BrParams &p, bool matrix) {
  if (matrix && p.H == 0 && p.Q <= 640 && p.N > 16) return false;
  return p.Q > 512 && p.Q <= 1024 && p.R_max <= 8 && p.H <= BR_HP && p.N <= (p.H > 0 ? 512 : 768);
}
// BR-0, Q <= 1024: snapshot reductions and assignment in one launch
void br_launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// BR-H (H <= BR_HP), Q <= 512: the same in one launch
void br_launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, bool steps, hipStream_t st);  // steps: p.adv_t decode steps by its waves
bool br_route_h_advances(const BrParams &p, int t);  // t decode steps there and not in the projection (br_project_advances)
// batches below BR_FULL_BATCH_N without decode steps in the launch, queues of up to 512 (BR-0: 1024), windows of up to 8: the
// round with the reductions (BR-0: and the matrix) on other waves of the cluster's block
void br_launch_route_helped(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
void br_launch_route_h_helped(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
void br_launch_bypass(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// comparison policies (Random, RR, P2C, JSQ): FIFO dispatch of the waiting queue, BR-0 contexts
void br_launch_baseline(const BrParams &p, const BrArr &a, const BrOut &o, int *pol, int policy, unsigned long long seed,
                        hipStream_t st);
// BR-0 with decode steps, queues of up to 512, windows of up to 8: round and decode steps on two waves per cluster;
// the snapshot reductions and the matrix, where asked for, on a third
bool br_split_shape(const BrParams &p);   // a shape it serves (when there are decode steps)
bool br_split_serves(const BrParams &p);
void br_launch_route_split(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
