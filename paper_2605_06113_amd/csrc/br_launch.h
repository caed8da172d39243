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
// the snapshot reductions of these shapes ride on that kernel's helper waves (where o.best_g / o.best_i are set)
bool br_long_helped(const BrParams &p);
// candidate windows of 9..32 requests (H <= BR_HP); no fused decode steps
void br_launch_assign_bigr(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
void br_launch_assign_br0(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// BR-H, H <= 4
void br_launch_assign_brh4(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// BR-0, Q <= 1024: snapshot reductions and assignment in one launch
void br_launch_route(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
// BR-H (H <= BR_HP), Q <= 512: the same in one launch
void br_launch_route_h(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st);
bool br_route_h_advances(const BrParams &p);  // its decode steps ride in that launch
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
