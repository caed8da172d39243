// Long horizons: the dispatch by queue size, and the instantiations for queues of up to 256 entries (the wider ones
// are translation units of their own so that they compile side by side).
#include "br_assign_long_kernel.h"

// Waves per cluster: as many as still leave every cluster of the batch resident at once (registers allow about
// 4 / 3 / 2 / 1 waves per SIMD for queues of up to 256 / 512 / 1024 / 2048 on 1024 SIMDs).
int br_long_waves(const BrParams &p) {
  const long long room = 1024ll * (p.Q <= 256 ? 4 : p.Q <= 512 ? 3 : p.Q <= 1024 ? 2 : 1);
  return (long long)p.N * 4 <= room ? 4 : (long long)p.N * 2 <= room ? 2 : 1;
}

// Queues of up to 256, several waves a cluster: the blocks that route form the projections, where a launch of their own came before.
// Whole pass, us, so / a launch of their own, H = 80 unless given, decode lists 90 % full: one cluster of 8 workers, H = 40 16.2 / 18.0, library-
// maintained estimates 18.7 / 20.8; 100 clusters, G = 8 34.0 / 35.3; 256, G = 16 51.7 / 55.8; 1000, G = 24 72.1 / 75.1; 2048, G = 8 65.7 /
// 69.4; G = 64, H = 48 340.5 / 339.8.  One wave a cluster loses what the more waves of a launch of its own hide (4096, G = 8 91.9 / 89.9; 6000,
// H = 16 68.1 / 66.7), and with longer queues the round takes far longer than the projection (G = 32, Q = 512, H = 16 59.4 / 59.4).
bool br_long_projects(const BrParams &p) { return p.Q <= 256 && br_long_waves(p) > 1; }

// The reductions on the round's helper waves, up to 32 pairs (tile of 64 requests, worker) per wave that serves its searches; a pair
// whose worker has a free slot is about 1200 cycles, and few of them hide behind the round (BR_LONG_ALONE: many).  Up to 256 clusters
// have more waves for them (br_launch_assign_long_one).  Whole pass, us, a launch of their own / so, H = 80: one cluster, G = 8 21.8 / 19.4;
// overloaded / lightly loaded / under a watermark that keeps slots free everywhere, 1000 clusters, G = 24, Q = 256 84 / 74, 73 / 59, 175 / 167;
// 700, G = 12, Q = 512 72 / 73, 54 / 49, 125 / 123; 2048, G = 8, Q = 256 73 / 73, 61 / 60, 123 / 114, and with 128 admissions each 533 / 526.
bool br_long_helped(const BrParams &p) {
  const int nw = br_long_waves(p), T = (p.Q + BR_WAVE - 1) / BR_WAVE;
  return nw > 1 && T * p.G <= 32 * (nw - 1);
}

extern template void br_launch_assign_long_one<8>(const BrParams &, const BrArr &, const BrOut &, hipStream_t);
extern template void br_launch_assign_long_one<16>(const BrParams &, const BrArr &, const BrOut &, hipStream_t);
extern template void br_launch_assign_long_one<32>(const BrParams &, const BrArr &, const BrOut &, hipStream_t);

void br_launch_assign_long(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.Q <= 256)
    br_launch_assign_long_one<4>(p, a, o, st);
  else if (p.Q <= 512)
    br_launch_assign_long_one<8>(p, a, o, st);
  else if (p.Q <= 1024)
    br_launch_assign_long_one<16>(p, a, o, st);
  else
    br_launch_assign_long_one<32>(p, a, o, st);
}
