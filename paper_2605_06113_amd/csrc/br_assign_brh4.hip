// BR-H instantiations of the assignment kernel for horizons of 1..4 offsets: half the registers and instructions per
// margin and score of the ones for up to 8.
#include "br_assign_kernel.h"

void br_launch_assign_brh4(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  br_launch_assign_sized<BR_HP / 2>(p, a, o, st);
}
