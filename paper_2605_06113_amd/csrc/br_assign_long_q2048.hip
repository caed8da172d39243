// Long-horizon assignment kernels for queues of up to 2048 entries.
#include "br_assign_long_kernel.h"

template void br_launch_assign_long_one<32>(const BrParams &, const BrArr &, const BrOut &, hipStream_t);
