// Long-horizon assignment kernels for queues of up to 1024 entries.
#include "br_assign_long_kernel.h"

template void br_launch_assign_long_one<16>(const BrParams &, const BrArr &, const BrOut &, hipStream_t);
