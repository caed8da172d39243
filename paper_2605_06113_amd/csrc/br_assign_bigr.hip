// Instantiations of the assignment kernel for candidate windows of 9..32 requests (R_max > 8; Appendix
// "Bit-set subset selection" is about exactly this regime).  Up to 16 requests the search covers every admissible subset:
// the masks that a cardinality limit leaves, from a list (br_subset_list.h), or all of them, 1024 per lane at a few
// integer operations each (br_bigr_scan); BR-0 forms the sums themselves at limits of 3 to 5 (br_subset_few.h) and decides longer
// searches by the sums of the window's halves (br_subset_halves.h).  Rows of reachable sums (br_subset_dp.h) would need hundreds of kilobytes per worker popped and
// serve the wider windows, which no enumeration reaches.
#include "br_assign_kernel.h"

void br_launch_assign_bigr(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  if (p.H > 0)
    br_launch_assign_sized<BR_HP, true>(p, a, o, st);
  else
    br_launch_assign_sized<0, true>(p, a, o, st);
}
