// Sector kernel variants for c128 storage, fused energy (Section 2.4, Eq. sreverse_sum).
#include "sector.h"

namespace pbs {

void* sector_kernel_c128_expval(Form form, bool r16, bool rowlds, bool realc) {
  return sector_variants<double2, true>(form, r16, rowlds, realc);
}

}  // namespace pbs
