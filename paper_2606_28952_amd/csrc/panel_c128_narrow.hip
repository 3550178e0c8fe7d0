// complex128 panel kernels for at most 1,024 beta columns (panel.h; the
// variants are those of kPanelVariants in host_plan.h).
#include "panel.h"

namespace pbs {

void* panel_kernel_c128_narrow(bool expval, Form form, int variant) {
  switch (variant) {
    case 0: return panel_variant<double2, 1, 2, 8, 4>(expval, form);
    case 1: return panel_variant<double2, 1, 3, 13, 4>(expval, form);
    case 2: return panel_variant<double2, 2, 3, 10, 4>(expval, form);
    default: return panel_variant<double2, 2, 3, 13, 4>(expval, form);
  }
}

}  // namespace pbs
