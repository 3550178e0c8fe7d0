// complex64 panel kernels for more than 1,024 beta columns (panel.h; the
// variants are those of kPanelVariants in host_plan.h).
#include "panel.h"

namespace pbs {

void* panel_kernel_c64_wide(bool expval, Form form, int variant) {
  switch (variant) {
    case 4: return panel_variant<float2, 4, 3, 11, 4>(expval, form);
    case 5: return panel_variant<float2, 4, 3, 13, 4>(expval, form);
    default: return panel_variant<float2, 7, 3, 13, 2>(expval, form);
  }
}

}  // namespace pbs
