// complex64 panel kernels of a part of a row (panel.h; the variants are those of
// kPanelVariants in host_plan.h).
#include "panel.h"

namespace pbs {

void* panel_part_c64(bool expval, bool two, int variant) {
  switch (variant) {
    case 2: return panel_part_variant<float2, 3, 10>(expval, two);
    case 4: return panel_part_variant<float2, 3, 11>(expval, two);
    default: return panel_part_variant<float2, 3, 13>(expval, two);
  }
}

}  // namespace pbs
