// fused_tab2.hip -- part 2 of the fused kernel's launch geometries (tables.hpp).
#include <hip/hip_runtime.h>

#include "tables.hpp"

namespace cglbm {
const FusedKernels kFusedPart2[2] = {CGLBM_FK(FG256W, 4), CGLBM_FK(FG128, 4)};
}  // namespace cglbm
