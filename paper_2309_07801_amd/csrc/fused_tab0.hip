// fused_tab0.hip -- part 0 of the fused kernel's launch geometries (tables.hpp).
#include <hip/hip_runtime.h>

#include "tables.hpp"

namespace cglbm {
const FusedKernels kFusedPart0[3] = {CGLBM_FK(FG256, 4), CGLBM_FK(FG256, 1), CGLBM_FK(FG256, 5)};
}  // namespace cglbm
