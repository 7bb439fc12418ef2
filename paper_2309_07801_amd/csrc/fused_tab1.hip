// fused_tab1.hip -- part 1 of the fused kernel's launch geometries (tables.hpp).
#include <hip/hip_runtime.h>

#include "tables.hpp"

namespace cglbm {
const FusedKernels kFusedPart1[2] = {CGLBM_FK(FG512, 4), CGLBM_FK(FG1024, 4)};
}  // namespace cglbm
