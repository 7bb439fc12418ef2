// cpull_tab.hip -- launch geometries of the compact schedule's pull (tables.hpp).
#include <hip/hip_runtime.h>

#include "tables.hpp"

namespace cglbm {
#define CK_M(G, GEN)                                                              \
  {k_cpull<G, false, StoreF32, GEN>, k_cpull<G, true, StoreF32, GEN>,             \
   k_cpull<G, true, StoreF32P, GEN>}
#define CK(G)                                                                     \
  {G::NT, G::R1, {CK_M(G, false), CK_M(G, true)},                                 \
   {k_cpull<G, false, StoreF32X, false>, k_cpull<G, true, StoreF32X, false>}}
const CPullKernels kCPull256 = CK(CG256), kCPull512 = CK(CG512);
#undef CK
#undef CK_M
}  // namespace cglbm
