// tables.hpp -- launch-geometry tables of the templated kernels.
//
// Each table is defined in a translation unit of its own (fused_tab0..2.hip,
// cpull_tab.hip, d2q9_tab.hip), so that the library's many kernel
// instantiations compile in parallel; the host code (cglbm.hip) reaches them
// through the accessors below.  The entries are host-side kernel handles:
// hipLaunchKernel resolves them to the device code of the unit that
// instantiated them.
#pragma once

#include "kernels.hpp"

namespace cglbm {

// Launch geometries of the fused kernel: nominal column extent in x and y
// (their product is the block's threads; fit_tile shapes the column to each
// box), longest z chunk, minimum waves per SIMD requested from the register
// allocator.  Every variant performs the same arithmetic per node (results
// are bitwise equal); cglbm_autotune picks the fastest for the boxes at hand.
using FusedFn = void (*)(const BoxDev *, const TileEntry *, float *, void *, int64_t, uint32_t);
struct FusedKernels {
  int nt, r3, r2, r1;  // threads; points of the tile + 3, + 2 and + 1 its LDS arrays hold
  // time step: [streaming stores, plain ones][storage][0: tiles away from
  // solid layers, 1: near them]
  FusedFn fn[2][7][2];
  FusedFn fx[2];       // field export (no population store): [near solid layers]
  FusedFn fc[2];       // compact schedule: compact state out (FP32): [near solid layers]
  FusedFn fcx[2];      // compact schedule, mass-exact storage (FP64 densities): [near solid layers]
};
#define CGLBM_FK_S(G, MW, P, S) \
  {k_fused<G, MW, false, S, false, false, P>, k_fused<G, MW, true, S, false, false, P>}
#define CGLBM_FK_P(G, MW, P)                                                                 \
  {CGLBM_FK_S(G, MW, P, StoreF32),  CGLBM_FK_S(G, MW, P, StoreF16),                           \
   CGLBM_FK_S(G, MW, P, StoreBF16), CGLBM_FK_S(G, MW, P, StoreF32X),                          \
   CGLBM_FK_S(G, MW, P, StoreF32P), CGLBM_FK_S(G, MW, P, StoreF16C),                          \
   CGLBM_FK_S(G, MW, P, StoreBF16C)}
#define CGLBM_FK(G, MW)                                                                      \
  {G::NT, G::R3, G::R2, G::R1,                                                                \
   {CGLBM_FK_P(G, MW, false), CGLBM_FK_P(G, MW, true)},                                      \
   {k_fused<G, MW, false, StoreF32, true>, k_fused<G, MW, true, StoreF32, true>},            \
   {k_fused<G, MW, false, StoreF32, false, true>, k_fused<G, MW, true, StoreF32, false, true>}, \
   {k_fused<G, MW, false, StoreF32X, false, true>, k_fused<G, MW, true, StoreF32X, false, true>}}
// Blocks of 128 to 1024 threads.  The rings' room fits the nominal shapes
// (32 x 4, 32 x 8, 64 x 4, 32 x 16 and 64 x 8, 64 x 16) and what LDS allows
// beyond them at the same blocks per CU (two of FG512, four of FG256).
using FG128 = FusedGeom<128, 384, 288, 208>;
using FG256 = FusedGeom<256, 552, 440, 350>;
using FG256W = FusedGeom<256, 704, 544, 400>;
using FG512 = FusedGeom<512, 1024, 856, 684>;
using FG1024 = FusedGeom<1024, 1540, 1360, 1188>;
// the kernels of the geometries, in three units
extern const FusedKernels kFusedPart0[3];
extern const FusedKernels kFusedPart1[2];
extern const FusedKernels kFusedPart2[2];
struct FusedVariant {
  int tx, ty, zc, minw;
  const FusedKernels *k;
};
constexpr int kNumFusedVariants = 13;
inline const FusedVariant &fused_variant(int v) {
  static const FusedVariant t[kNumFusedVariants] = {
      {32, 8, 32, 4, &kFusedPart0[0]},  {32, 8, 64, 4, &kFusedPart0[0]},
      {32, 8, 16, 4, &kFusedPart0[0]},  {32, 8, 32, 1, &kFusedPart0[1]},
      {32, 16, 32, 4, &kFusedPart1[0]}, {32, 16, 64, 4, &kFusedPart1[0]},
      {64, 4, 32, 4, &kFusedPart2[0]},  {32, 4, 32, 4, &kFusedPart2[1]},
      {32, 8, 32, 5, &kFusedPart0[2]},  {64, 8, 64, 4, &kFusedPart1[0]},
      {64, 8, 32, 4, &kFusedPart1[0]},  {64, 16, 64, 4, &kFusedPart1[1]},
      {64, 16, 32, 4, &kFusedPart1[1]}};
  return t[v];
}

// The compact schedule's pull (nominal column and longest z chunk, chosen by
// the autotuner; equal results).
using CPullFn = void (*)(const BoxDev *, const TileEntry *, const float *, float *, int64_t,
                         const void *, void *, int64_t);
struct CPullKernels {
  int nt, r1;  // threads, points of the tile + 1 its LDS array holds
  // [general equilibrium family][0 tiles away from solid layers, 1 tiles near
  // them with FP32 planes, 2 tiles near them with FP32 pairs]
  CPullFn fn[2][3];
  CPullFn fx[2];  // mass-exact storage, Model D with Q: [near solid layers]
};
using CG256 = CPullGeom<256, 400>;
using CG512 = CPullGeom<512, 684>;
extern const CPullKernels kCPull256, kCPull512;
struct CPullVariant {
  int tx, ty, zc;
  const CPullKernels *k;
};
constexpr int kNumCPullVariants = 5;
inline const CPullVariant &cpull_variant(int v) {
  static const CPullVariant t[kNumCPullVariants] = {{64, 8, 64, &kCPull512},
                                                    {64, 8, 32, &kCPull512},
                                                    {32, 8, 32, &kCPull256},
                                                    {64, 4, 32, &kCPull256},
                                                    {32, 8, 64, &kCPull256}};
  return t[v];
}

// Tile shapes of the two-dimensional (D2Q9) step kernel, 256 threads each;
// bitwise equal results, picked by cglbm_autotune.  Kernels per storage slot:
// FP32 pairs (for FP32 and FP32_PAIRS), FP16, BF16, FP32X.
using Step2Fn = void (*)(const BoxDev *, const int32_t *, const void *, void *, float *, int64_t);
struct Variant2 {
  int tx, ty;
  Step2Fn step[2][4];  // [streaming stores, plain ones][storage slot]
  Step2Fn fields[4];
};
extern const Variant2 kVariants2Table[4];
constexpr int kNumVariants2 = 4;
inline const Variant2 &variant2(int v) { return kVariants2Table[v]; }

// Initial-state kernels (three dimensions in cglbm.hip; D2Q9 per storage slot).
using InitFn = void (*)(const BoxDev *, const int32_t *, const float *, const float *,
                        const float *, void *, int64_t, uint64_t, float);
extern const InitFn kInit2[4];

}  // namespace cglbm
