// cglbm.hip -- host side of the C ABI declared in include/cglbm.h.
//
// Parameter validation, layout of the concatenated boxes, block and tile
// tables, launches on the caller's stream, FP64 diagnostics and per-kernel
// event timing.  All kernels live in kernels.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/cglbm.h"
#include "d2q9.hpp"
#include "diag.hpp"
#include "kernels.hpp"
#include "tables.hpp"

using namespace cglbm;

namespace {

thread_local std::string g_err;

// Scratch of cglbm_reduce_noalloc, a file-scope device array (each GPU the
// library runs on holds its own copy until the process ends): the chunk
// partials of the two reduction passes (kNPart doubles per chunk, at most
// kScratchChunks chunks), then the per-box diagnostics (kNPart doubles per
// box, at most kScratchBoxes boxes): 8.5 MiB.  Host code never uses the
// array's name as an address: cglbm_init looks up its device address once
// per device (g_scratch) and only that address is passed to kernels.
constexpr size_t kScratchChunks = (size_t)1 << 16;
constexpr size_t kScratchBoxes = 4096;
constexpr size_t kScratchDoubles = (kScratchChunks + kScratchBoxes) * kNPart;
static __device__ __align__(256) double scratch[kScratchDoubles];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch[kMaxDevices] = {};

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return fail(CGLBM_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),    \
                  __FILE__, __LINE__);                                                  \
  } while (0)

// Tiles of k_interface (three-kernel schedule), and the threads of its block.
// A layout takes the smallest of which all its boxes make no more than one
// tile a CU: such a launch lasts as long as one tile's chain of loads, stencils
// and barriers.  Beyond, a smaller tile only reads and computes more of its
// halo.  Measured, k_interface of 8x4x4, 8x8x4 and 8x8x8 tiles: 32^3 (256, 128
// and 64 tiles) 10.6, 11.9 and 14.2 us; 40x48x36 (540, 270, 150) 16.1, 15.3 and
// 14.3 us; 64^3 35.7, 25.9 and 20.4 us.
constexpr int kIfaceThreads = 1024;
constexpr int kCUs = 256;
using IfaceFn = void (*)(const BoxDev *, const int32_t *, float *, int64_t, int);
struct IfaceTile {
  int tx, ty, tz;
  IfaceFn fn;
};
const IfaceTile kIfaceTiles[3] = {{8, 4, 4, k_interface<8, 4, 4, kIfaceThreads>},
                                  {8, 8, 4, k_interface<8, 8, 4, kIfaceThreads>},
                                  {8, 8, 8, k_interface<8, 8, 8, kIfaceThreads>}};

using EmitFn = void (*)(const BoxDev *, const int32_t *, const float *, void *, int64_t, int64_t);
constexpr int kNumFused = kNumFusedVariants;
constexpr int kNumCPull = kNumCPullVariants;
constexpr int kNumV2 = kNumVariants2;
enum { LATTICE_D3Q27 = 0, LATTICE_D2Q9 = 1 };
constexpr int64_t kAlign = 64;             // node alignment of each box's base
// Limit of all boxes together: every plane of 8-byte values (with the plane
// length's padding of at most 2 * kAlign nodes) stays below 4 GiB, so that
// kernels address a plane with 32-bit byte offsets.
constexpr int64_t kMaxNodes = (1ll << 29) - (1ll << 20);
constexpr double kXi = 9.0 / 19.0;   // D3Q27 (Sec. II.A)
constexpr double kXi2 = 3.0 / 5.0;   // D2Q9: the rest fractions of Eq. (8) sum to one

// Kinds of timed launches: the pull of a step (k_pull, or k_cpull in the
// compact schedule), the interface and collide kernels of the three-kernel
// schedule, the fused kernel (the compact fused kernel in schedule 2), and
// the population pull that starts and the emission that ends a compact call.
enum {
  KIND_PULL = 0,
  KIND_IFACE = 1,
  KIND_COLLIDE = 2,
  KIND_FUSED = 3,
  KIND_PULL_FIRST = 4,
  KIND_EMIT = 5,
  KIND_N = 6
};

int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// Kernels by storage format (index = cglbm_storage).
using PullFn = void (*)(const BoxDev *, const int32_t *, void *, void *, float *, int64_t, int,
                        void *, int64_t, int64_t);
using WallCopyFn = void (*)(const BoxDev *, const int32_t *, const void *, void *, int64_t,
                            int64_t);
using CollideFn = void (*)(const BoxDev *, const int32_t *, float *, const void *, void *,
                          int64_t);
// [stash][storage]: the in-place layout's pull writes solid nodes to the stash
const PullFn kPull[2][7] = {{k_pull<StoreF32, false>, k_pull<StoreF16, false>,
                             k_pull<StoreBF16, false>, k_pull<StoreF32X, false>,
                             k_pull<StoreF32P, false>, k_pull<StoreF16C, false>,
                             k_pull<StoreBF16C, false>},
                            {k_pull<StoreF32, true>, k_pull<StoreF16, true>,
                             k_pull<StoreBF16, true>, k_pull<StoreF32X, true>,
                             k_pull<StoreF32P, true>, k_pull<StoreF16C, true>,
                             k_pull<StoreBF16C, true>}};
using ZeroPadFn = void (*)(const BoxDev *, void *, int64_t);
const ZeroPadFn kZeroPad[7] = {k_zero_pad<StoreF32>,  k_zero_pad<StoreF16>,
                               k_zero_pad<StoreBF16>, k_zero_pad<StoreF32X>,
                               k_zero_pad<StoreF32P>, k_zero_pad<StoreF16C>,
                               k_zero_pad<StoreBF16C>};
const CollideFn kCollide[7] = {k_collide<StoreF32>,  k_collide<StoreF16>,  k_collide<StoreBF16>,
                               k_collide<StoreF32X>, k_collide<StoreF32P>, k_collide<StoreF16C>,
                               k_collide<StoreBF16C>};
const InitFn kInit[7] = {k_init<StoreF32>,  k_init<StoreF16>,  k_init<StoreBF16>, k_init<StoreF32X>,
                         k_init<StoreF32P>, k_init<StoreF16C>, k_init<StoreBF16C>};
// [FP32 pairs][general equilibrium family]
const EmitFn kEmit[2][2] = {{k_emit<StoreF32, false>, k_emit<StoreF32, true>},
                            {k_emit<StoreF32P, false>, k_emit<StoreF32P, true>}};
// the mass-exact storages (Model D with Q), by storage (none for the plain
// FP32 layouts)
const EmitFn kEmitX[7] = {nullptr,
                          k_emit<StoreF16, false>,
                          k_emit<StoreBF16, false>,
                          k_emit<StoreF32X, false>,
                          nullptr,
                          k_emit<StoreF16C, false>,
                          k_emit<StoreBF16C, false>};
// the compact schedule of the 16-bit formats: the first pull writes the
// solid nodes' reversed populations decoded into a mass-exact FP32 stash,
// and the call's end encodes the last stash into the stored format
// [stash][storage]: the first pull of a compact call
const PullFn kPullFirst[2][7] = {
    {k_pull<StoreF32, false, StoreF32, true>, k_pull<StoreF16, false, StoreF16, true>,
     k_pull<StoreBF16, false, StoreBF16, true>, k_pull<StoreF32X, false, StoreF32X, true>,
     k_pull<StoreF32P, false, StoreF32P, true>, k_pull<StoreF16C, false, StoreF16C, true>,
     k_pull<StoreBF16C, false, StoreBF16C, true>},
    {k_pull<StoreF32, true, StoreF32, true>, k_pull<StoreF16, true, StoreF32X, true>,
     k_pull<StoreBF16, true, StoreF32X, true>, k_pull<StoreF32X, true, StoreF32X, true>,
     k_pull<StoreF32P, true, StoreF32P, true>, k_pull<StoreF16C, true, StoreF32X, true>,
     k_pull<StoreBF16C, true, StoreF32X, true>}};
const WallCopyFn kWallEncode[7] = {nullptr,
                                   k_wall_encode<StoreF16>,
                                   k_wall_encode<StoreBF16>,
                                   nullptr,
                                   nullptr,
                                   k_wall_encode<StoreF16C>,
                                   k_wall_encode<StoreBF16C>};
const WallCopyFn kWallCopy[7] = {k_wall_copy<StoreF32>,  k_wall_copy<StoreF16>,
                                 k_wall_copy<StoreBF16>, k_wall_copy<StoreF32X>,
                                 k_wall_copy<StoreF32P>, k_wall_copy<StoreF16C>,
                                 k_wall_copy<StoreBF16C>};

// D2Q9 keeps FP32 in colour pairs in either FP32 format
int storage2_slot(int32_t st) { return st == CGLBM_FP32_PAIRS ? 0 : st; }
bool storage_exact(int32_t st) { return st != CGLBM_FP32 && st != CGLBM_FP32_PAIRS; }
bool storage_16bit(int32_t st) { return storage_exact(st) && st != CGLBM_FP32_EXACT; }
size_t storage_bytes(int32_t st) {
  return (st == CGLBM_FP16_SHIFT || st == CGLBM_BF16_SHIFT || st == CGLBM_FP16_CSHIFT ||
          st == CGLBM_BF16_CSHIFT)
             ? 2
             : 4;
}
// the colour-fraction-shifted formats keep one 16-bit fraction per node
bool storage_cshift(int32_t st) { return st == CGLBM_FP16_CSHIFT || st == CGLBM_BF16_CSHIFT; }

// Bytes of one population buffer and of the aux buffer for `total` nodes.
void buffer_sizes(int32_t st, int64_t total, size_t *pop, size_t *aux, int lattice = LATTICE_D3Q27) {
  if (lattice == LATTICE_D2Q9) {
    // pair planes (9, or 8 and the FP64 rest planes of the mass-exact formats)
    const int64_t word = 2 * (int64_t)storage_bytes(st);
    if (storage_exact(st))
      *pop = (size_t)align256(8 * total * word) + (size_t)(2 * total * 8);
    else
      *pop = (size_t)(d2q9::kQ * total * word);
    *aux = (size_t)align256((int64_t)A_COUNT * total * 4) + (storage_exact(st) ? (size_t)(2 * total * 8) : 0);
    return;
  }
  if (storage_exact(st))
    *pop = (size_t)align256(52 * total * (int64_t)storage_bytes(st)) + (size_t)(2 * total * 8) +
           (storage_cshift(st) ? (size_t)(2 * total) : 0);
  else
    *pop = (size_t)(54 * total * 4);
  *aux = (size_t)align256((int64_t)A_COUNT * total * 4) + (storage_exact(st) ? (size_t)(2 * total * 8) : 0);
}

struct Layout {
  std::vector<BoxDev> boxes;
  std::vector<int32_t> blk_box, tile_box, col_box;
  std::vector<int32_t> wblk_box;  // k_wall_copy blocks (in-place layouts with walls)
  std::vector<TileEntry> col_tiles;   // k_fused blocks (D3Q27)
  std::vector<TileEntry> ccol_tiles;  // k_cpull blocks
  std::vector<int32_t> rch_box;   // reduction chunks (kRedChunk nodes of one box each)
  int64_t wtotal = 0;             // wall-node slots of all boxes (stash plane length)
  int64_t total = 0;  // plane length (nodes, all boxes, aligned)
  int64_t ctotal = 0; // plane length of the compact schedule's arrays (padded rows)
  int32_t itile = 2;  // tile of k_interface (kIfaceTiles)
  int32_t nblk = 0, ntile = 0, ncol = 0, nblk_pad = 0;
  // longest z chunk of each geometry (fit_chunk; 0 until it was selected once:
  // the autotuner selects each several times)
  int32_t cchunk[kNumCPull] = {}, fchunk[kNumFused] = {};
  // D3Q27: col_tiles and ccol_tiles hold first the tiles that run the kernel
  // without wall logic (ncol_plain, nccol_plain entries, padded to a
  // multiple of 8), then those whose stencils or rings reach a solid layer
  int32_t ncol_plain = 0, nccol_plain = 0;
  // boxes with z walls: the slabs next to them form short chunks of their
  // own (else the first and last chunks of every column are near walls)
  bool zedge = true;
  // most nodes lie in boxes whose rows of stored words are not whole 128-byte
  // lines (or sectors, see build_layout): the fused kernel's population stores
  // are plain ones
  bool ragged = false;
  // share of the fused kernel's slabs (over its columns) that lie near solid
  // layers in boxes with y walls
  double near_y = 0.0;
  bool walls = false;
  bool general = false;  // a box with Model A, B or C or without Q: three-kernel schedule
  bool full_rates = false;  // a box with a higher-order rate other than 1
  int lattice = LATTICE_D3Q27;
};

int validate(int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage) {
  if (n_boxes <= 0 || !boxes) return fail(CGLBM_EINVAL, "n_boxes must be > 0 and boxes non-NULL");
  if (storage < CGLBM_FP32 || storage > CGLBM_BF16_CSHIFT)
    return fail(CGLBM_EINVAL, "unknown storage format %d", storage);
  int64_t total = 0;
  for (int b = 0; b < n_boxes; ++b) {
    const cglbm_box_params &P = boxes[b];
    if (P.nx < 1 || P.ny < 1 || P.nz < 1)
      return fail(CGLBM_EINVAL, "box %d: extents must be >= 1", b);
    total += align_up((int64_t)P.nx * P.ny * P.nz, kAlign);
    if (total > kMaxNodes)
      return fail(CGLBM_EINVAL, "all boxes together exceed %lld nodes", (long long)kMaxNodes);
    if ((int64_t)P.nx * P.ny * P.nz > kMaxNodes)
      return fail(CGLBM_EINVAL, "box %d: more than %lld nodes", b, (long long)kMaxNodes);
    if (P.walls & ~3u) return fail(CGLBM_EINVAL, "box %d: unknown wall bits 0x%x", b, P.walls);
    if ((P.walls & 1u) && P.ny < 3) return fail(CGLBM_EINVAL, "box %d: y walls need ny >= 3", b);
    if ((P.walls & 2u) && P.nz < 3) return fail(CGLBM_EINVAL, "box %d: z walls need nz >= 3", b);
    const cglbm_phase *ph[2] = {&P.red, &P.blue};
    for (int c = 0; c < 2; ++c) {
      if (!(ph[c]->rho0 > 0.0) || !std::isfinite(ph[c]->rho0))
        return fail(CGLBM_EINVAL, "box %d: rho0 of colour %d must be > 0", b, c);
      if (!(ph[c]->alpha >= 0.0 && ph[c]->alpha < 1.0))
        return fail(CGLBM_EINVAL, "box %d: alpha of colour %d must lie in [0, 1)", b, c);
      if (!(ph[c]->nu >= 0.0) || !std::isfinite(ph[c]->nu))
        return fail(CGLBM_EINVAL, "box %d: nu of colour %d must be >= 0", b, c);
    }
    if (!std::isfinite(P.sigma) || P.sigma < 0.0)
      return fail(CGLBM_EINVAL, "box %d: sigma must be finite and >= 0", b);
    if (!std::isfinite(P.beta) || P.beta < 0.0)
      return fail(CGLBM_EINVAL, "box %d: beta must be finite and >= 0", b);
    for (int a = 0; a < 3; ++a)
      if (!std::isfinite(P.gravity[a]) || !std::isfinite(P.body_force[a]))
        return fail(CGLBM_EINVAL, "box %d: body force and gravity must be finite", b);
    if (!std::isfinite(P.rho_ref)) return fail(CGLBM_EINVAL, "box %d: rho_ref must be finite", b);
    if (P.model < CGLBM_MODEL_A || P.model > CGLBM_MODEL_D)
      return fail(CGLBM_EINVAL, "box %d: unknown equilibrium model %d", b, P.model);
    if (P.q_correction != 0 && P.q_correction != 1)
      return fail(CGLBM_EINVAL, "box %d: q_correction must be 0 or 1", b);
    if (!(P.omega_bulk > 0.0 && P.omega_bulk < 2.0))
      return fail(CGLBM_EINVAL, "box %d: omega_bulk must lie in (0, 2)", b);
    for (int k = 0; k < 9; ++k)
      if (!(P.omega_hi[k] > 0.0 && P.omega_hi[k] <= 2.0))
        return fail(CGLBM_EINVAL, "box %d: omega_hi[%d] = %g must lie in (0, 2]", b, k,
                    P.omega_hi[k]);
    for (int k = 0; k < 3; ++k)
      if (!std::isfinite(P.body_force[k]))
        return fail(CGLBM_EINVAL, "box %d: body force must be finite", b);
  }
  return CGLBM_OK;
}

// The D2Q9 lattice of App. A: one-layer boxes, the generalized equilibrium
// of Eq. (A10) with unit rates above second order.
int validate_d2q9(int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage) {
  int rc = validate(n_boxes, boxes, storage);
  if (rc) return rc;
  for (int b = 0; b < n_boxes; ++b) {
    const cglbm_box_params &P = boxes[b];
    if (P.nz != 1) return fail(CGLBM_EINVAL, "box %d: a D2Q9 box has nz = 1", b);
    if (storage_cshift(storage))
      return fail(CGLBM_EUNSUPPORTED, "the colour-fraction-shifted formats are built for D3Q27 only");
    if (P.walls & 2u) return fail(CGLBM_EINVAL, "box %d: a D2Q9 box has no z walls", b);
    if (P.model != CGLBM_MODEL_D)
      return fail(CGLBM_EUNSUPPORTED, "box %d: D2Q9 implements the equilibrium of Eq. (A10) only", b);
    for (int k = 0; k < 9; ++k)
      if (P.omega_hi[k] != 1.0)
        return fail(CGLBM_EUNSUPPORTED, "box %d: D2Q9 relaxes the higher moments at rate 1", b);
    for (int a = 0; a < 3; ++a)
      if (P.gravity[a] != 0.0) return fail(CGLBM_EUNSUPPORTED, "box %d: no buoyancy force in D2Q9", b);
  }
  return CGLBM_OK;
}

void build_layout(int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage, Layout &L,
                  int lattice = LATTICE_D3Q27) {
  L = Layout();
  L.lattice = lattice;
  const double xi = lattice == LATTICE_D2Q9 ? kXi2 : kXi;
  int64_t off = 0;
  int32_t blk = 0, tile = 0;
  for (L.itile = 0; L.itile < 2; ++L.itile) {
    const IfaceTile &it = kIfaceTiles[L.itile];
    int64_t n = 0;
    for (int b = 0; b < n_boxes; ++b)
      n += (((int64_t)boxes[b].nx + it.tx - 1) / it.tx) * ((boxes[b].ny + it.ty - 1) / it.ty) *
           ((boxes[b].nz + it.tz - 1) / it.tz);
    if (n <= kCUs) break;
  }
  const IfaceTile &it = kIfaceTiles[L.itile];
  for (int b = 0; b < n_boxes; ++b) {
    const cglbm_box_params &P = boxes[b];
    BoxDev B;
    std::memset(&B, 0, sizeof(B));
    B.nx = P.nx;
    B.ny = P.ny;
    B.nz = P.nz;
    B.walls = P.walls;
    B.n = (int64_t)P.nx * P.ny * P.nz;
    B.base = B.pbase = off;
    B.px = P.nx;
    off = align_up(off + B.n, kAlign);
    B.blk0 = blk;
    const int32_t nb = (int32_t)((B.n + kBlock - 1) / kBlock);
    for (int32_t k = 0; k < nb; ++k) L.blk_box.push_back(b);
    blk += nb;
    B.rch0 = (int32_t)L.rch_box.size();
    for (int64_t k = 0; k < (B.n + kRedChunk - 1) / kRedChunk; ++k) L.rch_box.push_back(b);
    B.tile0 = tile;
    B.tnx = (P.nx + it.tx - 1) / it.tx;
    B.tny = (P.ny + it.ty - 1) / it.ty;
    const int32_t tnz = (P.nz + it.tz - 1) / it.tz;
    const int32_t nt = B.tnx * B.tny * tnz;
    for (int32_t k = 0; k < nt; ++k) L.tile_box.push_back(b);
    tile += nt;
    B.fdx = make_fastdiv((uint32_t)P.nx);
    B.fdy = make_fastdiv((uint32_t)P.ny);
    B.ftx = make_fastdiv((uint32_t)B.tnx);
    B.fty = make_fastdiv((uint32_t)B.tny);
    B.cs2r = (float)(xi * (1.0 - P.red.alpha));
    B.cs2b = (float)(xi * (1.0 - P.blue.alpha));
    B.d2q9 = lattice == LATTICE_D2Q9 ? 1 : 0;
    B.ir0r = (float)(1.0 / P.red.rho0);
    B.ir0b = (float)(1.0 / P.blue.rho0);
    B.nu_r = (float)P.red.nu;
    B.nu_b = (float)P.blue.nu;
    B.sigma = (float)P.sigma;
    B.beta = (float)P.beta;
    B.omega2 = (float)P.omega_bulk;
    B.Gx = (float)P.body_force[0];
    B.Gy = (float)P.body_force[1];
    B.Gz = (float)P.body_force[2];
    B.bgx = (float)P.gravity[0];
    B.bgy = (float)P.gravity[1];
    B.bgz = (float)P.gravity[2];
    B.rho_ref = (float)P.rho_ref;
    B.model = P.model;
    B.qcorr = P.q_correction;
    B.full_rates = 0;
    for (int k = 0; k < 9; ++k) {
      B.omh[k] = (float)P.omega_hi[k];
      if (P.omega_hi[k] != 1.0) B.full_rates = 1;
    }
    if (P.model != CGLBM_MODEL_D || !P.q_correction || B.full_rates) L.general = true;
    if (B.full_rates) L.full_rates = true;
    {
      // pure-phase rest equilibrium of each colour: w_i rho_k^0 (c_s^k)^2 / c_s^2,
      // by speed class |c_i|^2 (D3Q27 weights, or the D2Q9 ones of Eq. A2)
      const double w3[4] = {8.0 / 27.0, 2.0 / 27.0, 1.0 / 54.0, 1.0 / 216.0};
      const double w2[4] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 36.0, 0.0};
      const double *w = lattice == LATTICE_D2Q9 ? w2 : w3;
      const double p0[2] = {P.red.rho0 * xi * (1.0 - P.red.alpha),
                            P.blue.rho0 * xi * (1.0 - P.blue.alpha)};
      for (int c = 0; c < 2; ++c)
        for (int k = 0; k < 4; ++k) B.shift[c][k] = (float)(w[k] * p0[c] * 3.0);
      // k_cpull's reference for the z momentum: the rest-state populations
      // 3 w_i p_ref (D3Q27 weights)
      const double pref = std::min(p0[0], p0[1]);
      for (int k = 0; k < 4; ++k) B.cdev[k] = (float)(-3.0 * w3[k] * pref);
      // power-of-two scale of each colour's stored values (colour-fraction
      // formats): 2^(10 - floor(log2 rho_k^0))
      const double r0[2] = {P.red.rho0, P.blue.rho0};
      for (int c = 0; c < 2; ++c) {
        const int e = std::max(-60, std::min(60, std::ilogb(r0[c]))) - 10;
        B.pscale[c] = (float)std::ldexp(1.0, -e);
        B.pinv[c] = (float)std::ldexp(1.0, e);
      }
    }
    // solid nodes: the z-wall planes, then the y-wall rows of the other layers
    {
      const int64_t nzw = (P.walls & 2u) ? 2 : 0;
      const int64_t wn = nzw * P.nx * P.ny + ((P.walls & 1u) ? 2 * (int64_t)P.nx * (P.nz - nzw) : 0);
      B.wbase = (int32_t)L.wtotal;
      B.wn = (int32_t)wn;
      B.wblk0 = (int32_t)L.wblk_box.size();
      for (int64_t k = 0; k < (wn + kBlock - 1) / kBlock; ++k) L.wblk_box.push_back(b);
      L.wtotal = align_up(L.wtotal + wn, kAlign);
    }
    L.boxes.push_back(B);
    if (P.walls) L.walls = true;
  }
  // words of the population planes: a float, or a colour pair
  const int64_t word = storage == CGLBM_FP32 && lattice == LATTICE_D3Q27
                           ? 4
                           : 2 * (int64_t)storage_bytes(storage);
  // D3Q27 rows of whole 64-byte sectors but not of whole lines keep the hint
  // beyond 128 nodes, where a row is cut into tiles that start on sectors: pull
  // and fused kernel of 200x144x177 nodes in words of 8 bytes 592 us with it,
  // 614 plain, 272x144x200 in words of 4 bytes 981 and 1027; 112x144x200 in words
  // of 4 bytes 477 and 430, 88x144x200 in words of 8 323 and 311.  D2Q9 does not
  // (1544x1203 in words of 8 bytes 80.9 us a step with it, 61.2 plain).
  int64_t ragged = 0, nodes = 0;
  for (const BoxDev &B : L.boxes) {
    const int64_t row = B.nx * word, unit = lattice == LATTICE_D3Q27 && B.nx > 128 ? 64 : 128;
    nodes += B.n;
    if (row % unit) ragged += B.n;
  }
  L.ragged = 2 * ragged > nodes;
  // Plane length: an odd multiple of kAlign nodes, so that consecutive
  // planes of 4-byte words start an odd number of 256-byte units apart and
  // one wave's accesses to the 27 planes spread over more memory channels
  // (16-bit storage measured 1-3 % faster than with power-of-two planes).
  L.total = std::max<int64_t>(off, kAlign);
  if ((L.total / kAlign) % 2 == 0) L.total += kAlign;
  L.ctotal = L.total;
  L.nblk = blk;
  L.ntile = tile;
  // grids remapped across XCDs are padded to a multiple of 8 idle blocks
  L.nblk_pad = (int32_t)align_up(blk, 8);
  while ((int32_t)L.blk_box.size() < L.nblk_pad) L.blk_box.push_back(-1);
}

// Rows of the compact schedule's arrays (the compact state in a population
// buffer, the moments in aux): padded to 64 bytes if all boxes' padded planes
// fit the caller's buffers (whose sizes are those of the unpadded populations
// and of 21 aux planes; the schedule uses 15 and 11, and two FP64 planes with
// the mass-exact formats), else not.  A tile's row segments then start on a
// sector and its streaming stores fill whole ones: unpadded, the 16-bit
// 190x131x150 box took 182 + 218 us a step, padded 157 + 171.  (To 128 bytes:
// the same there, but 24 boxes of 24 to 128 nodes an edge take 5 % longer.)
void pad_rows(Layout &L, int32_t storage) {
  constexpr int32_t kUnit = 16;
  size_t pop = 0, aux = 0;
  buffer_sizes(storage, L.total, &pop, &aux);
  const int64_t extra = storage_exact(storage) ? 16 : 0;
  int64_t off = 0;
  for (const BoxDev &B : L.boxes)
    off = align_up(off + align_up(B.nx, kUnit) * B.ny * B.nz, kAlign);
  int64_t total = std::max<int64_t>(off, kAlign);
  if ((total / kAlign) % 2 == 0) total += kAlign;
  if (total > kMaxNodes + 2 * kAlign ||
      align256(kCompact * total * 4) + extra * total > (int64_t)pop ||
      align256(kMoments * total * 4) + extra * total > (int64_t)aux)
    return;
  off = 0;
  for (BoxDev &B : L.boxes) {
    B.pbase = off;
    B.px = (int32_t)align_up(B.nx, kUnit);
    off = align_up(off + (int64_t)B.px * B.ny * B.nz, kAlign);
  }
  L.ctotal = total;
}

// Split of a box's tiles between the launch without wall logic and the one
// with it: a tile goes to the latter if the y rows or z slabs it reads
// (its extent widened by `halo`) come within one node of a solid layer.
bool tile_near_walls(const BoxDev &B, int y0, int ty, int z0, int z1, int halo) {
  const bool yw = (B.walls & 1u) && !(y0 - halo - 1 >= 1 && y0 + ty + halo <= B.ny - 2);
  const bool zw = (B.walls & 2u) && !(z0 - halo - 1 >= 1 && z1 + halo <= B.nz - 2);
  return yw || zw;
}

// The tiles of one launch as the XCD remap deals them: eighth k of the list
// runs on XCD k, in order.  The tiles of one box, and chunks of one length,
// keep their order; else the chunks go longest first, each to the XCD with the
// least work so far, in pieces of an eighth of a chunk's tiles (neighbours
// share halo lines), so that the XCDs end together and the last blocks are
// short.  24 boxes of 24 to 128 nodes an edge, compact pull and fused kernel:
// 408 + 427 us in order, 379 + 421 dealt; 50 boxes 757 + 813 and 724 + 779;
// 9 boxes 157 + 157 and 140 + 146.
void deal_tiles(std::vector<TileEntry> &t, bool deal) {
  const TileEntry pad = {-1, 0, 0, 0};
  auto len = [](const TileEntry &e) { return e.z1 - e.z0; };
  auto shorter = [&](const TileEntry &a, const TileEntry &b) { return len(a) < len(b); };
  if (deal && !t.empty() && len(*std::max_element(t.begin(), t.end(), shorter)) >
                        len(*std::min_element(t.begin(), t.end(), shorter)) + 1) {
    std::stable_sort(t.begin(), t.end(),
                     [&](const TileEntry &a, const TileEntry &b) { return len(a) > len(b); });
    std::vector<TileEntry> xcd[8];
    int64_t work[8] = {};
    for (size_t i = 0; i < t.size();) {
      size_t run = i + 1;  // the chunk's tiles
      while (run < t.size() && t[run].box == t[i].box && t[run].z0 == t[i].z0) ++run;
      for (const size_t piece = (run - i + 7) / 8; i < run;) {
        const size_t n = std::min(piece, run - i);
        const size_t k = (size_t)(std::min_element(work, work + 8) - work);
        xcd[k].insert(xcd[k].end(), t.begin() + (int64_t)i, t.begin() + (int64_t)(i + n));
        work[k] += (int64_t)n * (len(t[i]) + 2);
        i += n;
      }
    }
    size_t most = 0;
    for (const auto &x : xcd) most = std::max(most, x.size());
    t.clear();
    for (auto &x : xcd) {
      x.resize(most, pad);
      t.insert(t.end(), x.begin(), x.end());
    }
  }
  while (t.size() % 8) t.push_back(pad);
}

// Plain tiles first, then the tiles near walls, each list a multiple of 8
// long (the XCD remap); returns the length of the first list.
int32_t pack_tiles(std::vector<TileEntry> &out, std::vector<TileEntry> &plain,
                   std::vector<TileEntry> &near, bool deal) {
  deal_tiles(plain, deal);
  deal_tiles(near, deal);
  out = plain;
  out.insert(out.end(), near.begin(), near.end());
  return (int32_t)plain.size();
}

// Column tile of an nx x ny box for a block of nt threads whose LDS rings
// hold r3, r2 and r1 points of the tile + 3, + 2 and + 1 (0: no such ring):
// of the shapes that fit, the one that covers the box with the fewest tiles,
// counting 4 / w of a tile for its short rows (each row segment of w nodes
// touches one more cache line than it fills; twice that where its neighbours
// share 64-byte sectors with it); the nominal shape wins ties.
// A fixed shape left most lanes of ragged boxes idle: a 70 x 70 layer takes
// 18 tiles of 64 x 8 but 12 of 80 x 6.
void fit_tile(int nx, int ny, int tx, int ty, int nt, int r3, int r2, int r1, TileShape &T) {
  double best = 1e300;
  auto consider = [&](int w, int h) {
    if (w < 1 || h < 1 || w * h > nt || h > 48) return;
    if (2 * (w + 2 + h) > nt || ((2 * w + 63) & ~63) + 2 * (h + 2) > nt) return;
    if ((r3 && (w + 6) * (h + 6) > r3) || (r2 && (w + 4) * (h + 4) > r2)) return;
    if ((w + 2) * (h + 2) > r1) return;
    const double lines = w % 16 && w < nx ? 8.0 : 4.0;
    const double n = (double)((nx + w - 1) / w) * ((ny + h - 1) / h) * (1.0 + lines / w);
    if (n < best * (1.0 - 1e-9)) {
      best = n;
      T.w = w;
      T.h = h;
    }
  };
  consider(tx, ty);
  for (int w = 8; w <= 128; w += 8)
    for (int h = std::min(48, nt / w); h >= 1; --h) consider(w, h);
  if (nx <= 128)
    for (int h = std::min(48, nt / nx); h >= 1; --h) consider(nx, h);
  T.d0 = make_fastdiv((uint32_t)T.w);
  T.d4 = make_fastdiv((uint32_t)T.w + 4);
  T.d6 = make_fastdiv((uint32_t)T.w + 6);
}

// z chunks [z0, z1) of a box: as few as zc slabs a chunk allow, of even
// length, except that a box with z walls gets a chunk of `edge` slabs at each
// wall, so that the chunks between them (whose stencils then stay clear of
// the walls) run without wall logic.
std::vector<std::pair<int, int>> z_chunks(const BoxDev &B, int zc, int edge) {
  std::vector<std::pair<int, int>> out;
  int lo = 0, hi = B.nz;
  if (edge > 0 && (B.walls & 2u) && B.nz > 2 * edge + zc) {
    out.push_back({0, edge});
    lo = edge;
    hi = B.nz - edge;
  }
  const int n = (hi - lo + zc - 1) / zc;
  for (int k = 0; k < n; ++k)
    out.push_back({lo + (int)((int64_t)(hi - lo) * k / n), lo + (int)((int64_t)(hi - lo) * (k + 1) / n)});
  if (hi < B.nz) out.push_back({hi, B.nz});
  return out;
}

// Longest chunk to cut the boxes into, at most zc and at least zc / 2: the
// one with the least estimated time.  The blocks, longest first, are assigned
// to the places the GPU has for them (256 CUs of 1024 threads, the occupancy of the
// tiled kernels); a block takes its slabs and `lead` more iterations, and an
// iteration the longer the more of the places are taken: measured for the
// compact fused kernel at 192^3, 4.1 us with 216 blocks and 6.3 us with 432
// of 512 places, so a + b (places taken) with a : b = 2.1 : 4.6.
int fit_chunk(const Layout &L, bool cpull, int zc, int nt, double lead) {
  const size_t places = 256 * (size_t)(1024 / nt);
  int best = zc;
  double best_t = 1e300;
  std::vector<double> busy;
  for (int k = 0; k <= 8; ++k) {
    const int z = std::max(1, zc - zc * k / 16);
    size_t blocks = 0;
    for (const BoxDev &B : L.boxes) {
      const TileShape &T = cpull ? B.cs : B.fs;
      blocks += (size_t)((B.nx + T.w - 1) / T.w) * ((B.ny + T.h - 1) / T.h) * ((B.nz + z - 1) / z);
    }
    if (blocks > 16 * places) return zc;  // many rounds: the last one matters little
    std::vector<std::pair<double, size_t>> lens;  // blocks of each box
    for (const BoxDev &B : L.boxes) {
      const TileShape &T = cpull ? B.cs : B.fs;
      const size_t cols = (size_t)((B.nx + T.w - 1) / T.w) * ((B.ny + T.h - 1) / T.h);
      const int n = (B.nz + z - 1) / z;
      lens.push_back({(double)B.nz / n + lead, cols * n});
    }
    std::sort(lens.begin(), lens.end(), std::greater<std::pair<double, size_t>>());
    busy.assign(places, 0.0);             // a min-heap of the places' end times
    for (const auto &[len, count] : lens) {
      // (end times within one block of each other: whole rounds give each
      // place one block)
      const auto [lo, hi] = std::minmax_element(busy.begin(), busy.end());
      const size_t rounds = *hi - *lo <= len ? count / places : 0;
      for (double &t : busy) t += (double)rounds * len;
      for (size_t c = rounds * places; c < count; ++c) {
        std::pop_heap(busy.begin(), busy.end(), std::greater<double>());
        busy.back() += len;
        std::push_heap(busy.begin(), busy.end(), std::greater<double>());
      }
    }
    const double t = *std::max_element(busy.begin(), busy.end()) *
                     (2.1 + 4.6 * std::min(1.0, (double)blocks / places));
    if (t < best_t * 0.98) {
      best_t = t;
      best = z;
    }
  }
  return best;
}

// Tile lists of one kernel geometry: every (chunk, column) of every box,
// split by tile_near_walls with the kernel's reach `halo`; `edge` slabs form
// the chunks at z walls.
void build_tiles(Layout &L, int zc, int halo, int edge, std::vector<TileEntry> &out,
                 int32_t &nplain, bool cpull) {
  std::vector<TileEntry> plain, near;
  for (size_t b = 0; b < L.boxes.size(); ++b) {
    BoxDev &B = L.boxes[b];
    const TileShape &T = cpull ? B.cs : B.fs;
    const int32_t ncx = (B.nx + T.w - 1) / T.w, ncy = (B.ny + T.h - 1) / T.h;
    if (cpull) {
      B.cncx = ncx;
      B.cncy = ncy;
      B.fccx = make_fastdiv((uint32_t)ncx);
      B.fccy = make_fastdiv((uint32_t)ncy);
    } else {
      B.ncx = ncx;
      B.ncy = ncy;
      B.fcx = make_fastdiv((uint32_t)ncx);
      B.fcy = make_fastdiv((uint32_t)ncy);
    }
    for (const auto &zr : z_chunks(B, zc, edge))
      for (int32_t cy = 0; cy < ncy; ++cy)
        for (int32_t cx = 0; cx < ncx; ++cx) {
          auto walled = [&](int z0, int z1) {
            return tile_near_walls(B, cy * T.h, T.h, z0, z1, halo);
          };
          const int32_t xy = cx + ncx * cy, len = zr.second - zr.first;
          if (!walled(zr.first, zr.second)) {
            plain.push_back({(int32_t)b, xy, zr.first, zr.second});
            continue;
          }
          // near a wall: halves of a full chunk, but what stays clear of the
          // wall in one piece with the plain tiles.  The few blocks beside a
          // wall march with wall logic at half the speed, and a launch lasts
          // as long as they do: 384x192x192 between walls, 10 steps 9.70 ms in
          // whole chunks, 9.45-9.50 in halves, 9.46-9.73 with the pull's in
          // quarters, 9.93 with both in quarters; 300x150x170 6.32,
          // 6.11-6.33, 6.11 ms
          const int n = std::max(1, len / std::max(8, zc / 2));
          int open = zr.first;  // first slab of the plain pieces not yet listed
          for (int k = 0; k < n; ++k) {
            const int z0 = zr.first + len * k / n, z1 = zr.first + len * (k + 1) / n;
            if (!walled(z0, z1)) continue;
            if (open < z0) plain.push_back({(int32_t)b, xy, open, z0});
            near.push_back({(int32_t)b, xy, z0, z1});
            open = z1;
          }
          if (open < zr.second) plain.push_back({(int32_t)b, xy, open, zr.second});
        }
  }
  nplain = pack_tiles(out, plain, near, L.boxes.size() > 1);
}

// Column table of k_cpull variant v.  Its ring reaches one node around the
// column and one slab beyond the chunk.
void build_ccolumns(Layout &L, int v) {
  const CPullVariant &C = cpull_variant(v);
  for (BoxDev &B : L.boxes) fit_tile(B.nx, B.ny, C.tx, C.ty, C.k->nt, 0, 0, C.k->r1, B.cs);
  if (!L.cchunk[v]) L.cchunk[v] = fit_chunk(L, true, C.zc, C.k->nt, 2.0);
  build_tiles(L, L.cchunk[v], 1, L.zedge ? 3 : 0, L.ccol_tiles, L.nccol_plain, true);
}

// Column table of fused variant v.  Its stencils reach three nodes around
// the column, and its march three slabs beyond the chunk, plus the slabs its
// loads run ahead (five below the chunk).
void build_columns(Layout &L, int v) {
  const FusedVariant &F = fused_variant(v);
  for (BoxDev &B : L.boxes)
    fit_tile(B.nx, B.ny, F.tx, F.ty, F.k->nt, F.k->r3, F.k->r2, F.k->r1, B.fs);
  if (!L.fchunk[v]) L.fchunk[v] = fit_chunk(L, false, F.zc, F.k->nt, 3.0);
  build_tiles(L, L.fchunk[v], 4, L.zedge ? 6 : 0, L.col_tiles, L.ncol_plain, false);
  L.ncol = (int32_t)L.col_tiles.size();
  double all = 0.0, near = 0.0;
  for (int32_t k = 0; k < L.ncol; ++k) {
    const TileEntry &e = L.col_tiles[(size_t)k];
    if (e.box < 0) continue;
    all += e.z1 - e.z0;
    if (k >= L.ncol_plain && (L.boxes[(size_t)e.box].walls & 1u)) near += e.z1 - e.z0;
  }
  L.near_y = near / all;
}

// Tile table of the D2Q9 step kernel for variant v (kept in the column
// table's place): per box tile0, tnx, tny, ftx.
void build_tiles2(Layout &L, int v) {
  const Variant2 &V = variant2(v);
  L.col_box.clear();
  int32_t tile = 0;
  for (size_t b = 0; b < L.boxes.size(); ++b) {
    BoxDev &B = L.boxes[b];
    B.tile0 = tile;
    B.tnx = (B.nx + V.tx - 1) / V.tx;
    B.tny = (B.ny + V.ty - 1) / V.ty;
    B.ftx = make_fastdiv((uint32_t)B.tnx);
    const int32_t nt = B.tnx * B.tny;
    for (int32_t k = 0; k < nt; ++k) L.col_box.push_back((int32_t)b);
    tile += nt;
  }
  L.ncol = (int32_t)align_up(tile, 8);
  while ((int32_t)L.col_box.size() < L.ncol) L.col_box.push_back(-1);
}

// Host check of the division helper on the values a box can produce.
bool fastdiv_ok(uint32_t d, uint32_t nmax) {
  FastDiv f = make_fastdiv(d);
  const uint32_t probes[] = {0u, 1u, d - 1, d, d + 1, 2 * d - 1, 2 * d, nmax / 2, nmax - 1, nmax};
  for (uint32_t n : probes)
    if (n <= nmax && fdiv(n, f) != n / d) return false;
  for (uint32_t k = 0; k < 4096; ++k) {
    uint32_t n = (uint32_t)(((uint64_t)k * 2654435761u) % ((uint64_t)nmax + 1));
    if (fdiv(n, f) != n / d) return false;
  }
  return true;
}

}  // namespace

struct cglbm_handle {
  int32_t n_boxes = 0;
  std::vector<cglbm_box_params> params;
  Layout L;
  int32_t storage = CGLBM_FP32;
  void *pop[2] = {nullptr, nullptr};
  float *aux = nullptr;
  int cur = 0;  // buffer holding the stored (post-collision) state
  bool inplace = false;          // pop[0] == pop[1]: one population buffer
  void *stash = nullptr;         // in-place layouts with walls: solid nodes' populations
  int32_t *d_wblk_box = nullptr;
  TileEntry *d_ccol_tiles = nullptr;  // k_cpull blocks
  void *cstash[2] = {nullptr, nullptr};  // compact schedule with walls: solid nodes' populations
  size_t ccol_cap = 0;             // capacity of d_ccol_tiles (entries)
  int32_t cvariant = 0;            // k_cpull geometry
  int device = 0;
  BoxDev *d_boxes = nullptr;
  int32_t *d_blk_box = nullptr;
  int32_t *d_tile_box = nullptr;
  int32_t *d_col_box = nullptr;       // D2Q9 tiles
  TileEntry *d_col_tiles = nullptr;    // D3Q27 k_fused blocks
  size_t col_tiles_cap = 0;            // capacity of d_col_tiles (entries)
  int32_t schedule = 0;        // 0 fused, 1 three kernels (D3Q27)
  int32_t lattice = LATTICE_D3Q27;
  int32_t variant = 0;         // fused launch geometry (its column table is loaded)
  int32_t fvar_pop = 0;        // fused geometry for schedules 0 and 1
  int32_t fvar_compact = 0;    // fused geometry for schedule 2
  // wall mode (boxes with walls): bit 0 short z-edge chunks (Layout::zedge),
  // bit 1 the launches over tiles near walls on the side stream; the current
  // one and the autotuner's choices per schedule
  int32_t wmode = 3, wmode_pop = 3, wmode_compact = 3;
  size_t col_cap = 0;          // capacity of d_col_box (entries)
  int32_t *d_rch_box = nullptr;  // reduction chunk -> box
  double *d_part = nullptr;    // chunk partials of the reduction (kNPart doubles each)
  double *d_diag = nullptr;    // per box kNPart doubles
  double *d_centre = nullptr;  // per box 3 doubles
  double *d_out = nullptr;     // per box CGLBM_NDIAG doubles (host-output reduce)
  // time steps as a captured graph: two steps from each buffer parity
  int32_t use_graph = 1;
  hipStream_t cap_stream = nullptr;
  // the launch over the tiles near walls runs on `side`, beside the one over
  // the other tiles on the caller's stream (fork and join by events)
  hipStream_t side = nullptr;
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  hipGraphExec_t graphc[2] = {nullptr, nullptr};  // compact schedule: two inner steps
  std::vector<hipGraphExec_t> retired;  // dropped graphs whose replays may be pending
  // compact schedule with the state resident between calls
  // (cglbm_set_resident): clive is set while the other population buffer
  // holds the compact state of the last step and the state buffer is stale;
  // cwi is the wall stash that step wrote, cstream the stream it ran on
  bool resident = false, clive = false;
  // population buffer whose padding the compact schedule's arrays have
  // overwritten (-1: neither); zeroed before a step may make it the state
  int pad_dirty = -1;
  bool pad_replayed = false;  // a caller's graph holds such writes: never clean for good
  int32_t cwi = 0;
  hipStream_t cstream = nullptr;
  // profiling
  bool prof = false;
  std::vector<hipEvent_t> ev;
  std::vector<int> ev_kind;
  size_t ev_used = 0;
};

namespace {

// The pull (bounce != 0: with the bounce-back writes of a time step).  In
// place, the solid nodes' reversed populations go to the stash and
// k_wall_copy moves them into the buffer after the pull has completed.
int launch_pull(cglbm_handle *h, hipStream_t s, int bounce) {
  void *stash = bounce && h->stash ? h->stash : nullptr;
  hipLaunchKernelGGL(kPull[stash ? 1 : 0][h->storage], dim3(h->L.nblk_pad), dim3(kBlock), 0, s,
                     h->d_boxes,
                     h->d_blk_box, h->pop[h->cur], h->pop[1 - h->cur], h->aux, h->L.total,
                     bounce, stash, h->L.wtotal, (int64_t)0);
  if (stash && !h->L.wblk_box.empty())
    hipLaunchKernelGGL(kWallCopy[h->storage], dim3((unsigned)h->L.wblk_box.size()), dim3(kBlock),
                       0, s, h->d_boxes, h->d_wblk_box, (const void *)stash, h->pop[1 - h->cur],
                       h->L.total, h->L.wtotal);
  return CGLBM_OK;
}

int launch_fused(cglbm_handle *h, hipStream_t s, uint32_t need);

// Interface fields of every node into aux (those in `need` at least): the
// tiled kernel, or from kIfaceNodes nodes on the fused kernel's field export
// (the same bits), whose columns share their halos along z.  Measured, the
// kernels: 64x64x64 21 us against 45, 97x80x113 61 against 75, 200x180x160 283
// against 188; a step of the three-kernel schedule: 64 boxes of 32^3 330 us
// against 292, 300 of 20^3 489 and 413, 24 of 24 to 128 nodes an edge 1980 and
// 1740.  The export's kernel with wall logic takes a select per stencil point
// for rows in solid layers: with more than a quarter of the slabs near those of
// y walls the tiled kernel stays (near share 0.14: 2341 against 1962 us,
// 0.21: 639 and 587, 0.27: 301 and 340, 0.39: 323 and 371, 0.67: 416 and 458,
// 1.0: 328 and 364; z walls alone: 394 and 380, 418 and 393).
constexpr int64_t kIfaceNodes = 2 << 20;
bool iface_fused(const Layout &L) { return L.total >= kIfaceNodes && L.near_y <= 0.25; }
int launch_iface(cglbm_handle *h, hipStream_t s, uint32_t need = NEED_N | NEED_F | NEED_Q) {
  if (iface_fused(h->L)) return launch_fused(h, s, need);
  hipLaunchKernelGGL(kIfaceTiles[h->L.itile].fn, dim3(h->L.ntile),
                     dim3(kIfaceThreads), 0, s, h->d_boxes, h->d_tile_box, h->aux, h->L.total,
                     (int)(need & NEED_KAPPA));
  return CGLBM_OK;
}

int fork_side(cglbm_handle *h, hipStream_t s) {
  HIP_TRY(hipEventRecord(h->fork_ev, s));
  HIP_TRY(hipStreamWaitEvent(h->side, h->fork_ev, 0));
  return CGLBM_OK;
}
int join_side(cglbm_handle *h, hipStream_t s) {
  HIP_TRY(hipEventRecord(h->join_ev, h->side));
  HIP_TRY(hipStreamWaitEvent(s, h->join_ev, 0));
  return CGLBM_OK;
}

// The fused kernel over the tiles near walls (fn[1], the column entries
// after the first `nplain`), then over the others (fn[0]).  Both lists
// non-empty and bit 1 of the wall mode set: the first goes to the handle's
// side stream, which waits for everything before it on s, and s waits for it
// afterwards (also under graph capture, where the events become the graph's
// dependencies).
int launch_split(cglbm_handle *h, int32_t ncol, int32_t nplain, const FusedFn *fn, int nthreads,
                 hipStream_t s, const BoxDev *boxes, const TileEntry *cols, float *aux,
                 void *dst, int64_t plane, uint32_t need = 0) {
  const int32_t n[2] = {nplain, ncol - nplain};
  const bool both = (h->wmode & 2) && n[0] > 0 && n[1] > 0;
  if (both) {
    const int rc = fork_side(h, s);
    if (rc) return rc;
  }
  for (int w = 1; w >= 0; --w) {
    if (n[w] <= 0) continue;
    const TileEntry *c = cols + (w ? nplain : 0);
    void *args[] = {(void *)&boxes, (void *)&c, (void *)&aux, (void *)&dst, (void *)&plane,
                    (void *)&need};
    HIP_TRY(hipLaunchKernel((const void *)fn[w], dim3((unsigned)n[w]), dim3(nthreads), args, 0,
                            (both && w) ? h->side : s));
  }
  return both ? join_side(h, s) : CGLBM_OK;
}

// Compact schedule: the fused kernel writes the compact state into the
// other population buffer; k_cpull turns it into the moments of the next
// step; k_emit stores it as populations in the state buffer.
int launch_fused_compact(cglbm_handle *h, hipStream_t s) {
  h->pad_dirty = 1 - h->cur;
  const FusedVariant &F = fused_variant(h->variant);
  const BoxDev *boxes = h->d_boxes;
  const TileEntry *cols = h->d_col_tiles;
  float *aux = h->aux;
  void *dst = h->pop[1 - h->cur];
  int64_t plane = h->L.ctotal;
  const FusedFn *fn = storage_exact(h->storage) ? F.k->fcx : F.k->fc;
  return launch_split(h, h->L.ncol, h->L.ncol_plain, fn, F.k->nt, s, boxes, cols, aux, dst,
                      plane);
}
// rd: the wall stash this step's solid points emit from; the arrivals at
// solid nodes go to the other one
int launch_cpull(cglbm_handle *h, hipStream_t s, int rd = 0) {
  const CPullVariant &C = cpull_variant(h->cvariant);
  const bool x = storage_exact(h->storage);
  const int g = h->L.general ? 1 : 0;
  // the tiles away from walls, then those near them
  const CPullFn fn[2] = {x ? C.k->fx[0] : C.k->fn[g][0],
                         x ? C.k->fx[1] : C.k->fn[g][h->storage == CGLBM_FP32_PAIRS ? 2 : 1]};
  const int32_t n[2] = {h->L.nccol_plain, (int32_t)h->L.ccol_tiles.size() - h->L.nccol_plain};
  const bool both = (h->wmode & 2) && n[0] > 0 && n[1] > 0;
  if (both) {
    const int rc = fork_side(h, s);
    if (rc) return rc;
  }
  for (int w = 1; w >= 0; --w)
    if (n[w] > 0)
      hipLaunchKernelGGL(fn[w], dim3((unsigned)n[w]), dim3((unsigned)C.k->nt), 0,
                         (both && w) ? h->side : s, h->d_boxes, h->d_ccol_tiles + (w ? n[0] : 0),
                         (const float *)h->pop[1 - h->cur], h->aux, h->L.ctotal,
                         (const void *)h->cstash[rd], h->cstash[1 - rd], h->L.wtotal);
  return both ? join_side(h, s) : CGLBM_OK;
}
// wi: the wall stash the last step wrote (the solid nodes' stored values)
int launch_emit(cglbm_handle *h, hipStream_t s, int wi = 0) {
  hipLaunchKernelGGL(storage_exact(h->storage)
                         ? kEmitX[h->storage]
                         : kEmit[h->storage == CGLBM_FP32_PAIRS ? 1 : 0][h->L.general ? 1 : 0],
                     dim3(h->L.nblk_pad), dim3(kBlock), 0, s, h->d_boxes, h->d_blk_box,
                     (const float *)h->pop[1 - h->cur], h->pop[h->cur], h->L.total, h->L.ctotal);
  if (h->L.walls && !h->L.wblk_box.empty())
    hipLaunchKernelGGL(storage_16bit(h->storage) ? kWallEncode[h->storage]
                                                 : kWallCopy[h->storage],
                       dim3((unsigned)h->L.wblk_box.size()), dim3(kBlock),
                       0, s, h->d_boxes, h->d_wblk_box, (const void *)h->cstash[wi],
                       h->pop[h->cur], h->L.total, h->L.wtotal);
  return CGLBM_OK;
}
// The first step of a compact call: the population pull, with the solid
// nodes' reversed populations going to wall stash 0 (decoded to the
// mass-exact FP32 format for the 16-bit storages).
int launch_pull_compact(cglbm_handle *h, hipStream_t s) {
  void *stash = h->L.walls ? h->cstash[0] : nullptr;
  hipLaunchKernelGGL(kPullFirst[stash ? 1 : 0][h->storage], dim3(h->L.nblk_pad), dim3(kBlock), 0, s,
                     h->d_boxes, h->d_blk_box, h->pop[h->cur], h->pop[1 - h->cur], h->aux,
                     h->L.total, 1, stash, h->L.wtotal, h->L.ctotal);
  return CGLBM_OK;
}
// Layouts the compact schedule serves: D3Q27, FP32 storage (either layout,
// any equilibrium family), or a mass-exact storage (FP32 or 16-bit; Model D
// with Q), two buffers, unit higher rates.  With a 16-bit storage the
// compact state (15 floats and the FP64 colour densities, 76 bytes a node)
// fits the other population buffer (at least 120 bytes a node).
bool compact_ok(const cglbm_handle *h) {
  return h->lattice == LATTICE_D3Q27 && !h->inplace && !h->L.full_rates &&
         (h->storage == CGLBM_FP32 || h->storage == CGLBM_FP32_PAIRS ||
          (storage_exact(h->storage) && !h->L.general));
}

// need == 0: interface stencils + collision of a time step; else the interface
// fields in `need` into aux, populations untouched.
int launch_fused(cglbm_handle *h, hipStream_t s, uint32_t need) {
  const FusedVariant &F = fused_variant(h->variant);
  const BoxDev *boxes = h->d_boxes;
  const TileEntry *cols = h->d_col_tiles;
  float *aux = h->aux;
  void *dst = h->pop[1 - h->cur];
  int64_t plane = h->L.total;
  const FusedFn *fn = need ? F.k->fx : F.k->fn[h->L.ragged ? 1 : 0][h->storage];
  return launch_split(h, h->L.ncol, h->L.ncol_plain, fn, F.k->nt, s, boxes, cols, aux, dst,
                      plane, need);
}

// Graphs captured under another geometry, mode or schedule are not replayed
// again.  Their last replays may still be running, on whatever stream the
// caller stepped on: they are destroyed only once the device has been waited
// for (destroy_retired), not here, where a caller expects no wait.
void drop_graphs(cglbm_handle *h) {
  for (hipGraphExec_t *g : {&h->graph[0], &h->graph[1], &h->graphc[0], &h->graphc[1]})
    if (*g) {
      h->retired.push_back(*g);
      *g = nullptr;
    }
}

// Wait for all work on the handle's device.
hipError_t wait_device(const cglbm_handle *h) {
  int now = h->device;
  (void)hipGetDevice(&now);
  if (now != h->device) (void)hipSetDevice(h->device);
  const hipError_t e = hipDeviceSynchronize();
  if (now != h->device) (void)hipSetDevice(now);
  return e;
}

int destroy_retired(cglbm_handle *h) {
  if (h->retired.empty()) return CGLBM_OK;
  HIP_TRY(wait_device(h));
  for (hipGraphExec_t g : h->retired) (void)hipGraphExecDestroy(g);
  h->retired.clear();
  return CGLBM_OK;
}

// Before a capture: a program that switches schedules back and forth leaves no
// more than a few graphs behind.
int bound_retired(cglbm_handle *h) {
  return h->retired.size() > 8 ? destroy_retired(h) : CGLBM_OK;
}

// Select k_cpull variant v: rebuild and upload its column table.
int select_cvariant(cglbm_handle *h, int v, hipStream_t s) {
  drop_graphs(h);
  if (const int rc = destroy_retired(h)) return rc;
  build_ccolumns(h->L, v);
  for (const BoxDev &B : h->L.boxes)
    if (!fastdiv_ok((uint32_t)B.cncx, 1u << 20) || !fastdiv_ok((uint32_t)B.cncy, 1u << 20))
      return fail(CGLBM_EINVAL, "index division self-check failed");
  if (h->L.ccol_tiles.size() > h->ccol_cap) {
    if (h->d_ccol_tiles) HIP_TRY(hipFree(h->d_ccol_tiles));
    h->d_ccol_tiles = nullptr;
    HIP_TRY(hipMalloc(&h->d_ccol_tiles, sizeof(TileEntry) * h->L.ccol_tiles.size()));
    h->ccol_cap = h->L.ccol_tiles.size();
  }
  HIP_TRY(hipMemcpyAsync(h->d_ccol_tiles, h->L.ccol_tiles.data(),
                         sizeof(TileEntry) * h->L.ccol_tiles.size(), hipMemcpyHostToDevice, s));
  HIP_TRY(hipMemcpyAsync(h->d_boxes, h->L.boxes.data(), sizeof(BoxDev) * h->L.boxes.size(),
                         hipMemcpyHostToDevice, s));
  HIP_TRY(hipStreamSynchronize(s));
  h->cvariant = v;
  return CGLBM_OK;
}

// Select fused variant v: rebuild and upload the column tables.
int select_variant(cglbm_handle *h, int v, hipStream_t s) {
  drop_graphs(h);
  if (const int rc = destroy_retired(h)) return rc;
  if (h->lattice == LATTICE_D2Q9) {
    build_tiles2(h->L, v);
    for (const BoxDev &B : h->L.boxes)
      if (!fastdiv_ok((uint32_t)B.tnx, (uint32_t)(B.tnx * B.tny)))
        return fail(CGLBM_EINVAL, "index division self-check failed");
    if (h->L.col_box.size() > h->col_cap) {
      if (h->d_col_box) HIP_TRY(hipFree(h->d_col_box));
      h->d_col_box = nullptr;
      HIP_TRY(hipMalloc(&h->d_col_box, sizeof(int32_t) * h->L.col_box.size()));
      h->col_cap = h->L.col_box.size();
    }
    HIP_TRY(hipMemcpyAsync(h->d_col_box, h->L.col_box.data(),
                           sizeof(int32_t) * h->L.col_box.size(), hipMemcpyHostToDevice, s));
  } else {
    build_columns(h->L, v);
    if (h->L.col_tiles.size() > h->col_tiles_cap) {
      if (h->d_col_tiles) HIP_TRY(hipFree(h->d_col_tiles));
      h->d_col_tiles = nullptr;
      HIP_TRY(hipMalloc(&h->d_col_tiles, sizeof(TileEntry) * h->L.col_tiles.size()));
      h->col_tiles_cap = h->L.col_tiles.size();
    }
    HIP_TRY(hipMemcpyAsync(h->d_col_tiles, h->L.col_tiles.data(),
                           sizeof(TileEntry) * h->L.col_tiles.size(), hipMemcpyHostToDevice, s));
  }
  HIP_TRY(hipMemcpyAsync(h->d_boxes, h->L.boxes.data(), sizeof(BoxDev) * h->L.boxes.size(),
                         hipMemcpyHostToDevice, s));
  // pageable host sources: make sure the copies completed before the vectors change
  HIP_TRY(hipStreamSynchronize(s));
  h->variant = v;
  return CGLBM_OK;
}

// Fused variant v under wall mode m: rebuild the tile lists whose chunking
// changes (the k_cpull list too); graphs captured under another mode are
// dropped.
int select_mode(cglbm_handle *h, int v, int32_t m, hipStream_t s) {
  const bool zedge = (m & 1) != 0, rebuild_c = zedge != h->L.zedge;
  if (m != h->wmode) drop_graphs(h);
  h->wmode = m;
  h->L.zedge = zedge;
  int rc = select_variant(h, v, s);
  if (!rc && rebuild_c) rc = select_cvariant(h, h->cvariant, s);
  return rc;
}

int launch_collide(cglbm_handle *h, hipStream_t s) {
  hipLaunchKernelGGL(kCollide[h->storage], dim3(h->L.nblk_pad), dim3(kBlock), 0, s, h->d_boxes,
                     h->d_blk_box, h->aux, (const void *)h->pop[h->cur], h->pop[1 - h->cur],
                     h->L.total);
  return CGLBM_OK;
}

template <class F>
int timed(cglbm_handle *h, hipStream_t s, int kind, F &&launch) {
  if (h->prof && h->ev_used + 2 <= h->ev.size()) {
    HIP_TRY(hipEventRecord(h->ev[h->ev_used], s));
    int rc = launch();
    HIP_TRY(hipEventRecord(h->ev[h->ev_used + 1], s));
    h->ev_kind[h->ev_used / 2] = kind;
    h->ev_used += 2;
    return rc;
  }
  return launch();
}

// The caller is capturing stream s (the null stream cannot be captured).
bool capturing(hipStream_t s) {
  if (!s) return false;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &st) == hipSuccess && st != hipStreamCaptureStatusNone;
}

int check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CGLBM_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
  return CGLBM_OK;
}

// Local moments and interface fields of the current state into aux.
// The fused kernel implements Model D with the correction term; layouts with
// any other box run the three-kernel schedule, whose collision takes each
// box's equilibrium family and correction switch.
int effective_schedule(const cglbm_handle *h) {
  if (h->schedule == 2) return 2;  // set only where compact_ok holds
  return h->L.general ? 1 : h->schedule;
}

// D2Q9: one launch of the step kernel (export != 0: the fields of the
// stored state into aux, populations untouched).
int launch_step2(cglbm_handle *h, hipStream_t s, int export_fields) {
  const Variant2 &V = variant2(h->variant);
  const int slot = storage2_slot(h->storage);
  hipLaunchKernelGGL(export_fields ? V.fields[slot] : V.step[h->L.ragged ? 1 : 0][slot], dim3(h->L.ncol), dim3(256), 0,
                     s, h->d_boxes, h->d_col_box, (const void *)h->pop[h->cur],
                     h->pop[1 - h->cur], h->aux, h->L.total);
  return CGLBM_OK;
}

// One time step on stream s (launches only); flips the buffer parity.
int launch_step(cglbm_handle *h, hipStream_t s) {
  if (h->lattice == LATTICE_D2Q9) {
    int rc = timed(h, s, KIND_FUSED, [&] { return launch_step2(h, s, 0); });
    if (!rc) rc = check_launch();
    if (!rc) h->cur = 1 - h->cur;
    return rc;
  }
  int rc = timed(h, s, KIND_PULL, [&] { return launch_pull(h, s, 1); });
  if (effective_schedule(h) == 0) {
    if (!rc) rc = timed(h, s, KIND_FUSED, [&] { return launch_fused(h, s, 0); });
  } else {
    if (!rc) rc = timed(h, s, KIND_IFACE, [&] { return launch_iface(h, s); });
    if (!rc) rc = timed(h, s, KIND_COLLIDE, [&] { return launch_collide(h, s); });
  }
  if (!rc) rc = check_launch();
  if (!rc) h->cur = 1 - h->cur;
  return rc;
}

// n steps of the compact schedule (launches only).  The state between calls
// stays in stored populations: the first step pulls them, the last converts
// the compact state back, and the state buffer parity is unchanged.
int capture_compact_pair(cglbm_handle *h) {
  if (const int rc = bound_retired(h)) return rc;
  if (!h->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
  HIP_TRY(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal));
  int rc = CGLBM_OK;
  for (int k = 0; k < 2 && !rc; ++k) {
    rc = launch_cpull(h, h->cap_stream, k);
    if (!rc) rc = launch_fused_compact(h, h->cap_stream);
  }
  hipGraph_t g = nullptr;
  const hipError_t e = hipStreamEndCapture(h->cap_stream, &g);
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return fail(CGLBM_EHIP, "graph capture: %s", hipGetErrorString(e));
  const hipError_t ei = hipGraphInstantiate(&h->graphc[h->cur], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ei != hipSuccess) {
    h->graphc[h->cur] = nullptr;
    return fail(CGLBM_EHIP, "graph instantiate: %s", hipGetErrorString(ei));
  }
  return CGLBM_OK;
}

// Milliseconds of launch() over `reps` runs of before() and launch() on stream
// s, after one of each untimed; only launch() is timed.  The median is what
// candidates are compared by, the mean what callers are told.
struct Timing {
  double median = 0.0, mean = 0.0;
};
template <class B, class F>
int time_in_step(hipStream_t s, int reps, B &&before, F &&launch, Timing &out) {
  const int kEvents = 64;  // pairs of events, used again after each 64 runs
  std::vector<hipEvent_t> ev(2 * (size_t)std::min(reps, kEvents), nullptr);
  std::vector<float> t;
  int rc = CGLBM_OK;
  for (hipEvent_t &e : ev)
    if (!rc && hipEventCreate(&e) != hipSuccess) rc = fail(CGLBM_EHIP, "autotune: event create failed");
  if (!rc) rc = before();
  if (!rc) rc = launch();
  for (int r0 = 0; r0 < reps && !rc; r0 += kEvents) {
    const int n = std::min(reps - r0, kEvents);
    for (int r = 0; r < n && !rc; ++r) {
      if ((rc = before())) break;
      (void)hipEventRecord(ev[2 * (size_t)r], s);
      rc = launch();
      (void)hipEventRecord(ev[2 * (size_t)r + 1], s);
    }
    if (!rc) rc = check_launch();
    if (!rc && hipEventSynchronize(ev[2 * (size_t)n - 1]) != hipSuccess)
      rc = fail(CGLBM_EHIP, "autotune: event synchronize failed");
    for (int r = 0; r < n && !rc; ++r) {
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, ev[2 * (size_t)r], ev[2 * (size_t)r + 1]);
      t.push_back(ms);
    }
  }
  for (hipEvent_t e : ev)
    if (e) (void)hipEventDestroy(e);
  if (rc) return rc;
  for (float ms : t) out.mean += (double)ms / reps;
  std::nth_element(t.begin(), t.begin() + (reps - 1) / 2, t.end());
  out.median = (double)t[(size_t)(reps - 1) / 2];
  return CGLBM_OK;
}

// The fastest of n candidates by time(v, reps, Timing): each over `first`
// launches, then those close to the best once more (medians of a few
// launches differ by 3 %, and most candidates are further off than that).
// ms_out (optional) receives the means of the first launches; best_ms the
// fastest's time.  (Candidates timed over all `reps` at first are looked at
// again over half as many.)
template <class T>
int fastest(int n, int first, int reps, T &&time, double *ms_out, int &best, double &best_ms) {
  std::vector<Timing> t((size_t)n);
  double limit = 1e300;
  for (int v = 0; v < n; ++v) {
    const int rc = time(v, first, t[(size_t)v]);
    if (rc) return rc;
    if (ms_out) ms_out[v] = t[(size_t)v].mean;
    limit = std::min(limit, (first < reps ? 1.08 : 1.04) * t[(size_t)v].median);
  }
  if (first == reps) reps = std::max(1, reps / 2);
  best_ms = 1e300;
  for (int v = 0; v < n; ++v) {
    if (!(t[(size_t)v].median <= limit)) continue;
    Timing again;
    const int rc = time(v, reps, again);
    if (rc) return rc;
    const double ms = (first * t[(size_t)v].median + reps * again.median) / (first + reps);
    if (ms < best_ms) {
      best_ms = ms;
      best = v;
    }
  }
  return CGLBM_OK;
}

// Resident compact state (cglbm_set_resident): store it as populations in the
// state buffer if the last call left it in compact form.  The next compact
// call then starts from the populations again.
int flush_compact(cglbm_handle *h, hipStream_t s) {
  if (!h->clive) return CGLBM_OK;
  h->clive = false;
  const int rc = timed(h, s, KIND_EMIT, [&] { return launch_emit(h, s, h->cwi); });
  return rc ? rc : check_launch();
}

int step_compact(cglbm_handle *h, int32_t n, hipStream_t s) {
  if (n == 0) return CGLBM_OK;
  if (!h->pad_replayed) h->pad_replayed = capturing(s);
  // wall stashes (boxes with solid layers): step k's solid points emit from
  // stash wi, its arrivals at solid nodes go to 1 - wi; the first step
  // (the population pull) writes stash 0
  int wi = 0;
  int rc = CGLBM_OK;
  int32_t k = 0;
  if (h->clive) {
    // resident: continue from the compact state of the last call, with one
    // direct step first if it left the stashes at odd parity (the captured
    // pair starts from stash 0)
    wi = h->cwi;
    h->clive = false;
    if (wi == 1) {
      rc = timed(h, s, KIND_PULL, [&] { return launch_cpull(h, s, 1); });
      if (!rc) rc = timed(h, s, KIND_FUSED, [&] { return launch_fused_compact(h, s); });
      wi = 0;
      k = 1;
    }
  } else {
    rc = timed(h, s, KIND_PULL_FIRST, [&] { return launch_pull_compact(h, s); });
    if (!rc) rc = timed(h, s, KIND_FUSED, [&] { return launch_fused_compact(h, s); });
    k = 1;
  }
  if (!rc && h->use_graph && !h->prof && n - k >= 2) {
    if (!h->graphc[h->cur]) rc = capture_compact_pair(h);
    for (; !rc && k + 1 < n; k += 2) HIP_TRY(hipGraphLaunch(h->graphc[h->cur], s));
  }
  for (; k < n && !rc; ++k) {
    rc = timed(h, s, KIND_PULL, [&] { return launch_cpull(h, s, wi); });
    if (!rc) rc = timed(h, s, KIND_FUSED, [&] { return launch_fused_compact(h, s); });
    wi = 1 - wi;
  }
  if (rc) return rc;
  if (h->resident) {
    h->clive = true;
    h->cwi = wi;
    h->cstream = s;
  } else {
    rc = timed(h, s, KIND_EMIT, [&] { return launch_emit(h, s, wi); });
  }
  if (!rc) rc = check_launch();
  return rc;
}

// Capture two steps from the current parity (which they restore) on the
// handle's private stream and instantiate them as an executable graph.
int capture_pair(cglbm_handle *h) {
  if (const int rc = bound_retired(h)) return rc;
  if (!h->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
  const int c0 = h->cur;
  HIP_TRY(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal));
  int rc = launch_step(h, h->cap_stream);
  if (!rc) rc = launch_step(h, h->cap_stream);
  hipGraph_t g = nullptr;
  const hipError_t e = hipStreamEndCapture(h->cap_stream, &g);
  h->cur = c0;
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return fail(CGLBM_EHIP, "graph capture: %s", hipGetErrorString(e));
  const hipError_t ei = hipGraphInstantiate(&h->graph[c0], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ei != hipSuccess) {
    h->graph[c0] = nullptr;
    return fail(CGLBM_EHIP, "graph instantiate: %s", hipGetErrorString(ei));
  }
  return CGLBM_OK;
}

// need: the interface fields wanted (NEED_*; others may be written too).
int compute_fields(cglbm_handle *h, hipStream_t s, uint32_t need) {
  if (h->clive) {
    const int rc = flush_compact(h, s);
    if (rc) return rc;
  }
  if (h->lattice == LATTICE_D2Q9) {
    const int rc = launch_step2(h, s, 1);
    return rc ? rc : check_launch();
  }
  int rc = launch_pull(h, s, 0);
  if (rc) return rc;
  if (!need) return check_launch();
  rc = effective_schedule(h) != 1 ? launch_fused(h, s, need) : launch_iface(h, s, need);
  if (rc) return rc;
  return check_launch();
}

// Device address of this GPU's copy of `scratch`, looked up once per device
// with that device current (the caller's).
int scratch_lookup(int device) {
  if (device < 0 || device >= kMaxDevices)
    return fail(CGLBM_EUNSUPPORTED, "device %d beyond the library's %d", device, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[device]) return CGLBM_OK;
  void *ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr)
    return fail(CGLBM_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
  g_scratch[device] = (double *)ptr;
  return CGLBM_OK;
}

// The diagnostics of the current state: local moments and interface fields
// into aux, then the two chunked passes and the per-box finals (launches
// only).  centre: device array of 3 doubles per box, or NULL for the box
// centres; part: room for one partial per reduction chunk; diag: kNPart
// doubles per box; out: the packed CGLBM_NDIAG doubles per box, device.
int reduce_launch(cglbm_handle *h, hipStream_t s, const double *centre, double *part,
                  double *diag, double *out) {
  int rc = compute_fields(h, s, NEED_F);
  if (rc) return rc;
  const double *rho64 =
      storage_exact(h->storage)
          ? (const double *)((const char *)h->aux + align256((int64_t)A_COUNT * h->L.total * 4))
          : nullptr;
  const unsigned nch = (unsigned)h->L.rch_box.size();
  hipLaunchKernelGGL(k_reduce1, dim3(nch), dim3(kBlock), 0, s, h->d_boxes, h->d_rch_box, h->aux,
                     h->L.total, rho64, centre, part);
  hipLaunchKernelGGL(k_reduce_final, dim3(h->n_boxes), dim3(kBlock), 0, s, h->d_boxes,
                     (const double *)part, 1, diag, (double *)nullptr);
  hipLaunchKernelGGL(k_reduce2, dim3(nch), dim3(kBlock), 0, s, h->d_boxes, h->d_rch_box, h->aux,
                     h->L.total, centre, (const double *)diag, part);
  hipLaunchKernelGGL(k_reduce_final, dim3(h->n_boxes), dim3(kBlock), 0, s, h->d_boxes,
                     (const double *)part, 2, diag, out);
  return check_launch();
}

// D2Q9: time every tile variant of the step kernel on the same stored state
// (the kernel reads one buffer and writes the other, so repeated launches
// are idempotent) and keep the fastest.
int autotune2(cglbm_handle *h, int32_t reps, double *ms_per_variant, hipStream_t s) {
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  int rc = CGLBM_OK, best = h->variant;
  double best_ms = 1e300;
  for (int v = 0; v < kNumV2 && !rc; ++v) {
    if ((rc = select_variant(h, v, s)) || (rc = launch_step2(h, s, 0))) break;
    (void)hipEventRecord(e0, s);
    for (int r = 0; r < reps && !rc; ++r) rc = launch_step2(h, s, 0);
    (void)hipEventRecord(e1, s);
    if (rc || (rc = check_launch())) break;
    if (hipEventSynchronize(e1) != hipSuccess) {
      rc = fail(CGLBM_EHIP, "autotune: event synchronize failed");
      break;
    }
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    const double avg = (double)ms / reps;
    if (ms_per_variant) ms_per_variant[v] = avg;
    if (avg < best_ms) {
      best_ms = avg;
      best = v;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) return rc;
  return select_variant(h, best, s);
}

}  // namespace

extern "C" {

const char *cglbm_last_error(void) { return g_err.c_str(); }

const char *cglbm_version(void) { return "cglbm-gfx950 0.1"; }

}  // extern "C"

namespace {

int query_sizes(int lattice, int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage,
                size_t *pop_bytes, size_t *aux_bytes, int64_t *total_nodes) {
  g_err.clear();
  int rc = lattice == LATTICE_D2Q9 ? validate_d2q9(n_boxes, boxes, storage)
                                   : validate(n_boxes, boxes, storage);
  if (rc) return rc;
  Layout L;
  build_layout(n_boxes, boxes, storage, L, lattice);
  size_t pb, ab;
  buffer_sizes(storage, L.total, &pb, &ab, lattice);
  if (pop_bytes) *pop_bytes = pb;
  if (aux_bytes) *aux_bytes = ab;
  if (total_nodes) *total_nodes = L.total;
  return CGLBM_OK;
}

int init_handle(int lattice, cglbm_handle **out, int32_t n_boxes, const cglbm_box_params *boxes,
                int32_t storage, void *pop_a, void *pop_b, void *aux, const float *init_rho_r,
                const float *init_rho_b, const float *init_u, uint64_t noise_seed,
                double noise_amp, void *stream);

}  // namespace

extern "C" {

int cglbm_query_sizes(int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage,
                      size_t *pop_bytes, size_t *aux_bytes, int64_t *total_nodes) {
  return query_sizes(LATTICE_D3Q27, n_boxes, boxes, storage, pop_bytes, aux_bytes, total_nodes);
}

int cglbm_query_sizes_d2q9(int32_t n_boxes, const cglbm_box_params *boxes, int32_t storage,
                           size_t *pop_bytes, size_t *aux_bytes, int64_t *total_nodes) {
  return query_sizes(LATTICE_D2Q9, n_boxes, boxes, storage, pop_bytes, aux_bytes, total_nodes);
}

int cglbm_init(cglbm_handle **out, int32_t n_boxes, const cglbm_box_params *boxes,
               int32_t storage, void *pop_a, void *pop_b, void *aux, const float *init_rho_r,
               const float *init_rho_b, const float *init_u, uint64_t noise_seed,
               double noise_amp, void *stream) {
  return init_handle(LATTICE_D3Q27, out, n_boxes, boxes, storage, pop_a, pop_b, aux, init_rho_r,
                     init_rho_b, init_u, noise_seed, noise_amp, stream);
}

int cglbm_init_d2q9(cglbm_handle **out, int32_t n_boxes, const cglbm_box_params *boxes,
                    int32_t storage, void *pop_a, void *pop_b, void *aux, const float *init_rho_r,
                    const float *init_rho_b, const float *init_u, uint64_t noise_seed,
                    double noise_amp, void *stream) {
  return init_handle(LATTICE_D2Q9, out, n_boxes, boxes, storage, pop_a, pop_b, aux, init_rho_r,
                     init_rho_b, init_u, noise_seed, noise_amp, stream);
}

int cglbm_lattice(const cglbm_handle *h) { return h ? h->lattice : -1; }

int64_t cglbm_box_offset(const cglbm_handle *h, int32_t box) {
  if (!h || box < 0 || box >= h->n_boxes) return -1;
  return h->L.boxes[box].base;
}

void *cglbm_state_buffer(const cglbm_handle *h) { return h ? h->pop[h->cur] : nullptr; }

int cglbm_load_state(cglbm_handle *h, const void *src, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (!src) return fail(CGLBM_EINVAL, "src must not be NULL");
  size_t pop = 0, aux = 0;
  buffer_sizes(h->storage, h->L.total, &pop, &aux, h->lattice);
  h->clive = false;  // a resident compact state is replaced by the loaded one
  if (src == h->pop[h->cur]) return CGLBM_OK;
  HIP_TRY(hipMemcpyAsync(h->pop[h->cur], src, pop, hipMemcpyDeviceToDevice, (hipStream_t)stream));
  return CGLBM_OK;
}

}  // extern "C"

namespace {

int init_handle(int lattice, cglbm_handle **out, int32_t n_boxes, const cglbm_box_params *boxes,
                int32_t storage, void *pop_a, void *pop_b, void *aux, const float *init_rho_r,
                const float *init_rho_b, const float *init_u, uint64_t noise_seed,
                double noise_amp, void *stream) {
  g_err.clear();
  if (!out) return fail(CGLBM_EINVAL, "out must not be NULL");
  *out = nullptr;
  int rc = lattice == LATTICE_D2Q9 ? validate_d2q9(n_boxes, boxes, storage)
                                   : validate(n_boxes, boxes, storage);
  if (rc) return rc;
  if (!pop_a) return fail(CGLBM_EINVAL, "pop_a must not be NULL");
  if (pop_a == pop_b) return fail(CGLBM_EINVAL, "pop_a and pop_b must differ");
  const bool inplace = pop_b == nullptr;
  if (inplace) {
    // one buffer works where populations are read by the pull alone
    if (lattice == LATTICE_D2Q9)
      return fail(CGLBM_EUNSUPPORTED, "D2Q9 steps read and write populations in one kernel: pass pop_b");
    for (int b = 0; b < n_boxes; ++b)
      for (int k = 0; k < 9; ++k)
        if (boxes[b].omega_hi[k] != 1.0)
          return fail(CGLBM_EUNSUPPORTED,
                      "box %d: non-unit higher-order rates pull the populations again: pass pop_b", b);
  }
  if (!aux || !init_rho_r || !init_rho_b || !init_u)
    return fail(CGLBM_EINVAL, "aux and the initial fields must not be NULL");
  if (!std::isfinite(noise_amp) || noise_amp < 0.0)
    return fail(CGLBM_EINVAL, "noise_amp must be finite and >= 0");
  cglbm_handle *h = new cglbm_handle();
  h->n_boxes = n_boxes;
  h->params.assign(boxes, boxes + n_boxes);
  h->storage = storage;
  h->lattice = lattice;
  build_layout(n_boxes, boxes, storage, h->L, lattice);
  if (lattice == LATTICE_D3Q27) pad_rows(h->L, storage);
  build_ccolumns(h->L, 0);
  h->ccol_cap = h->L.ccol_tiles.size();
  for (const BoxDev &B : h->L.boxes) {
    if (!fastdiv_ok((uint32_t)B.nx, (uint32_t)B.n) || !fastdiv_ok((uint32_t)B.ny, (uint32_t)B.n) ||
        !fastdiv_ok((uint32_t)B.tnx, 1u << 20) || !fastdiv_ok((uint32_t)B.tny, 1u << 20) ||
        !fastdiv_ok((uint32_t)B.cncx, 1u << 20) || !fastdiv_ok((uint32_t)B.cncy, 1u << 20)) {
      delete h;
      return fail(CGLBM_EINVAL, "index division self-check failed");
    }
  }
  h->pop[0] = pop_a;
  h->pop[1] = inplace ? pop_a : pop_b;
  h->inplace = inplace;
  h->aux = (float *)aux;
  hipStream_t s = (hipStream_t)stream;
  auto cleanup = [&](int code) {
    cglbm_destroy(h);
    return code;
  };
  hipError_t e;
  if ((e = hipGetDevice(&h->device)) != hipSuccess ||
      (e = hipMalloc(&h->d_boxes, sizeof(BoxDev) * n_boxes)) != hipSuccess ||
      (e = hipMalloc(&h->d_blk_box, sizeof(int32_t) * h->L.blk_box.size())) != hipSuccess ||
      (e = hipMalloc(&h->d_tile_box, sizeof(int32_t) * h->L.tile_box.size())) != hipSuccess ||
      (e = hipMalloc(&h->d_rch_box, sizeof(int32_t) * h->L.rch_box.size())) != hipSuccess ||
      (e = hipMalloc(&h->d_part, sizeof(double) * kNPart * h->L.rch_box.size())) != hipSuccess ||
      (e = hipMalloc(&h->d_diag, sizeof(double) * kNPart * (size_t)n_boxes)) != hipSuccess ||
      (e = hipMalloc(&h->d_centre, sizeof(double) * 3 * (size_t)n_boxes)) != hipSuccess ||
      (e = hipMalloc(&h->d_out, sizeof(double) * CGLBM_NDIAG * (size_t)n_boxes)) != hipSuccess ||
      (e = hipMemcpyAsync(h->d_rch_box, h->L.rch_box.data(),
                          sizeof(int32_t) * h->L.rch_box.size(), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = hipMalloc(&h->d_ccol_tiles, sizeof(TileEntry) * h->L.ccol_tiles.size())) !=
          hipSuccess ||
      (e = hipMemcpyAsync(h->d_ccol_tiles, h->L.ccol_tiles.data(),
                          sizeof(TileEntry) * h->L.ccol_tiles.size(), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = hipMemcpyAsync(h->d_boxes, h->L.boxes.data(), sizeof(BoxDev) * n_boxes,
                          hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipMemcpyAsync(h->d_blk_box, h->L.blk_box.data(),
                          sizeof(int32_t) * h->L.blk_box.size(), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = hipMemcpyAsync(h->d_tile_box, h->L.tile_box.data(),
                          sizeof(int32_t) * h->L.tile_box.size(), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking)) != hipSuccess ||
      (e = hipEventCreateWithFlags(&h->fork_ev, hipEventDisableTiming)) != hipSuccess ||
      (e = hipEventCreateWithFlags(&h->join_ev, hipEventDisableTiming)) != hipSuccess) {
    return cleanup(fail(CGLBM_EHIP, "init: %s", hipGetErrorString(e)));
  }
  if ((rc = scratch_lookup(h->device))) return cleanup(rc);
  if (h->L.walls) {
    // wall stashes: the in-place layout's, or the compact schedule's pair
    // (the compact schedule of the 16-bit storages keeps its stashes in the
    // mass-exact FP32 format)
    size_t sb = 0, ab = 0, csb = 0;
    buffer_sizes(storage, h->L.wtotal, &sb, &ab, lattice);
    buffer_sizes(storage_16bit(storage) ? CGLBM_FP32_EXACT : storage, h->L.wtotal, &csb, &ab,
                 lattice);
    const bool cst = lattice == LATTICE_D3Q27 && !inplace;
    if ((e = hipMalloc(&h->d_wblk_box, sizeof(int32_t) * h->L.wblk_box.size())) != hipSuccess ||
        (e = hipMemcpyAsync(h->d_wblk_box, h->L.wblk_box.data(),
                            sizeof(int32_t) * h->L.wblk_box.size(), hipMemcpyHostToDevice, s)) !=
            hipSuccess ||
        (inplace && (e = hipMalloc(&h->stash, sb)) != hipSuccess) ||
        (cst && ((e = hipMalloc(&h->cstash[0], csb)) != hipSuccess ||
                 (e = hipMalloc(&h->cstash[1], csb)) != hipSuccess)))
      return cleanup(fail(CGLBM_EHIP, "init: %s", hipGetErrorString(e)));
  }
  if ((rc = select_variant(h, 0, s))) return cleanup(rc);
  // the stored state lives in pop[0]
  h->cur = 0;
  if (lattice == LATTICE_D2Q9)
    hipLaunchKernelGGL(kInit2[storage2_slot(storage)], dim3(h->L.nblk), dim3(kBlock), 0, s,
                       h->d_boxes, h->d_blk_box, init_rho_r, init_rho_b, init_u, h->pop[0],
                       h->L.total, noise_seed, (float)noise_amp);
  else
    hipLaunchKernelGGL(kInit[storage], dim3(h->L.nblk), dim3(kBlock), 0, s, h->d_boxes,
                       h->d_blk_box, init_rho_r, init_rho_b, init_u, h->pop[0], h->L.total,
                       noise_seed, (float)noise_amp);
  if ((rc = check_launch())) return cleanup(rc);
  *out = h;
  return CGLBM_OK;
}

}  // namespace

extern "C" {

int cglbm_step(cglbm_handle *h, int32_t n_steps, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (n_steps < 0) return fail(CGLBM_EINVAL, "n_steps must be >= 0");
  hipStream_t s = (hipStream_t)stream;
  if (effective_schedule(h) == 2) return step_compact(h, n_steps, s);
  if (h->clive) {
    const int rc = flush_compact(h, s);
    if (rc) return rc;
  }
  if (h->pad_dirty >= 0 && n_steps > 0) {
    hipLaunchKernelGGL(kZeroPad[h->storage], dim3((unsigned)h->n_boxes), dim3(kPadBlock), 0, s,
                       h->d_boxes, h->pop[h->pad_dirty], h->L.total);
    // (captured by the caller, it has not run yet)
    if (!h->pad_replayed && !capturing(s)) h->pad_dirty = -1;
  }
  int32_t k = 0;
  if (h->use_graph && !h->prof && n_steps >= 2) {
    if (!h->graph[h->cur]) {
      const int rc = capture_pair(h);
      if (rc) return rc;
    }
    for (; k + 1 < n_steps; k += 2) HIP_TRY(hipGraphLaunch(h->graph[h->cur], s));
  }
  for (; k < n_steps; ++k) {
    const int rc = launch_step(h, s);
    if (rc) return rc;
  }
  return CGLBM_OK;
}

int cglbm_set_graph(cglbm_handle *h, int32_t enable) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (enable != 0 && enable != 1) return fail(CGLBM_EINVAL, "enable must be 0 or 1");
  h->use_graph = enable;
  return CGLBM_OK;
}

int cglbm_moments(cglbm_handle *h, int32_t box, uint32_t field_mask, float *out_dev,
                  void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (box < 0 || box >= h->n_boxes) return fail(CGLBM_EINVAL, "box %d out of range", box);
  if (field_mask == 0 || (field_mask >> 17)) return fail(CGLBM_EINVAL, "bad field mask 0x%x", field_mask);
  if (!out_dev) return fail(CGLBM_EINVAL, "out_dev must not be NULL");
  hipStream_t s = (hipStream_t)stream;
  // u and F take F, then n, kappa and Q by themselves
  const uint32_t need = (field_mask & 0x3870u ? (uint32_t)NEED_F : 0u) |
                        (field_mask & 0x380u ? (uint32_t)NEED_N : 0u) |
                        (field_mask & 0x400u ? (uint32_t)NEED_KAPPA : 0u) |
                        (field_mask & 0x1C000u ? (uint32_t)NEED_Q : 0u);
  int rc = compute_fields(h, s, need);
  if (rc) return rc;
  const int64_t n = h->L.boxes[box].n;
  hipLaunchKernelGGL(k_fields, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     h->d_boxes, box, h->aux, h->L.total, field_mask, out_dev);
  return check_launch();
}

int cglbm_reduce(cglbm_handle *h, const double *centre, double *out, int32_t out_is_host,
                 void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (!out) return fail(CGLBM_EINVAL, "out must not be NULL");
  hipStream_t s = (hipStream_t)stream;
  const double *dc = nullptr;  // NULL: the kernels use each box's centre
  if (centre) {
    HIP_TRY(hipMemcpyAsync(h->d_centre, centre, sizeof(double) * 3 * (size_t)h->n_boxes,
                           hipMemcpyHostToDevice, s));
    dc = h->d_centre;
  }
  double *dout = out_is_host ? h->d_out : out;
  int rc = reduce_launch(h, s, dc, h->d_part, h->d_diag, dout);
  if (rc) return rc;
  if (!out_is_host) return CGLBM_OK;
  HIP_TRY(hipMemcpyAsync(out, h->d_out, sizeof(double) * CGLBM_NDIAG * (size_t)h->n_boxes,
                         hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  for (int b = 0; b < h->n_boxes; ++b)
    if (out[(size_t)b * CGLBM_NDIAG + 12] != 0.0)
      return fail(CGLBM_EUNSTABLE, "non-finite values in the state");
  return CGLBM_OK;
}

int cglbm_reduce_noalloc(cglbm_handle *h, const double *centre, double *out, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (!out) return fail(CGLBM_EINVAL, "out must not be NULL");
  if (h->L.rch_box.size() > kScratchChunks || (size_t)h->n_boxes > kScratchBoxes)
    return fail(CGLBM_EINVAL,
                "%zu reduction chunks of %lld nodes and %d boxes exceed the static scratch "
                "(at most %zu chunks and %zu boxes): use cglbm_reduce",
                h->L.rch_box.size(), (long long)kRedChunk, h->n_boxes, kScratchChunks,
                kScratchBoxes);
  double *sp = h->device >= 0 && h->device < kMaxDevices ? g_scratch[h->device] : nullptr;
  if (!sp) return fail(CGLBM_ESTATE, "scratch of device %d was not looked up", h->device);
  return reduce_launch(h, (hipStream_t)stream, centre, sp, sp + kScratchChunks * kNPart, out);
}

int cglbm_set_schedule(cglbm_handle *h, int32_t schedule) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (schedule < 0 || schedule > 2) return fail(CGLBM_EINVAL, "unknown schedule %d", schedule);
  if (schedule != 0 && h->lattice == LATTICE_D2Q9)
    return fail(CGLBM_EUNSUPPORTED, "D2Q9 steps have one schedule (0)");
  if (schedule == 2 && !compact_ok(h))
    return fail(CGLBM_EUNSUPPORTED,
                "the compact schedule needs D3Q27, FP32 storage (or a mass-exact FP32 or "
                "16-bit storage with Model D and Q), two buffers and unit higher-order rates");
  if (h->clive) {
    const int rc = flush_compact(h, h->cstream);
    if (rc) return rc;
  }
  if (schedule != h->schedule) drop_graphs(h);
  h->schedule = schedule;
  // the fused geometry preferred by the schedule (the autotuner's choices);
  // work still running on any stream may read the column tables, so the
  // device is synchronized before they are replaced
  if (h->lattice == LATTICE_D3Q27) {
    const int32_t v = schedule == 2 ? h->fvar_compact : h->fvar_pop;
    const int32_t m = schedule == 2 ? h->wmode_compact : h->wmode_pop;
    if (v != h->variant || m != h->wmode) {
      HIP_TRY(hipDeviceSynchronize());
      return select_mode(h, v, m, nullptr);
    }
  }
  return CGLBM_OK;
}

int cglbm_get_schedule(const cglbm_handle *h) { return h ? effective_schedule(h) : -1; }

int cglbm_num_variants(void) { return kNumFused; }

int cglbm_variant_info(int32_t v, int32_t *info) {
  g_err.clear();
  if (v < 0 || v >= kNumFused || !info) return fail(CGLBM_EINVAL, "bad variant %d", v);
  info[0] = fused_variant(v).tx;
  info[1] = fused_variant(v).ty;
  info[2] = fused_variant(v).zc;
  info[3] = fused_variant(v).minw;
  return CGLBM_OK;
}

int cglbm_variant_info_d2q9(int32_t v, int32_t *info) {
  g_err.clear();
  if (v < 0 || v >= kNumV2 || !info) return fail(CGLBM_EINVAL, "bad D2Q9 variant %d", v);
  info[0] = variant2(v).tx;
  info[1] = variant2(v).ty;
  return CGLBM_OK;
}

int cglbm_set_variant(cglbm_handle *h, int32_t v, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  const int nv = h->lattice == LATTICE_D2Q9 ? kNumV2 : kNumFused;
  if (v < 0 || v >= nv) return fail(CGLBM_EINVAL, "variant %d out of range", v);
  if (h->clive) {
    const int rc = flush_compact(h, h->cstream);
    if (rc) return rc;
  }
  h->fvar_pop = h->fvar_compact = v;
  return select_variant(h, v, (hipStream_t)stream);
}

int cglbm_get_variant(const cglbm_handle *h) { return h ? h->variant : -1; }

int cglbm_set_wall_mode(cglbm_handle *h, int32_t mode, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (h->lattice != LATTICE_D3Q27) return fail(CGLBM_EUNSUPPORTED, "D2Q9 has no wall modes");
  if (mode < 0 || mode > 3) return fail(CGLBM_EINVAL, "wall mode %d out of range", mode);
  if (h->clive) {
    const int rc = flush_compact(h, h->cstream);
    if (rc) return rc;
  }
  h->wmode_pop = h->wmode_compact = mode;
  return select_mode(h, h->variant, mode, (hipStream_t)stream);
}

int cglbm_get_wall_mode(const cglbm_handle *h) { return h ? h->wmode : -1; }

int cglbm_set_compact_variant(cglbm_handle *h, int32_t v, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (v < 0 || v >= kNumCPull) return fail(CGLBM_EINVAL, "compact variant %d out of range", v);
  if (h->clive) {
    const int rc = flush_compact(h, h->cstream);
    if (rc) return rc;
  }
  return select_cvariant(h, v, (hipStream_t)stream);
}

int cglbm_set_resident(cglbm_handle *h, int32_t enable, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (enable != 0 && enable != 1) return fail(CGLBM_EINVAL, "enable must be 0 or 1, not %d", enable);
  h->resident = enable == 1;
  return enable ? CGLBM_OK : flush_compact(h, (hipStream_t)stream);
}

int cglbm_get_resident(const cglbm_handle *h) { return h ? (h->resident ? 1 : 0) : -1; }

int cglbm_sync_state(cglbm_handle *h, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  return flush_compact(h, (hipStream_t)stream);
}

int cglbm_compact_variant(const cglbm_handle *h, int32_t *info) {
  if (!h) return -1;
  if (info) {
    const CPullVariant &C = cpull_variant(h->cvariant);
    info[0] = C.tx;
    info[1] = C.ty;
    info[2] = C.zc;
  }
  return h->cvariant;
}

int cglbm_autotune(cglbm_handle *h, int32_t reps, double *ms_per_variant, void *stream) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (reps < 1) return fail(CGLBM_EINVAL, "reps must be >= 1");
  hipStream_t s = (hipStream_t)stream;
  if (h->lattice == LATTICE_D2Q9) return autotune2(h, reps, ms_per_variant, s);
  if (h->clive) {
    const int rc = flush_compact(h, s);
    if (rc) return rc;
  }
  // Each candidate is timed as a step runs it: after the kernel before it in
  // the step, which leaves its inputs where a step finds them.  (Launched back
  // to back on one set of inputs, the candidates found them in the memory-side
  // cache, and a geometry won that was 12 % slower in a step: 128x112x96 with
  // 16-bit storage.)  The pull of the population schedules reads the stored
  // state, which nothing here advances; in place, where the candidates
  // themselves write the next state into the one buffer, they run on the one
  // pull, and the call advances the state by exactly one step.
  auto pull = [&] { return h->inplace ? CGLBM_OK : launch_pull(h, s, 1); };
  int rc = launch_pull(h, s, 1);
  if (rc || (rc = check_launch())) return rc;
  const int few = std::max(1, (int)reps / 2);
  // (layouts that the fused kernel does not step use it, if at all, for the
  // fields of large boxes)
  const bool fields = h->L.general && h->L.total >= kIfaceNodes;
  auto fused = [&] { return launch_fused(h, s, fields ? NEED_N | NEED_F | NEED_Q : 0); };
  int best = h->variant;
  double best_ms = 1e300;
  rc = fastest(kNumFused, reps, reps,
               [&](int v, int n, Timing &t) {
                 const int r = select_variant(h, v, s);
                 return r ? r : time_in_step(s, n, pull, fused, t);
               },
               ms_per_variant, best, best_ms);
  // the three-kernel schedule after the same pull
  Timing three;
  if (!rc && !(rc = select_variant(h, best, s)))
    rc = time_in_step(s, reps, pull,
                      [&] {
                        const int r = launch_iface(h, s);
                        return r ? r : launch_collide(h, s);
                      },
                      three);
  if (!rc && ms_per_variant) ms_per_variant[kNumFused] = three.mean;
  // the compact schedule's fused kernel (its own best geometry), then its
  // pull, in steps of that schedule: they advance only the compact state in
  // the other buffer, which the first collision writes from the pull above,
  // and the wall stashes, each pull from the one that the pull before it wrote
  int cfbest = best;
  auto compact_start = [&] {
    const int r = launch_pull_compact(h, s);
    return r ? r : launch_fused_compact(h, s);
  };
  if (!rc && compact_ok(h)) {
    rc = compact_start();
    int stash = 0;
    auto cpull = [&] {
      const int rd = stash;
      stash = 1 - stash;
      return launch_cpull(h, s, rd);
    };
    auto collide = [&] { return launch_fused_compact(h, s); };
    int cbest = h->cvariant;
    double c_ms = 1e300;
    if (!rc)
      rc = fastest(kNumFused, few, reps,
                   [&](int v, int n, Timing &t) {
                     const int r = select_variant(h, v, s);
                     return r ? r : time_in_step(s, n, cpull, collide, t);
                   },
                   nullptr, cfbest, c_ms);
    if (!rc) rc = select_variant(h, cfbest, s);
    if (!rc)
      rc = fastest(kNumCPull, few, reps,
                   [&](int v, int n, Timing &t) {
                     const int r = select_cvariant(h, v, s);
                     return r ? r : time_in_step(s, n, collide, cpull, t);
                   },
                   nullptr, cbest, c_ms);
    if (!rc) rc = select_cvariant(h, cbest, s);
  }
  h->fvar_pop = best;
  h->fvar_compact = cfbest;
  // boxes with walls: the wall mode of each schedule with its chosen
  // geometries, in steps as well: the fused kernel after a pull for the
  // population schedule (layouts with the three-kernel schedule may run it for
  // the fields of large boxes, else they have no launch in parts there), the
  // pull and the fused kernel for the compact one.  (Direct
  // launches: replays of throw-away graphs with the fork and join had timed
  // them closer to what a step's graph does, but processes that made many of
  // those ended in a damaged heap.)
  for (int cmp = 0; cmp < 2 && !rc && h->L.walls && !h->inplace; ++cmp) {
    if (cmp ? !compact_ok(h) : h->L.general && !iface_fused(h->L)) continue;
    rc = select_variant(h, cmp ? cfbest : best, s);
    if (!rc && cmp) rc = compact_start();
    if (rc) break;
    int stash = 0;
    auto before = [&] { return cmp ? CGLBM_OK : launch_pull(h, s, 1); };
    auto launch = [&] {
      if (!cmp) return fused();
      const int r = launch_cpull(h, s, stash);
      stash = 1 - stash;
      return r ? r : launch_fused_compact(h, s);
    };
    int32_t mbest = cmp ? h->wmode_compact : h->wmode_pop;
    double mbest_ms = 1e300;
    rc = fastest(4, few, reps,
                 [&](int m, int n, Timing &t) {
                   const int r = select_mode(h, cmp ? cfbest : best, m, s);
                   return r ? r : time_in_step(s, n, before, launch, t);
                 },
                 nullptr, mbest, mbest_ms);
    (cmp ? h->wmode_compact : h->wmode_pop) = mbest;
  }
  if (!rc) rc = select_mode(h, best, h->wmode_pop, s);
  if (rc) return rc;
  const int32_t sched = three.median < best_ms ? 1 : 0;
  if (sched != h->schedule) drop_graphs(h);
  h->schedule = sched;
  if (h->inplace) h->cur = 1 - h->cur;
  return CGLBM_OK;
}

int cglbm_profile_begin(cglbm_handle *h, int32_t max_launches) {
  g_err.clear();
  if (!h) return fail(CGLBM_ESTATE, "null handle");
  if (max_launches <= 0) return fail(CGLBM_EINVAL, "max_launches must be > 0");
  for (hipEvent_t e : h->ev) (void)hipEventDestroy(e);
  h->ev.assign(2 * (size_t)max_launches, nullptr);
  h->ev_kind.assign((size_t)max_launches, -1);
  for (auto &e : h->ev) HIP_TRY(hipEventCreate(&e));
  h->ev_used = 0;
  h->prof = true;
  return CGLBM_OK;
}

int cglbm_profile_end(cglbm_handle *h, double *total_ms, int64_t *launches, int32_t n_kinds) {
  g_err.clear();
  if (!h || !h->prof) return fail(CGLBM_ESTATE, "profiling was not started");
  h->prof = false;
  std::vector<double> ms(KIND_N, 0.0);
  std::vector<int64_t> cnt(KIND_N, 0);
  for (size_t k = 0; k < h->ev_used / 2; ++k) {
    HIP_TRY(hipEventSynchronize(h->ev[2 * k + 1]));
    float t = 0.f;
    HIP_TRY(hipEventElapsedTime(&t, h->ev[2 * k], h->ev[2 * k + 1]));
    ms[h->ev_kind[k]] += t;
    cnt[h->ev_kind[k]] += 1;
  }
  for (int k = 0; k < n_kinds && k < KIND_N; ++k) {
    if (total_ms) total_ms[k] = ms[k];
    if (launches) launches[k] = cnt[k];
  }
  for (hipEvent_t e : h->ev) (void)hipEventDestroy(e);
  h->ev.clear();
  h->ev_kind.clear();
  h->ev_used = 0;
  return CGLBM_OK;
}

void cglbm_destroy(cglbm_handle *h) {
  if (!h) return;
  // replays of the graphs and launches on the side stream may still be
  // running: wait first, then graphs, events, and the streams that they were
  // captured on (an event refers to its capture stream until it is destroyed)
  (void)wait_device(h);
  drop_graphs(h);
  for (hipGraphExec_t g : h->retired) (void)hipGraphExecDestroy(g);
  if (h->fork_ev) (void)hipEventDestroy(h->fork_ev);
  if (h->join_ev) (void)hipEventDestroy(h->join_ev);
  for (hipEvent_t e : h->ev)
    if (e) (void)hipEventDestroy(e);
  if (h->cap_stream) (void)hipStreamDestroy(h->cap_stream);
  if (h->side) (void)hipStreamDestroy(h->side);
  if (h->d_boxes) (void)hipFree(h->d_boxes);
  if (h->d_blk_box) (void)hipFree(h->d_blk_box);
  if (h->d_tile_box) (void)hipFree(h->d_tile_box);
  if (h->d_col_box) (void)hipFree(h->d_col_box);
  if (h->d_col_tiles) (void)hipFree(h->d_col_tiles);
  if (h->d_part) (void)hipFree(h->d_part);
  if (h->d_rch_box) (void)hipFree(h->d_rch_box);
  if (h->d_out) (void)hipFree(h->d_out);
  if (h->d_diag) (void)hipFree(h->d_diag);
  if (h->d_centre) (void)hipFree(h->d_centre);
  if (h->stash) (void)hipFree(h->stash);
  for (void *p : h->cstash)
    if (p) (void)hipFree(p);
  if (h->d_wblk_box) (void)hipFree(h->d_wblk_box);
  if (h->d_ccol_tiles) (void)hipFree(h->d_ccol_tiles);
  delete h;
}

}  // extern "C"
