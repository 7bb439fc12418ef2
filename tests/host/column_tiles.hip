// Host check of the column tiles (compiled for the host only): over every
// geometry of the z-marching kernels and boxes of 1 to 140 columns, narrower
// and wider than the tiles, fit_tile keeps to the geometry's threads and LDS
// room, and owned_node gives every node of the box to exactly one thread of
// one column; fit_chunk's estimate is that of assigning the blocks one by one.
#include <set>

#include "../../paper_2309_07801_amd/csrc/cglbm.hip"

namespace {

long checked = 0;

int check(const char *name, int nx, int ny, int tx, int ty, int nt, int r3, int r2, int r1) {
  TileShape T = {};
  fit_tile(nx, ny, tx, ty, nt, r3, r2, r1, T);
  if (T.w < 1 || T.h < 1 || T.w * T.h > nt || 2 * (T.w + 2 + T.h) > nt ||
      (r3 && (T.w + 6) * (T.h + 6) > r3) || (r2 && (T.w + 4) * (T.h + 4) > r2) ||
      (T.w + 2) * (T.h + 2) > r1) {
    std::printf("%s, box %dx%d: tile %dx%d does not fit\n", name, nx, ny, T.w, T.h);
    return 1;
  }
  std::vector<int> owners((size_t)nx * ny, 0);
  for (int y0 = 0; y0 < ny; y0 += T.h)
    for (int x0 = 0; x0 < nx; x0 += T.w)
      for (int t = 0; t < nt; ++t) {
        int x, y;
        if (!owned_node(T, t, x0, y0, nx, ny, x, y)) continue;
        if (x < 0 || y < 0 || x >= nx || y >= ny) {
          std::printf("%s, box %dx%d, tile %dx%d: (%d, %d) owned\n", name, nx, ny, T.w, T.h, x, y);
          return 1;
        }
        ++owners[(size_t)x + (size_t)nx * y];
      }
  for (size_t i = 0; i < owners.size(); ++i)
    if (owners[i] != 1) {
      std::printf("%s, box %dx%d, tile %dx%d: node (%zu, %zu) has %d owners\n", name, nx, ny, T.w,
                  T.h, i % nx, i / nx, owners[i]);
      return 1;
    }
  ++checked;
  return 0;
}

template <class G>
int fused(const char *name, int nx, int ny, int tx, int ty) {
  return check(name, nx, ny, tx, ty, G::NT, G::R3, G::R2, G::R1);
}
template <class G>
int cpull(const char *name, int nx, int ny, int tx, int ty) {
  return check(name, nx, ny, tx, ty, G::NT, 0, 0, G::R1);
}

// The chunk with the least time when blocks, longest first, go one by one to
// the place that is free first.
int plain_chunk(const Layout &L, bool cpull, int zc, int nt, double lead) {
  const size_t places = 256 * (size_t)(1024 / nt);
  int best = zc;
  double best_t = 1e300;
  for (int k = 0; k <= 8; ++k) {
    const int z = std::max(1, zc - zc * k / 16);
    std::vector<double> blocks;
    for (const BoxDev &B : L.boxes) {
      const TileShape &T = cpull ? B.cs : B.fs;
      const int n = (B.nz + z - 1) / z, cols = ((B.nx + T.w - 1) / T.w) * ((B.ny + T.h - 1) / T.h);
      blocks.insert(blocks.end(), (size_t)n * cols, (double)B.nz / n + lead);
    }
    if (blocks.size() > 16 * places) return zc;
    std::sort(blocks.begin(), blocks.end(), std::greater<double>());
    std::multiset<double> busy;
    for (size_t i = 0; i < places; ++i) busy.insert(0.0);
    for (double len : blocks) {
      const double t = *busy.begin() + len;
      busy.erase(busy.begin());
      busy.insert(t);
    }
    const double t = *busy.rbegin() * (2.1 + 4.6 * std::min(1.0, (double)blocks.size() / places));
    if (t < best_t * 0.98) {
      best_t = t;
      best = z;
    }
  }
  return best;
}

int chunks() {
  int bad = 0;
  uint32_t r = 1;
  auto rnd = [&](int lo, int hi) {
    r = r * 1664525u + 1013904223u;
    return lo + (int)((r >> 8) % (uint32_t)(hi - lo + 1));
  };
  for (int k = 0; k < 40; ++k) {
    Layout L;
    for (int b = k % 4 ? rnd(2, 30) : 1; b > 0; --b) {
      BoxDev B = {};
      B.nx = rnd(20, k % 4 ? 128 : 400);
      B.ny = rnd(20, k % 4 ? 128 : 400);
      B.nz = rnd(20, k % 4 ? 128 : 400);
      fit_tile(B.nx, B.ny, 64, 8, 512, 0, 0, CG512::R1, B.cs);
      fit_tile(B.nx, B.ny, 32, 8, 256, FG256::R3, FG256::R2, FG256::R1, B.fs);
      L.boxes.push_back(B);
    }
    for (int zc : {16, 32, 64}) {
      const int c[2] = {fit_chunk(L, true, zc, 512, 2.0), fit_chunk(L, false, zc, 256, 3.0)};
      const int p[2] = {plain_chunk(L, true, zc, 512, 2.0), plain_chunk(L, false, zc, 256, 3.0)};
      if (c[0] != p[0] || c[1] != p[1]) {
        std::printf("chunks of layout %d, zc %d: %d %d for %d %d\n", k, zc, c[0], c[1], p[0], p[1]);
        ++bad;
      }
    }
  }
  return bad;
}

}  // namespace

int main() {
  int bad = chunks();
  for (int nx = 1; nx <= 140; ++nx)
    for (int ny : {1, 2, 3, 5, 8, 9, 12, 17, 24, 33, 48, 49, 61, 130}) {
      bad += fused<FG128>("fused 32x4", nx, ny, 32, 4);
      bad += fused<FG256>("fused 32x8", nx, ny, 32, 8);
      bad += fused<FG256W>("fused 64x4", nx, ny, 64, 4);
      bad += fused<FG512>("fused 32x16", nx, ny, 32, 16);
      bad += fused<FG512>("fused 64x8", nx, ny, 64, 8);
      bad += fused<FG1024>("fused 64x16", nx, ny, 64, 16);
      bad += cpull<CG512>("pull 64x8", nx, ny, 64, 8);
      bad += cpull<CG256>("pull 32x8", nx, ny, 32, 8);
      bad += cpull<CG256>("pull 64x4", nx, ny, 64, 4);
    }
  if (!bad) std::printf("column tiles: %ld layouts ok\n", checked);
  return bad != 0;
}
