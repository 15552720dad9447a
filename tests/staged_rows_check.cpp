// Host check of the tile entries that the staged back-projector reads: for
// seeded random geometries, every launch shape that bp_tile_shape gives, and a
// sample of bricks and views of each, every column's
//  - tile column, which must lie in the tile (the kernels clamp it);
//  - rows of the row walk, by the kernels' own walk_start: in the tile, and each
//    slice's v within a row of the one that the walk takes for it;
//  - rows of the loop that finds each slice's by itself (which the shapes without
//    a walk take): from 0 to tv - 1.
//
// Usage: staged_rows_check SEED COUNT
// Prints "<kind> columns=.. walked=.. single=.. np16=.. np8=.. np4=.. col=.. low=.. high=.. off=..".
#include <algorithm>
#include <cinttypes>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1909_02724_amd/csrc/brick.h"
#include "../paper_1909_02724_amd/csrc/geometry_host.h"

namespace {

struct SplitMix64 {  // Steele, Lea and Flood (2014)
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
  }
  double uni(double a, double b) { return a + (b - a) * ((next() >> 11) * (1.0 / 9007199254740992.0)); }
  int irange(int a, int b) { return a + static_cast<int>(next() % static_cast<uint64_t>(b - a + 1)); }
};

struct Stats {
  long columns = 0, walked = 0, single = 0, np[3] = {0, 0, 0}, col = 0, low = 0, high = 0, off = 0;
};

void check_run(const fdk_geometry& g, const fdk::GeoConst& gc, const fdk::SliceRun& run,
               const fdk::ViewBatch& vb, SplitMix64* rng, Stats* st) {
  using namespace fdk;
  const TileShape ts = bp_tile_shape(&g, gc, run, vb, false);
  if (ts.vc <= 0) return;
  const bool mirror = run.mirror != 0;
  const int32_t bz = mirror ? ts.np : 2 * ts.np;
  const int32_t span = ts.groups == 0 ? 0 : ts.np == kSmallBrickZ ? std::min(ts.span, 4) : ts.span;
  ++st->np[ts.np == kBrickZ ? 0 : ts.np == kMidBrickZ ? 1 : 2];
  ++(span ? st->walked : st->single);
  const float kvf = static_cast<float>(gc.kv);
  for (int n = 0; n < 12; ++n) {
    const int32_t s = rng->irange(0, vb.nviews - 1);
    // Corner bricks first, then random ones.
    const int32_t bx = n < 4 ? (n & 1) * (ts.nbx - 1) : rng->irange(0, ts.nbx - 1);
    const int32_t by = n < 4 ? (n >> 1) * (ts.nby - 1) : rng->irange(0, ts.nby - 1);
    const int32_t seg = n & 1 ? ts.nseg - 1 : n & 2 ? 0 : rng->irange(0, ts.nseg - 1);
    const int32_t kb = run.k_first + seg * bz;
    const int32_t i_lo = bx * kBrickX, j_lo = by * kBrickY;
    const int32_t i_hi = std::min(i_lo + kBrickX - 1, gc.nx - 1);
    const int32_t j_hi = std::min(j_lo + kBrickY - 1, gc.ny - 1);
    const BrickView b = brick_setup(gc, view_geo(gc, vb.sn[s], vb.cs[s]), i_lo, i_hi, j_lo, j_hi, kb,
                                    ts.tu, ts.tv, bz, mirror);
    for (int32_t j = j_lo; j <= j_hi; ++j) {
      for (int32_t i = i_lo; i <= i_hi; ++i) {
        const ColumnF32 c = column_f32(b, static_cast<float>(i - i_lo), static_cast<float>(j - j_lo), kvf);
        ++st->columns;
        if (c.nu >= static_cast<uint32_t>(ts.tu)) ++st->col;
        for (int32_t k0 = 0; span && k0 < bz; k0 += span) {
          const WalkStart w = walk_start(c, k0, span);
          if (w.row < 0) ++st->low;
          if (w.row + span + 1 >= ts.tv) ++st->high;
          for (int32_t m = 0; m < span; ++m) {
            const float x = fmaf(static_cast<float>(m), c.eps, w.x);
            // The slice's own v, from the row that the walk gives weight 1 - |x|.
            const float v = fmaf(static_cast<float>(k0 + m), c.dvk, c.vl) - static_cast<float>(w.row + m + 1);
            if (!(std::fabs(x) < 1.0f + 1e-5f) || std::fabs(v - x) > 1e-4f) ++st->off;
          }
        }
        for (int32_t t = 0; !span && t < bz; ++t) {
          uint32_t dn;
          float fr;
          voxel_row_off(c.fvb, c.dvk, t, &dn, &fr);
          if (static_cast<int64_t>(c.nvb) + dn + 1 >= ts.tv) ++st->high;
        }
      }
    }
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 3) {
    std::fprintf(stderr, "usage: %s SEED COUNT\n", argv[0]);
    return 2;
  }
  SplitMix64 rng{std::strtoull(argv[1], nullptr, 10)};
  const long count = std::strtol(argv[2], nullptr, 10);
  Stats all[2];
  std::vector<double> ang(fdk::kMaxViewsPerLaunch);
  for (long n = 0; n < count; ++n) {
    fdk_geometry g{};
    const int big = n % 3 == 0 ? 400 : 150;
    g.nx = rng.irange(1, big);
    g.ny = rng.irange(1, big);
    g.nz = rng.irange(1, big);
    g.dx = g.dy = 1.0;
    g.dz = rng.uni(0.7, 1.4);
    g.nu = rng.irange(2, 500);
    g.nv = rng.irange(2, 500);
    const int kind = rng.irange(0, 2);
    g.off_u = rng.uni(-4.0, 4.0);
    g.off_v = kind == 0 ? 0.0 : kind == 1 ? 0.5 * rng.irange(-8, 8) : rng.uni(-4.0, 4.0);
    const double r = 0.5 * std::hypot(g.nx - 1, g.ny - 1);
    g.sod = std::max(r, 0.5) * rng.uni(1.5, 20.0) + 1.0;
    g.sdd = g.sod * rng.uni(1.05, 4.0);
    const double mag = g.sdd / g.sod;
    g.du = mag * g.dx / rng.uni(0.4, 2.5);
    g.dv = mag * g.dz / (n % 2 ? rng.uni(0.85, 1.2) : rng.uni(0.4, 2.5));
    const int nviews = rng.irange(1, fdk::kMaxViewsPerLaunch);
    for (int s = 0; s < nviews; ++s) ang[s] = rng.uni(0.0, 6.283185307179586);
    g.np = nviews;
    g.angles = ang.data();
    const fdk::GeoConst gc = fdk::make_geo(&g);
    fdk::ViewBatch vb{};
    vb.nviews = nviews;
    for (int s = 0; s < nviews; ++s) fdk::set_view(&vb, s, ang[s]);
    if (gc.mirror_g != INT32_MIN && g.nz >= 2)
      check_run(g, gc, fdk::SliceRun{0, g.nz / 2, 0, g.nz - 1, 1}, vb, &rng, &all[0]);
    check_run(g, gc, fdk::SliceRun{0, g.nz, 0, 0, 0}, vb, &rng, &all[1]);
  }
  const char* names[2] = {"mirror", "plain"};
  for (int k = 0; k < 2; ++k) {
    const Stats& s = all[k];
    std::printf("%s columns=%ld walked=%ld single=%ld np16=%ld np8=%ld np4=%ld col=%ld low=%ld high=%ld off=%ld\n",
                names[k], s.columns, s.walked, s.single, s.np[0], s.np[1], s.np[2], s.col, s.low, s.high, s.off);
  }
  return 0;
}
