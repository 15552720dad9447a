// Host check of the adjoint's 32-bit sums: over seeded random geometries, bricks
// and views, with the kernels' own brick setup, bounds and scale (brick.h), how
// coarse a unit of the sums is against the finest power of two that the exact
// count of a pixel's contributions allows, and whether a sum could leave int32.
//
// Usage: sum_unit_check SEED COUNT
// Prints "<kind> views=.. over=.. rms=R worst=W pow2=P": R, W the root mean square and
// largest ratio of the units, in per cent; P the former for a unit rounded up
// to a power of two.
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
  long views = 0, over = 0;
  double square = 0.0, worst = 0.0, pow2 = 0.0;
};

void check_run(const fdk_geometry& g, const fdk::GeoConst& gc, const fdk::SliceRun& run,
               const fdk::ViewBatch& vb, SplitMix64* rng, Stats* st) {
  using namespace fdk;
  const bool mirror = run.mirror != 0;
  const int32_t bz = mirror ? kBrickZ : kPlainBrickZ;
  const TileShape ts = fp_tile_shape(&g, gc, run, vb, false);
  if (ts.vc <= 0 || ts.wide) return;
  const float kvf = static_cast<float>(gc.kv);
  for (int n = 0; n < 8; ++n) {
    const int32_t s = rng->irange(0, vb.nviews - 1);
    const int32_t bx = n < 4 ? (n & 1) * (ts.nbx - 1) : rng->irange(0, ts.nbx - 1);
    const int32_t by = n < 4 ? (n >> 1) * (ts.nby - 1) : rng->irange(0, ts.nby - 1);
    const int32_t kb = run.k_first + rng->irange(0, ts.nseg - 1) * bz;
    const int32_t i_lo = bx * kBrickX, j_lo = by * kBrickY;
    const int32_t i_hi = std::min(i_lo + kBrickX - 1, gc.nx - 1);
    const int32_t j_hi = std::min(j_lo + kBrickY - 1, gc.ny - 1);
    const ViewGeo vg = view_geo(gc, vb.sn[s], vb.cs[s]);
    const BrickView b = brick_setup(gc, vg, i_lo, i_hi, j_lo, j_hi, kb, 0, 0, bz, mirror);
    float dvk = INFINITY, w = 0.0f;
    for (int c = 0; c < 4; ++c) {
      const ColumnF32 col = column_f32(b, (c & 1) ? static_cast<float>(i_hi - i_lo) : 0.0f,
                                       (c & 2) ? static_cast<float>(j_hi - j_lo) : 0.0f, kvf);
      dvk = std::fmin(dvk, col.dvk);
      w = std::fmax(w, col.w);
    }
    std::vector<float> hist(ts.tu + 2, 0.0f);
    float most = 0.0f, wmax = 0.0f;
    for (int32_t j = j_lo; j <= j_hi; ++j)
      for (int32_t i = i_lo; i <= i_hi; ++i) {
        const ColumnF32 c = column_f32(b, static_cast<float>(i - i_lo), static_cast<float>(j - j_lo), kvf);
        hist[std::min<uint32_t>(c.nu, ts.tu - 1) + 1] += slots_at_row(c.dvk, bz);
        wmax = std::fmax(wmax, c.w);
      }
    for (size_t p = 1; p < hist.size(); ++p) most = std::fmax(most, hist[p] + hist[p - 1]);
    // Voxels of magnitude 1 all over.
    const float bound = slots_at_row(dvk, bz) *
                        static_cast<float>(columns_at_pixel(gc, vg, i_lo, i_hi, j_lo, j_hi)) * w;
    const double scale = sum_scale(1.01f * bound);
    int e_exact, e_bound;
    std::frexp(1.01f * most * wmax, &e_exact);
    std::frexp(1.01f * bound, &e_bound);
    const double ratio = 1.0 / scale / std::ldexp(1.0, e_exact), pow2 = std::ldexp(1.0, e_bound - e_exact);
    ++st->views;
    // Half a unit more for each of up to 40 x 256 adds.
    if (!(scale * 2147483648.0 * most * wmax + 5120.0 < 2147483647.0)) ++st->over;
    st->square += ratio * ratio;
    st->worst = std::max(st->worst, ratio);
    st->pow2 += pow2 * pow2;
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
    g.nx = rng.irange(16, 300);
    g.ny = rng.irange(16, 300);
    g.nz = rng.irange(16, 300);
    g.dx = g.dy = 1.0;
    g.dz = rng.uni(0.8, 1.25);
    g.nu = rng.irange(32, 500);
    g.nv = rng.irange(32, 500);
    g.off_v = n % 2 ? 0.0 : 0.27;
    const double r = 0.5 * std::hypot(g.nx - 1, g.ny - 1);
    g.sod = r * rng.uni(2.0, 15.0);
    g.sdd = g.sod * rng.uni(1.2, 3.0);
    g.du = g.sdd / g.sod / rng.uni(0.6, 1.4);
    g.dv = g.sdd / g.sod * g.dz / rng.uni(0.6, 1.4);
    const int nviews = rng.irange(1, fdk::kMaxViewsPerLaunch);
    for (int s = 0; s < nviews; ++s) ang[s] = rng.uni(0.0, 6.283185307179586);
    g.np = nviews;
    g.angles = ang.data();
    const fdk::GeoConst gc = fdk::make_geo(&g);
    fdk::ViewBatch vb{};
    vb.nviews = nviews;
    for (int s = 0; s < nviews; ++s) fdk::set_view(&vb, s, ang[s]);
    if (gc.mirror_g != INT32_MIN)
      check_run(g, gc, fdk::SliceRun{0, g.nz / 2, 0, g.nz - 1, 1}, vb, &rng, &all[0]);
    else
      check_run(g, gc, fdk::SliceRun{0, g.nz, 0, 0, 0}, vb, &rng, &all[1]);
  }
  const char* names[2] = {"mirror", "plain"};
  for (int k = 0; k < 2; ++k) {
    const Stats& s = all[k];
    const double n = std::max(1l, s.views);
    std::printf("%s views=%ld over=%ld rms=%.1f worst=%.1f pow2=%.1f\n", names[k], s.views, s.over,
                100.0 * std::sqrt(s.square / n), 100.0 * s.worst, 100.0 * std::sqrt(s.pow2 / n));
  }
  return 0;
}
