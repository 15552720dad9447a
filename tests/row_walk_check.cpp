// Host check of the back-projector's launch shapes (bp_tile_shape) and of the
// rows its row walk reads: for seeded random geometries, the first and last
// row of every block of every column of every brick, computed with the
// kernels' own brick setup and FP32 column arithmetic (brick.h, built for the
// host), must lie in the staged tile, the block's offsets in [0, 2), and the
// shape must fit the staged kernels' passes and LDS. The columns of a view
// are walked on a sample of bricks.
//
// The adjoint's bounds are checked on the same bricks: its 8-slice walk stays in
// its tile where the brick's corners allow it, and no pixel can receive from
// more (column, slice) pairs than columns_at_pixel times slots_at_row, by a
// histogram of the columns' pixels.
//
// Usage: row_walk_check SEED COUNT
// Prints "<kind> launches=.. walked=.. columns=.. np16=.. np8=.. np4=..
// groups=.. bad_shape=.. load=.. low=.. high=.. offset=..
// adj_bricks=.. adj_walked=.. adj_wide=.. adj_low=.. adj_high=.. adj_over=.. adj_slack=.."
// (the mean of bound over histogram maximum, in per cent).
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
  long launches = 0, walked = 0, columns = 0, np[3] = {0, 0, 0}, groups = 0;
  long bad_shape = 0, load = 0, low = 0, high = 0, offset = 0;
  long adj_bricks = 0, adj_walked = 0, adj_wide = 0, adj_low = 0, adj_high = 0, adj_over = 0;
  double adj_slack = 0.0;  // sum of bound / histogram maximum
};

void check_run(const fdk_geometry& g, const fdk::GeoConst& gc, const fdk::SliceRun& run,
               const fdk::ViewBatch& vb, SplitMix64* rng, Stats* st) {
  using namespace fdk;
  const TileShape ts = bp_tile_shape(&g, gc, run, vb, false);
  ++st->launches;
  if (ts.groups == 0) return;
  const bool mirror = run.mirror != 0;
  const int32_t entry = mirror ? kTileEntryBytes : kPlainEntryBytes;
  const int32_t bz = mirror ? ts.np : 2 * ts.np;
  const int32_t span = ts.np == kSmallBrickZ ? std::min(ts.span, 4) : ts.span;
  ++st->np[ts.np == kBrickZ ? 0 : ts.np == kMidBrickZ ? 1 : 2];
  if (ts.groups > 1) ++st->groups;
  const bool five = !ts.wide;
  if (ts.rows > stage_passes(mirror, ts.np) || ts.rows * ts.rstep < ts.tv ||
      ts.lds_bytes < 2 * ts.groups * ts.tu * ts.tvp * entry ||
      ts.lds_bytes < ts.vc * ts.tu * ts.tvp * entry ||
      ts.lds_bytes < (ts.groups - 1) * ts.np * kBrickThreads * 4 || 
      ts.lds_bytes + kMaxViewsPerLaunch * static_cast<int>(sizeof(BrickView)) + 64 > 160 * 1024 ||
      ts.groups > kMaxGroups || ts.groups > vb.nviews || ts.nseg != (run.n + bz - 1) / bz ||
      (five && (ts.np != kBrickZ || ts.groups != 1 || ts.rows != stage_passes(mirror, 0) ||
                ts.lds_bytes > kBpTileLdsBytes)) ||
      (span && bz % span))
    ++st->bad_shape;
  // The staged loads' offsets (bp_staged_body): in the buffer exactly where the
  // pixel and its mirror are on the detector, and then theirs.
  for (int n = 0; n < 4; ++n) {
    const int32_t s = rng->irange(0, vb.nviews - 1), seg = rng->irange(0, ts.nseg - 1);
    const int32_t i_lo = rng->irange(0, ts.nbx - 1) * kBrickX, j_lo = rng->irange(0, ts.nby - 1) * kBrickY;
    const BrickView b = brick_setup(gc, view_geo(gc, vb.sn[s], vb.cs[s]), i_lo,
                                    std::min(i_lo + kBrickX - 1, gc.nx - 1), j_lo,
                                    std::min(j_lo + kBrickY - 1, gc.ny - 1),
                                    run.k_first + seg * bz, ts.tu, ts.tv, bz, mirror);
    StageOrigin at = {b.org_u, b.org_v, mirror ? gc.mirror_g - b.org_v : 0};
    if (!b.inside) at = stage_origin(gc, b.org_u, b.org_v, ts.rows * ts.rstep, mirror);
    const uint32_t es = n & 1 ? 2 : 4, row_es = gc.nu * es, nrec = row_es * gc.nv;
    for (int32_t r = 0; r < ts.tv; ++r) {
      for (int32_t col = 0; col <= ts.tu; ++col) {
        const int32_t u = b.org_u + col, v = b.org_v + r, vm = mirror ? gc.mirror_g - v : -1;
        const int32_t sr = r % ts.rstep, pass = r / ts.rstep;
        const bool on = b.inside || static_cast<uint32_t>(at.u + col) < static_cast<uint32_t>(gc.nu);
        const uint32_t down = pass * ts.rstep * row_es;
        const uint32_t o = stage_offset(on ? sr * row_es + col * es : kBadLane, at.u, at.v, row_es, es) + down;
        const uint32_t m = stage_offset(on ? col * es - sr * row_es : kBadLane, at.u, at.vm, row_es, es) - down;
        const bool in_u = u >= 0 && u < gc.nu;
        const bool want = in_u && v >= 0 && v < gc.nv, want_m = in_u && vm >= 0 && vm < gc.nv;
        if (want ? o != v * row_es + u * es : o < nrec) ++st->load;
        if (mirror && (want_m ? m != vm * row_es + u * es : m < nrec)) ++st->load;
      }
    }
  }
  if (span == 0) return;
  ++st->walked;
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
    const BrickView b = brick_setup(gc, view_geo(gc, vb.sn[s], vb.cs[s]), i_lo, i_hi, j_lo, j_hi,
                                    kb, ts.tu, ts.tv, bz, mirror);
    for (int32_t j = j_lo; j <= j_hi; ++j) {
      for (int32_t i = i_lo; i <= i_hi; ++i) {
        const ColumnF32 c = column_f32(b, static_cast<float>(i - i_lo), static_cast<float>(j - j_lo), kvf);
        ++st->columns;
        const float down = std::fmin(static_cast<float>(span - 1) * c.eps, 0.0f);
        for (int32_t t0 = 0; t0 < bz; t0 += span) {
          const float o = t0 ? fmaf(static_cast<float>(t0), c.eps, c.vl) : c.vl;
          const float fl = floorf(o + down);
          const int32_t first = t0 + static_cast<int32_t>(fl);
          if (first < 0) ++st->low;
          if (first + span + 1 >= ts.tv) ++st->high;
          for (int32_t q = 0; q < span; ++q) {
            const float oq = fmaf(static_cast<float>(q), c.eps, o - fl);
            if (!(oq >= -1e-5f) || !(oq < 2.0f)) ++st->offset;
          }
        }
      }
    }
  }
}

void check_adjoint(const fdk_geometry& g, const fdk::GeoConst& gc, const fdk::SliceRun& run,
                   const fdk::ViewBatch& vb, SplitMix64* rng, Stats* st) {
  using namespace fdk;
  const bool mirror = run.mirror != 0;
  const int32_t bz = mirror ? kBrickZ : kPlainBrickZ, walk = kBrickZ / 2;
  const TileShape ts = fp_tile_shape(&g, gc, run, vb, false);
  if (ts.vc <= 0) return;
  st->adj_wide += ts.wide;
  // Twice the bytes a view in the 64-bit sums: they stage vc / 2 views.
  const int64_t lds = static_cast<int64_t>(ts.vc) * (ts.tu + 1) * ts.tvp * fp_entry_bytes(mirror);
  if (lds > (ts.wide ? kFpWideLdsBytes : kTileLdsBytes) || ts.vc > kMaxStageViews ||
      ts.tu + 1 > kBrickThreads || ts.tvp < ts.tv)
    ++st->bad_shape;
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
    float drift = 0.0f, dvk = INFINITY;
    for (int c = 0; c < 4; ++c) {
      const ColumnF32 col = column_f32(b, (c & 1) ? static_cast<float>(i_hi - i_lo) : 0.0f,
                                       (c & 2) ? static_cast<float>(j_hi - j_lo) : 0.0f, kvf);
      drift = std::fmax(drift, std::fabs(col.eps));
      dvk = std::fmin(dvk, col.dvk);
    }
    const bool walks = static_cast<float>(walk - 1) * drift <= static_cast<float>(kSpanDrift);
    ++st->adj_bricks;
    st->adj_walked += walks;
    std::vector<float> hist(ts.tu + 2, 0.0f);
    for (int32_t j = j_lo; j <= j_hi; ++j) {
      for (int32_t i = i_lo; i <= i_hi; ++i) {
        const ColumnF32 c = column_f32(b, static_cast<float>(i - i_lo), static_cast<float>(j - j_lo), kvf);
        hist[std::min<uint32_t>(c.nu, ts.tu - 1) + 1] += slots_at_row(c.dvk, bz);
        // Highest row of the one-slice-at-a-time kernels (their first is >= 0).
        if (static_cast<float>(c.nvb) + c.fvb + static_cast<float>(bz - 1) * c.dvk + 1.0f >= static_cast<float>(ts.tv))
          ++st->adj_high;
        const float down = std::fmin(static_cast<float>(walk - 1) * c.eps, 0.0f);
        for (int32_t k0 = 0; walks && k0 < bz; k0 += walk) {
          const float fl = floorf(fmaf(static_cast<float>(k0), c.eps, c.vl) + down);
          if (k0 + static_cast<int32_t>(fl) < 0) ++st->adj_low;
          if (k0 + static_cast<int32_t>(fl) + walk + 1 >= ts.tv) ++st->adj_high;
        }
      }
    }
    float most = 0.0f;
    for (size_t p = 1; p < hist.size(); ++p) most = std::fmax(most, hist[p] + hist[p - 1]);
    const float bound = slots_at_row(dvk, bz) * static_cast<float>(columns_at_pixel(gc, vg, i_lo, i_hi, j_lo, j_hi));
    if (bound < most) ++st->adj_over;
    st->adj_slack += bound / most;
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
    // Pixels per voxel at the axis: around one for the row walk, 0.5 to 1.6.
    const double mag = g.sdd / g.sod;
    g.du = mag * g.dx / rng.uni(0.5, 1.6);
    g.dv = mag * g.dz / (n % 2 ? rng.uni(0.85, 1.2) : rng.uni(0.5, 1.6));
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
    if (gc.mirror_g != INT32_MIN && g.nz >= 2)
      check_adjoint(g, gc, fdk::SliceRun{0, g.nz / 2, 0, g.nz - 1, 1}, vb, &rng, &all[0]);
    check_adjoint(g, gc, fdk::SliceRun{0, g.nz, 0, 0, 0}, vb, &rng, &all[1]);
  }
  const char* names[2] = {"mirror", "plain"};
  for (int k = 0; k < 2; ++k) {
    const Stats& s = all[k];
    std::printf("%s launches=%ld walked=%ld columns=%ld np16=%ld np8=%ld np4=%ld groups=%ld "
                "bad_shape=%ld load=%ld low=%ld high=%ld offset=%ld adj_bricks=%ld adj_walked=%ld adj_wide=%ld adj_low=%ld "
                "adj_high=%ld adj_over=%ld adj_slack=%ld\n",
                names[k], s.launches, s.walked, s.columns, s.np[0], s.np[1], s.np[2], s.groups,
                s.bad_shape, s.load, s.low, s.high, s.offset, s.adj_bricks, s.adj_walked, s.adj_wide, s.adj_low, s.adj_high,
                s.adj_over, static_cast<long>(100.0 * s.adj_slack / std::max(1l, s.adj_bricks)));
  }
  return 0;
}
