// Host-side sizing of the back-projection and adjoint tiles: a bound on the
// detector footprint of one brick over the views of a launch, and the
// staging layout derived from it. Host code only (it is also built into the
// tile-bound test, which checks it against every voxel's taps).
#include <algorithm>
#include <cmath>
#include <limits>

#include "fdk_internal.h"

namespace fdk {

// Host-side bound of a brick's footprint (pixels) over the views of a
// launch, from derivative bounds over the whole volume: with r the x-y
// half-diagonal and zmin = d - r,
//   |du/di| <= ku Dx (|cos| + |sin| r / zmin) / zmin,
//   |du/dj| <= ku Dy (|sin| + |cos| r / zmin) / zmin,
// and v(k) - cv = kv (k - cz) / z, so over the brick's bz slices and its z
// spread dz the rows span at most kv ((bz - 1) / zmin + |k - cz| dz / zmin^2).
TileShape tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                     const ViewBatch& vb, int32_t bz, int32_t entry_bytes, int32_t slots,
                     bool direct, bool bp_staging, bool read_pitch) {
  TileShape ts{};
  ts.nbx = (gc.nx + kBrickX - 1) / kBrickX;
  ts.nby = (gc.ny + kBrickY - 1) / kBrickY;
  ts.nseg = (run.n + bz - 1) / bz;
  const double r = 0.5 * std::hypot((g->nx - 1) * g->dx, (g->ny - 1) * g->dy);
  const double zmin = g->sod - r, rho = r / zmin;
  if (direct) return ts;  // vc = 0: direct variant
  const double kmax = gc.cz + bz;
  double wu = 0.0, wv = 0.0;
  for (int32_t s = 0; s < vb.nviews; ++s) {
    const double as = std::fabs(vb.sn[s]), ac = std::fabs(vb.cs[s]);
    const double dui = gc.ku * g->dx * (ac + as * rho) / zmin;
    const double duj = gc.ku * g->dy * (as + ac * rho) / zmin;
    wu = std::fmax(wu, (kBrickX - 1) * dui + (kBrickY - 1) * duj);
    const double dz = (kBrickX - 1) * g->dx * as + (kBrickY - 1) * g->dy * ac;
    wv = std::fmax(wv, gc.kv * ((bz - 1) / zmin + kmax * dz / (zmin * zmin)));
  }
  // floor() of the extremes adds one pixel, the second tap one row, the
  // origin margin one pixel, FP32 column arithmetic up to one more.
  ts.tu = static_cast<int32_t>(std::ceil(wu)) + 4;
  ts.tv = static_cast<int32_t>(std::ceil(wv)) + 5;
  ts.tvp = ts.tv | 1;  // odd pitch: 16 neighbouring columns hit distinct LDS banks
  if (read_pitch) {
    // The back-projector's 16-byte entry reads are served 16 lanes at a
    // time over 64 four-byte banks, and those 16 lanes cover a 4 x 4 patch
    // of voxel columns: a few tile columns, rows n and n + 1. With the pitch
    // at 7 or 9 mod 16, entries nu tvp + n of two such lanes share a bank
    // only if their columns are 7 or more apart.
    while (ts.tvp % 16 != 7 && ts.tvp % 16 != 9) ts.tvp += 2;
  }
  // dv/dk over the volume's columns, z in [d - r, d + r].
  const double drift = std::fmax(std::fabs(gc.kv / zmin - 1.0), std::fabs(gc.kv / (g->sod + r) - 1.0));
  ts.span = 7.0 * drift <= kSpanDrift ? 8 : 3.0 * drift <= kSpanDrift ? 4 : 0;
  if (bp_staging) {
    // The back-projector stages a tile row with a group of 32 or 64 lanes
    // (one wave at most): a lane per column and one more.
    if (ts.tu + 1 > kWaveLanes) return ts;
    ts.rstep = kBrickThreads / (ts.tu + 1 <= kWaveLanes / 2 ? kWaveLanes / 2 : kWaveLanes);
  } else {
    // The adjoint's flush: a thread per column.
    if (ts.tu + 1 > kBrickThreads) return ts;
    ts.rstep = kBrickThreads / ts.tu;
  }
  ts.rows = (ts.tv + ts.rstep - 1) / ts.rstep;
  const int64_t per_view = static_cast<int64_t>(ts.tu) * ts.tvp * entry_bytes;
  if (!bp_staging) {
    const int64_t vc = std::min<int64_t>({kMaxStageViews, kTileLdsBytes / per_view, slots / ts.rows});
    ts.vc = static_cast<int32_t>(std::max<int64_t>(vc, 0));
    return ts;
  }
  // Back-projector: the five-wave kernel (slots prefetch slots, 27.4 KB of
  // tiles) when it stages all kBpStageViews views per stage, else the
  // four-wave one (more slots and 35.5 KB) if that stages more.
  const int64_t vc5 = std::min<int64_t>({kBpStageViews, kBpTileLdsBytes / per_view, slots / ts.rows});
  const int64_t wide_slots = static_cast<int64_t>(slots) * kWidePrefetchSlots / kPrefetchSlots;
  const int64_t vc4 = std::min<int64_t>({kBpStageViews, kTileLdsBytes / per_view, wide_slots / ts.rows});
  ts.wide = vc5 < kBpStageViews && vc4 > vc5;
  ts.vc = static_cast<int32_t>(std::max<int64_t>(ts.wide ? vc4 : vc5, 0));
  return ts;
}

// Tiles and stages of an adjoint launch (vc = 0: the direct kernel).
//
// A tile has one more column than the back-projector's and one 32-bit word a
// pixel and plane (main, plus mirror for mirrored runs). The column pitch is
// padded to 3, 5, 11 or 13 mod 16 words, which spreads lanes in neighbouring
// columns and rows over the banks (modelled clocks per wave instruction:
// 64-bit 8.2, 8.8 at 25; 32-bit 7.9-8.4, 11-12 at 1, 9 or 15 mod 16), but not
// where that costs the second view and with it the room for a view's 64-bit
// sums (148 x 176 x 132 plain from 8 views at 2.12 pixels a voxel, magnitudes
// over 2^22: 851 us with FP32 sums, 105 so). Sized
// at the back-projector's bytes an entry, twice these, one view's tile always
// fits. Where that leaves none, or its staging slots too few for a mirrored
// tile, the wide kernel still takes the adds off the global atomics, in tiles
// of 64-bit sums: as many views as three workgroups a CU hold, else one view at
// up to one workgroup a CU. (60^3 from 20 views at 2 pixels a voxel and a wide
// cone, one workgroup a CU: 960 us direct, 186 with FP32 sums in half the
// bytes, 55 so.)
TileShape fp_tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                        const ViewBatch& vb, bool direct) {
  const bool mirror = run.mirror != 0;
  const int32_t bz = mirror ? kBrickZ : kPlainBrickZ;
  TileShape ts = tile_shape(g, gc, run, vb, bz, mirror ? kTileEntryBytes : kPlainEntryBytes,
                            mirror ? kPrefetchSlots : std::numeric_limits<int32_t>::max(), direct);
  if (direct || ts.rstep == 0) return ts;
  ts.wide = ts.vc == 0;
  const int32_t narrow = ts.tvp;
  while (ts.tvp % 16 != 3 && ts.tvp % 16 != 5 && ts.tvp % 16 != 11 && ts.tvp % 16 != 13) ts.tvp += 2;
  auto view_bytes = [&](int32_t pitch) {
    return static_cast<int64_t>(ts.tu + 1) * pitch * fp_entry_bytes(mirror);
  };
  if (!ts.wide && 2 * view_bytes(ts.tvp) > kTileLdsBytes && 2 * view_bytes(narrow) <= kTileLdsBytes)
    ts.tvp = narrow;
  const int64_t per_view = view_bytes(ts.tvp);
  const int64_t views = !ts.wide                             ? kTileLdsBytes / per_view
                        : 2 * per_view <= kFpWideLdsBytes     ? kFpWideLdsBytes / (2 * per_view)
                        : 2 * per_view <= kFpWideMostLdsBytes ? 1
                                                              : 0;
  ts.vc = static_cast<int32_t>(std::min<int64_t>(kMaxStageViews, views));
  return ts;
}

// Brick height, kernel and workgroup of a back-projection launch.
//
// Bricks of 16 slices (pairs) a thread stage the fewest pixels per voxel, so
// large volumes take them, one 256-thread group a brick. Up to 1024 bricks
// are all resident at once, and a view's chain of loads, barrier and column
// sums is latency: there
//  - bricks shrink to 8 or 4 slices while they number at most one a CU
//    (96^3 from 90 views: 59 us at 16 slices, 71 at 4 (432 bricks), 46 at 8
//    (216); 80^3: 50 at 16, 39 at 4; 64^3 from 64 views: 91 -> 31 with groups; all of
//    these then with as many staging passes in the code as 16 slices need);
//  - groups of threads share a brick's views: 4 up to a brick a CU, which
//    fills it with 16 waves (128^3 from 180 views, 256 bricks: 238 -> 119 us,
//    147 with two), 2 up to 1.5 (500 bricks: 192 us with one, 201 with two;
//    864 bricks: 306 with one, 380 with two, which no longer fit at once).
// Tiles of which two do not fit the 35.5 KB of a quarter of a CU's LDS: plain
// runs take the staged kernel all the same (301 x 277 x 199 at 1.2 pixels a
// voxel: 2.08 -> 1.69 ms), small mirrored grids bricks of 8 slices (450
// bricks: 690 us general, 559 at 16 slices, 528 at 8), while the chip holds half of
// those at once (882 bricks, four of the halves a CU: 184 us general, 166 at 8 slices;
// three a CU, 840 bricks: 191, 210, 945: 27.1, 32.1). Large mirrored grids
// get a pitch of 3, 7, 9 or 13 mod 16, next to 7 or 9 only, if two tiles then
// fit (columns five apart may share a bank at 3 and 13; 340 x 347 x 389 from
// 78 views: 1.37 -> 1.27 ms, 406 x 245 x 313 from 132: 1.71 general, 1.76
// staged at the wider pitch, 1.57), and else the general kernel (400^3, wide
// cone: 4.0 ms, staged 4.1; 371 x 412 x 350: 4.62, 5.45, 4.49 with bricks of 8
// slices, which lose 10 % at 333 x 367 x 311 from 31 views). Tiles too small for
// the five-wave staged kernel's passes (about 0.8 pixels a voxel and less) gain
// nothing from the four-wave one unless they walk or share views, and run the
// general kernel, five waves and two views a barrier (300^3 plain from 25 views
// at 0.5 pixels a voxel 217 us general, 236 staged; 138 x 206 x 320 BF16 from 3
// views 16.4, 22.4).
TileShape bp_tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                        const ViewBatch& vb, bool direct) {
  const int32_t entry = run.mirror ? kTileEntryBytes : kPlainEntryBytes;
  auto shape = [&](int32_t np) {
    TileShape t = tile_shape(g, gc, run, vb, run.mirror ? np : 2 * np, entry,
                             run.mirror ? kPrefetchSlots : kPlainPrefetchSlots, direct, true,
                             run.mirror != 0);
    t.np = np;
    t.lds_bytes = t.vc * t.tu * t.tvp * entry;
    return t;
  };
  // Dynamic LDS of n groups: two tiles each, and at the end their sums.
  auto lds = [&](const TileShape& t, int32_t n) {
    return std::max(2 * n * t.tu * t.tvp * entry,
                    (n - 1) * t.np * kBrickThreads * static_cast<int32_t>(sizeof(float)));
  };
  auto bricks = [](const TileShape& t) { return static_cast<int64_t>(t.nbx) * t.nby * t.nseg; };
  auto staged = [&](const TileShape& t) {
    return t.vc > 0 && t.rows <= stage_passes(run.mirror, t.np) && lds(t, 1) <= kGroupLdsBytes &&
           stage_reach_ok(g->nu, g->nv, t.rows * t.rstep);
  };
  TileShape ts = shape(kBrickZ);
  if (ts.vc <= 0) return ts;
  // Whether wide tiles halve their bricks: the chip holds half of them at once.
  bool mid = false;
  if (ts.vc != kBpStageViews && bricks(ts) <= kResidentGroups) {
    const TileShape half = shape(kMidBrickZ);
    const int64_t per_cu = std::min(4, kCuLdsBytes / (lds(half, 1) + kBpStaticLdsBytes));
    mid = bricks(half) <= 2 * per_cu * kCus;
  }
  if (bricks(ts) <= kResidentGroups) {
    for (int32_t np : {kMidBrickZ, kSmallBrickZ}) {
      const TileShape t = shape(np);
      if (staged(t) && (bricks(t) <= kCus || (mid && ts.vc != kBpStageViews && np == kMidBrickZ)))
        ts = t;
    }
  }
  if (run.mirror && ts.vc != kBpStageViews && !mid) {
    TileShape t = ts;
    t.tvp = t.tv | 1;
    while (t.tvp % 16 != 3 && t.tvp % 16 != 7 && t.tvp % 16 != 9 && t.tvp % 16 != 13) t.tvp += 2;
    if (lds(t, 1) > kTileLdsBytes || !staged(t)) return ts;
    ts = t;
  }
  if (!staged(ts)) return ts;
  ts.groups = bricks(ts) <= kCus ? kMaxGroups : 2 * bricks(ts) <= 3 * kCus ? 2 : 1;
  while (ts.groups > 1 && (ts.groups > vb.nviews || lds(ts, ts.groups) > kGroupLdsBytes))
    ts.groups /= 2;
  if (ts.span == 0 && ts.groups == 1 && ts.np == kBrickZ && ts.vc == kBpStageViews && !ts.wide &&
      ts.rows < stage_passes(run.mirror, 0)) {
    ts.groups = 0;
    return ts;
  }
  ts.lds_bytes = lds(ts, ts.groups);
  ts.wide = ts.wide || ts.groups > 1 || ts.np != kBrickZ || ts.vc != kBpStageViews ||
            ts.rows != stage_passes(run.mirror, 0);
  return ts;
}

}  // namespace fdk
