// Internal launch descriptors shared by the host front end (fdk_api.cpp) and
// the HIP kernels. Not part of the public ABI.
#pragma once

#include <cstdint>

#include "../../include/fdk.h"

namespace fdk {

// Views per kernel launch: each view's sine and cosine travel in the kernel
// argument block (16 bytes a view), and each launch reads (and for the
// back-projector writes) the volume once and sets up each brick once; the
// views of a call are split evenly over the fewest launches. Measured at
// 2048^3: the back-projector 6 % faster with 64 views a launch than with
// 32, and 3 % faster again with 96.
constexpr int kMaxViewsPerLaunch = 96;

// Per-view geometry in the reduced-cost form of Alg. 4, evaluated in FP64
// from the sine and cosine of the view angle (Eq. 2 expanded; view_geo, on
// the host and in the kernels):
//   z(i, j)   = ci*i + cj*j + c0                      (Eq. 3, Theorem 3)
//   a(i, j)   = ai*i + aj*j + a0   gantry coordinate across the detector
//   u         = cu + ku * a / z                        (Theorem 2)
//   v(k)      = cv + kv * (k - cz) / z                 (linear in k)
struct ViewGeo {
  double ai, aj, a0;
  double ci, cj, c0;
};

// Launch-invariant geometry.
struct GeoConst {
  int32_t nx, ny, nz, nu, nv;
  double cu, cv, cz;  // principal point (pixels) and volume centre slice
  double ku;          // D / Du
  double kv;          // D * Dz / Dv
  double dx, dy, d;   // voxel pitches in x and y, source to axis
  double ox, oy;      // volume centre column (voxels)
  int32_t mirror_g;   // Nv - 1 + 2 off_v when that is an integer (Theorem 1)
};

// ViewGeo of the view with sin(beta) = s, cos(beta) = c (Eq. 2 expanded:
// world X = Dx (i - ox), Y = -Dy (j - oy); after the rotation,
// z = d + sin(b) X + cos(b) Y and a = cos(b) X - sin(b) Y). Host and device.
constexpr ViewGeo view_geo(const GeoConst& gc, double s, double c) {
  ViewGeo v{};
  v.ci = s * gc.dx;
  v.cj = -c * gc.dy;
  v.c0 = gc.d - s * gc.dx * gc.ox + c * gc.dy * gc.oy;
  v.ai = c * gc.dx;
  v.aj = s * gc.dy;
  v.a0 = -c * gc.dx * gc.ox - s * gc.dy * gc.oy;
  return v;
}

// A run of global slices processed by one launch family.
//  mirror = 0: slices k_first + t (t < n) stored at slab slice loc_lo + t.
//  mirror = 1: pairs (k_first + t, Nz - 1 - k_first - t), t < n; the lower
//              slice at loc_lo + t, its mirror at loc_hi - t.
struct SliceRun {
  int32_t k_first, n, loc_lo, loc_hi, mirror;
};

struct ViewBatch {
  double sn[kMaxViewsPerLaunch], cs[kMaxViewsPerLaunch];  // sin and cos of each view's angle
  int32_t nviews;
};

// Views of an adjoint launch: view s is projection idx[s] of the call. Chunk c,
// the blockIdx.y of a workgroup, takes views [first[c], first[c + 1]), whose
// rays run closer to y than to x up to chunk across_from, then closer to x: groups
// of 16 threads then run along x or y, across the rays. rot_a, rot_b: see
// slot_rotation (fp.hip).
constexpr int kMaxChunks = kMaxViewsPerLaunch;
// Views of a chunk at most: their constants (60 bytes a view) and the tiles share
// the LDS of a fifth of a CU. (With arrays for 96 views 11 % slower where that
// cost the fifth workgroup; in dynamic LDS 2 % slower throughout.)
constexpr int kFpMostViews = 80;
struct FpBatch {
  ViewBatch vb;
  int32_t idx[kMaxViewsPerLaunch];
  int32_t nchunks, across_from, rot_a, rot_b;
  uint8_t first[kMaxChunks + 1];
};

// Bricked back-projection: a workgroup of 256 threads owns a brick of
// kBrickX x kBrickY columns and kBrickZ consecutive slices of a slice run
// (plus their mirrors for a mirrored run). In the tiled variant it stages
// the brick's detector footprint for each view, a tile of tu x tv pixels,
// into LDS, vc views at a time (the staged kernel: two tiles in turn; bricks
// of small volumes hold 8 or 4 slices). tu and tv are host-side upper bounds.
constexpr int kBrickX = 16;
constexpr int kBrickY = 16;
constexpr int kBrickZ = 16;
constexpr int kBrickThreads = kBrickX * kBrickY;
constexpr int kWaveLanes = 64;
// Occupancy decides the back-projector's speed more than staging depth
// does (measured on MI355X): five 256-thread workgroups per CU, hence at
// most 27.4 KB of tiles (with the 4.5 KB of per-view brick constants, 32 KB
// a workgroup) and 102 VGPRs, with two tiles, run 5 %
// faster than four with three views a stage (and four with three 11 % (FP32)
// to 47 % (FP16) faster than three with four; six, at 80 VGPRs and 64 views a
// launch, spill: 16.1 against 12.7 ms at 512^3). The adjoint stages up to
// three views in 35.5 KB.
constexpr int kMaxStageViews = 3;
constexpr int kBpStageViews = 2;
constexpr int kPrefetchSlots = 6;       // tile entries a thread prefetches per stage
// Tiles too tall for the five-wave back-projector's slots (more than three
// staging passes per view) go to a four-wave instance with more slots.
constexpr int kWidePrefetchSlots = 12;
constexpr int kTileLdsBytes = 36352;    // LDS budget for the adjoint's and the four-wave tiles
constexpr int kBpTileLdsBytes = 28032;  // and for the five-wave back-projector's (27.4 KB)
constexpr int kTileEntryBytes = 16;     // (q, dq/du) of a row and of its mirror row

// For the adjoint's wide tiles, of 64-bit sums: three workgroups a CU, or one
// for a single view's tile past that.
constexpr int kFpWideLdsBytes = 47104;
constexpr int kFpWideMostLdsBytes = 2 * kFpWideLdsBytes;

struct TileShape {
  int32_t tu, tv, tvp;   // tile columns, rows, and the (odd) column pitch in entries
  int32_t vc;            // views staged at once; 0 selects the direct variant
  int32_t rstep, rows;   // staging: rows advanced per pass, passes per view
  int32_t wide;          // the back-projector's four-wave instances; the adjoint's wide kernel
  int32_t span;          // slices whose taps lie in span + 2 consecutive rows, at every column (0: none)
  int32_t np;            // back-projector: slices (pairs) per thread
  int32_t groups;        // back-projector: 256-thread groups per workgroup (0: the general kernel)
  int32_t lds_bytes;     // back-projector: dynamic LDS of a workgroup
  int32_t nbx, nby, nseg;  // bricks along x, y and z-segments of the run
};

// Kernel choice for a run and view batch: tiled unless the footprint tile
// exceeds the LDS or prefetch budget, or the caller asks for the direct
// variant (FDK_DIRECT).
// bz: slices per brick; entry_bytes: LDS bytes per tile entry; slots: tile
// entries a thread prefetches per stage; bp_staging: the back-projector's
// staging (lane groups per tile row) rather than the adjoint's; read_pitch:
// pad the column pitch for the mirrored back-projector's conflict-free
// entry reads.
TileShape tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                     const ViewBatch& vb, int32_t bz, int32_t entry_bytes, int32_t slots,
                     bool direct, bool bp_staging = false, bool read_pitch = false);
// Back-projector: brick heights (pairs per thread) and view groups of small
// volumes, and the row walk; the rules and what they measured are at
// bp_tile_shape (tiles.cpp) and span_column (bp.hip).
constexpr int kMidBrickZ = 8;
constexpr int kSmallBrickZ = 4;
constexpr int kMaxGroups = 4;  // 256-thread groups sharing a brick, each with its own views
constexpr int kCus = 256;
constexpr int kResidentGroups = 4 * kCus;   // groups the chip holds at four waves per SIMD
constexpr int kCuLdsBytes = 160 * 1024;
constexpr int kGroupLdsBytes = 154 * 1024;  // of these, beside the per-view brick constants
constexpr int kBpStaticLdsBytes = 48 * kMaxViewsPerLaunch;  // a workgroup's brick constants
// Staging passes of a view's tile: exactly so many in the five-wave kernel
// (np = 0), at most so many in the four-wave one with np slices a thread. Each
// pass costs its branches whether it is taken or not: with 8 and 14 for every
// np, 64^3 from 64 views took 31 us (24 now) and 96^3 from 90 views 46 (40).
constexpr int stage_passes(bool mirror, int np) {
  return np == 0              ? (mirror ? 3 : 6)
         : np == kSmallBrickZ ? (mirror ? 4 : 6)
         : np == kMidBrickZ   ? (mirror ? 6 : 9)
                              : (mirror ? 8 : 14);
}
// Whether byte offsets of rows up to reach off the detector, and 2^31 more,
// stay apart in 32 bits from those on it (stage_origin).
constexpr bool stage_reach_ok(int32_t nu, int32_t nv, int32_t reach) {
  return (static_cast<int64_t>(nv) + reach + 2) * nu * 4 + kBrickThreads * 4 <= INT64_C(1) << 31;
}
// Largest drift of v against rows one apart, in pixels, over the slices of a
// row walk: under 1, less a margin, so that its first row stays above the
// tile origin (which has a pixel of margin).
constexpr double kSpanDrift = 0.95;
// Tile, brick and workgroup of a back-projection launch.
TileShape bp_tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                        const ViewBatch& vb, bool direct);
// Bytes of an adjoint tile's pixel in 32-bit sums (in 64-bit ones twice as many),
// a launch's dynamic LDS, and its launches.
constexpr int32_t fp_entry_bytes(bool mirror) { return mirror ? 8 : 4; }
constexpr int32_t fp_lds_bytes(const TileShape& ts, bool mirror) {
  return ts.vc * (ts.tu + 1) * ts.tvp * fp_entry_bytes(mirror) * (ts.wide ? 2 : 1);
}
TileShape fp_tile_shape(const fdk_geometry* g, const GeoConst& gc, const SliceRun& run,
                        const ViewBatch& vb, bool direct);
// Plain (unmirrored) back-projection runs: 32 slices per brick, the tile
// holding (q, dq/du) of the main rows only; a prefetch slot holds one row's
// pair instead of two, so twice as many fit the same registers.
constexpr int kPlainBrickZ = 2 * kBrickZ;
constexpr int kPlainEntryBytes = 8;
constexpr int kPlainPrefetchSlots = 2 * kPrefetchSlots;

// Launchers (defined in the .hip files). They return a hipError_t as int.
int launch_backproject(const GeoConst& gc, const SliceRun& run, const ViewBatch& vb,
                       const TileShape& ts, const void* q, fdk_dtype q_dtype,
                       int64_t view_stride, float* vol, float scale, int accumulate,
                       void* stream);
int launch_forward_project(const GeoConst& gc, const SliceRun& run, const FpBatch& fb,
                           const TileShape& ts, const float* vol, float* q, int64_t view_stride,
                           float scale, bool fixed_sums, void* stream);
int launch_fill_zero(float* p, int64_t n, void* stream);
}  // namespace fdk
