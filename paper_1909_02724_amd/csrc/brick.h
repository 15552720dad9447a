// Brick geometry shared by the back-projector and its adjoint (gfx950).
//
// A workgroup of 256 threads owns a brick of 16 x 16 (x, y) columns and 16
// consecutive slices of a slice run; for a mirrored run (Theorem 1) each
// thread also owns the 16 mirror voxels of its column.
//
// Coordinates. For each (brick, view) one lane evaluates, in FP64, the
// tile origin (the floor of the smallest u and v over the brick's corners,
// minus one pixel) and a handful of brick constants; every thread then
// derives its column's u, v(kb), W = f^2 and dv/dk in FP32 from offsets
// relative to the brick origin (Theorems 2 and 3: u and z, hence f, are
// fixed along the column; v is affine in k). All FP32 quantities are small
// offsets, which keeps coordinates accurate to a few 1e-6 pixel at 4096
// pixels. Per voxel: v = v(kb) + t dv/dk, one truncation, one fraction.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "geom_device.h"

namespace fdk {
namespace {

constexpr int kThreads = kBrickThreads;

template <typename T>
__device__ __forceinline__ float tap(const T* __restrict__ qs, int32_t nu, int32_t nv, int32_t a,
                                     int32_t b) {
  // Taps outside the detector read zero.
  return (static_cast<uint32_t>(a) < static_cast<uint32_t>(nu) &&
          static_cast<uint32_t>(b) < static_cast<uint32_t>(nv))
             ? to_f32(qs[static_cast<int64_t>(b) * nu + a])
             : 0.0f;
}

// Per (brick, view) constants. With tx = i - i_lo, ty = j - j_lo and
// dz = ci tx + cj ty, f = 1 / (zo + dz):
//   u    - org_u = uo + (au tx + bu ty) f
//   v(kb) - org_v = vo + (av tx + bv ty) f
// (from u = cu + ku a / z and v = cv + kv (k - cz) / z, expanded about the
// brick origin column so every FP32 term is a small offset).
struct BrickView {
  float uo, vo, au, bu, av, bv, zo, ci, cj;
  int32_t org_u, org_v;
  // The tile (columns org_u .. org_u + tu, its rows and mirror rows) is on the
  // detector; in the adjoint, which sums off it too, that its row walk holds.
  int32_t inside;
};

// bz: slices per brick; mirror: whether the tile also holds the mirror rows
// (then `inside` requires them on the detector too). Also compiled for the
// host, where a test checks the tile bounds against every voxel's taps.
__host__ __device__ inline BrickView brick_setup(const GeoConst& gc, const ViewGeo& g, int32_t i_lo, int32_t i_hi,
                                 int32_t j_lo, int32_t j_hi, int32_t kb, int32_t tu = 0,
                                 int32_t tv = 0, int32_t bz = kBrickZ, bool mirror = true) {
  const double k0 = static_cast<double>(kb) - gc.cz;
  const double k1 = static_cast<double>(kb + bz - 1) - gc.cz;
  // u is a ratio of functions affine in (i, j) and v is affine in k at
  // fixed f: over the brick's (i, j, k) box both are extremal at corners.
  double umin = INFINITY, vmin = INFINITY;
  for (int c = 0; c < 4; ++c) {
    const double di = (c & 1) ? i_hi : i_lo, dj = (c & 2) ? j_hi : j_lo;
    const double z = fma(g.ci, di, fma(g.cj, dj, g.c0));
    const double f = 1.0 / z;
    const double a = fma(g.ai, di, fma(g.aj, dj, g.a0));
    umin = fmin(umin, fma(gc.ku * a, f, gc.cu));
    vmin = fmin(vmin, fmin(fma(gc.kv * k0, f, gc.cv), fma(gc.kv * k1, f, gc.cv)));
  }
  BrickView b;
  b.org_u = static_cast<int32_t>(floor(umin)) - 1;
  b.org_v = static_cast<int32_t>(floor(vmin)) - 1;
  const double zo = fma(g.ci, static_cast<double>(i_lo), fma(g.cj, static_cast<double>(j_lo), g.c0));
  const double fo = 1.0 / zo;
  const double ao = fma(g.ai, static_cast<double>(i_lo), fma(g.aj, static_cast<double>(j_lo), g.a0));
  const double ro = ao * fo;                 // a / z at the brick origin
  const double K = gc.kv * k0;               // v(kb) - cv = K f
  b.uo = static_cast<float>((gc.cu - b.org_u) + gc.ku * ro);
  b.vo = static_cast<float>((gc.cv - b.org_v) + K * fo);
  b.au = static_cast<float>(gc.ku * (g.ai - ro * g.ci));
  b.bu = static_cast<float>(gc.ku * (g.aj - ro * g.cj));
  b.av = static_cast<float>(-K * fo * g.ci);
  b.bv = static_cast<float>(-K * fo * g.cj);
  b.zo = static_cast<float>(zo);
  b.ci = static_cast<float>(g.ci);
  b.cj = static_cast<float>(g.cj);
  const bool cols_in = b.org_u >= 0 && b.org_u + tu < gc.nu;
  const bool rows_in = b.org_v >= 0 && b.org_v + tv <= gc.nv;
  // (mirror_g is INT32_MIN when there is no pixel-aligned mirror: only
  // mirrored runs, which have one, evaluate it.)
  const bool mirror_in =
      !mirror || (gc.mirror_g - b.org_v < gc.nv && gc.mirror_g - b.org_v - tv + 1 >= 0);
  b.inside = tu > 0 && cols_in && rows_in && mirror_in;
  return b;
}

// Where a staged tile is read from: its first column and row and the mirror of
// its first row, drawn in to at most one tile (reach rows) off the detector, so
// that every row off it lies off the buffer as well: above it at an offset
// below zero, which wraps, and below it at or past the end. stage_reach_ok keeps
// both, and lanes that start from kBadLane, within 32 bits.
constexpr uint32_t kBadLane = 0x80000000u;
struct StageOrigin {
  int32_t u, v, vm;
};
__host__ __device__ __forceinline__ int32_t clamp_i32(int32_t x, int32_t lo, int32_t hi) {
  return x < lo ? lo : x > hi ? hi : x;
}
__host__ __device__ __forceinline__ StageOrigin stage_origin(const GeoConst& gc, int32_t org_u,
                                                             int32_t org_v, int32_t reach,
                                                             bool mirror) {
  return StageOrigin{clamp_i32(org_u, -kBrickThreads, gc.nu), clamp_i32(org_v, -reach, gc.nv),
                     mirror ? clamp_i32(gc.mirror_g - org_v, -1, gc.nv + reach) : 0};
}
// Offset of a lane's pixel in pass 0; lane is its own part, row * row_es + column * es.
__host__ __device__ __forceinline__ uint32_t stage_offset(uint32_t lane, int32_t u, int32_t row,
                                                          uint32_t row_es, uint32_t es) {
  return lane + (static_cast<uint32_t>(row) * row_es + static_cast<uint32_t>(u) * es);
}

// FP32 column quantities of one view for a thread at (tx, ty) in the brick.
struct ColumnF32 {
  uint32_t nu, nvb;  // tile column and first row (relative to the origin)
  float du, fvb;     // fractions of u and of v(kb)
  float w, dvk;      // W_dis = f^2 and dv/dk
  float vl, eps;     // v(kb) relative to the origin, and dv/dk - 1
};

// Hardware reciprocal (1 ulp) and fraction on the GPU; the host build, used
// only by the tile-bound test, takes the correctly rounded forms.
__host__ __device__ __forceinline__ float rcp_f32(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
__host__ __device__ __forceinline__ float fract_f32(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_fractf(x);
#else
  return x - floorf(x);
#endif
}

__host__ __device__ __forceinline__ ColumnF32 column_f32(const BrickView& b, float txf, float tyf,
                                                         float kvf) {
  const float f = rcp_f32(b.zo + fmaf(b.ci, txf, b.cj * tyf));
  const float ul = fmaf(fmaf(b.au, txf, b.bu * tyf), f, b.uo);
  const float vl = fmaf(fmaf(b.av, txf, b.bv * tyf), f, b.vo);
  ColumnF32 c;
  c.nu = static_cast<uint32_t>(ul);  // ul, vl >= 1 by the origin margin
  c.du = fract_f32(ul);
  c.nvb = static_cast<uint32_t>(vl);
  c.fvb = fract_f32(vl);
  c.vl = vl;
  c.w = f * f;
  c.dvk = kvf * f;
  c.eps = fmaf(kvf, f, -1.0f);
  return c;
}

// Row walk of slices [k0, k0 + span) of a column: the first of its rows, the
// one above the smallest v less the slice's place (a row above one that v lies
// on), and the first slice's v against the row after.
struct WalkStart {
  int32_t row;
  float x;
};
__host__ __device__ __forceinline__ WalkStart walk_start(const ColumnF32& c, int32_t k0, int32_t span) {
  const float o = k0 ? fmaf(static_cast<float>(k0), c.eps, c.vl) : c.vl;
  const float next = ceilf(o + fminf(static_cast<float>(span - 1) * c.eps, 0.0f));
  return WalkStart{k0 - 1 + static_cast<int32_t>(next), o - next};
}

// The same quantities computed per column in FP64 (direct variant: it runs
// when footprints are too large for LDS, i.e. at strong magnification,
// where brick-relative FP32 offsets would span hundreds of pixels).
// Indices are relative to the brick's tile origin, as in column_f32.
__device__ __forceinline__ ColumnF32 column_f64(const GeoConst& gc, const ViewGeo& g,
                                                const BrickView& b, int32_t i, int32_t j,
                                                int32_t kb) {
  const double di = static_cast<double>(i), dj = static_cast<double>(j);
  const double z = fma(g.ci, di, fma(g.cj, dj, g.c0));
  const double f = 1.0 / z;
  const double a = fma(g.ai, di, fma(g.aj, dj, g.a0));
  const double ul = fma(gc.ku * a, f, gc.cu) - b.org_u;  // exact: integer shift
  const double vl = fma(gc.kv * (static_cast<double>(kb) - gc.cz), f, gc.cv) - b.org_v;
  const double fu = floor(ul), fv = floor(vl);
  ColumnF32 c;
  c.nu = static_cast<uint32_t>(fu);
  c.du = static_cast<float>(ul - fu);
  c.nvb = static_cast<uint32_t>(fv);
  c.fvb = static_cast<float>(vl - fv);
  c.vl = static_cast<float>(vl);
  c.w = static_cast<float>(f * f);
  c.dvk = static_cast<float>(gc.kv * f);
  c.eps = static_cast<float>(gc.kv * f - 1.0);
  return c;
}

// Bounds for the adjoint's fixed-point sums. Most columns of the brick with
// floor(u) in {p - 1, p} for any p. Along a row of the brick
// u(i + 1) - u(i) = ku (ai z - a ci)(j) / (z z'), whose numerator depends on j
// alone and is affine in it, so the smallest spacing follows from the brick's
// corners; an interval of two pixels then holds at most ceil(2 / spacing) of a
// row's columns (2.002: rounding of u). Likewise along j; the smaller total holds.
__host__ __device__ inline int32_t columns_at_pixel(const GeoConst& gc, const ViewGeo& g, int32_t i_lo,
                                                    int32_t i_hi, int32_t j_lo, int32_t j_hi) {
  const int32_t ni = i_hi - i_lo + 1, nj = j_hi - j_lo + 1;
  double zmax = 0.0;
  for (int c = 0; c < 4; ++c)
    zmax = fmax(zmax, fma(g.ci, (c & 1) ? i_hi : i_lo, fma(g.cj, (c & 2) ? j_hi : j_lo, g.c0)));
  auto most = [&](double m, double n0, int32_t lo, int32_t hi, int32_t len) {
    const double p = fma(m, lo, n0), q = fma(m, hi, n0);
    const float spacing = p * q > 0.0 ? static_cast<float>(gc.ku * fmin(fabs(p), fabs(q)) / (zmax * zmax)) : 0.0f;
    const float n = spacing > 0.0f ? ceilf(2.002f / spacing) : INFINITY;
    return n < static_cast<float>(len) ? static_cast<int32_t>(n) : len;
  };
  const double m = g.ai * g.cj - g.ci * g.aj;
  const int32_t along_i = most(m, g.ai * g.c0 - g.ci * g.a0, j_lo, j_hi, ni);
  const int32_t along_j = most(-m, g.aj * g.c0 - g.cj * g.a0, i_lo, i_hi, nj);
  const int32_t a = along_i * nj, b = along_j * ni;
  return a < b ? a : b;
}

// Most slices of a column (of bz in the brick) with a tap on one row: those
// with v in [r - 1, r + 1), one spare for the rounding of v. dvk: the
// smallest dv/dk.
__host__ __device__ inline float slots_at_row(float dvk, int32_t bz) {
  return fminf(static_cast<float>(bz), floorf(2.0f / dvk) + 2.0f);
}

// Scale of a view's fixed-point sums, as a fraction of the integers' range: 1
// over the bound km on a pixel's sum (which carries 1 % for the rounding of this
// and of the sums). Not rounded to a power of two, which would leave up to a bit
// of the range unused.
__host__ __device__ inline float sum_scale(float km) {
  if (!(km > 0.0f)) return 0.0f;
  int e;
  const float m = frexpf(fmaxf(km, 0x1p-126f), &e);
  return ldexpf(rcp_f32(m), -e);
}

struct BrickCoords {
  int32_t i_lo, i_hi, j_lo, j_hi, i, j, t0, kb;
  float txf, tyf;
  bool owner;
};

// Brick (bx, by, z-segment) of this workgroup. Workgroups are dealt
// round-robin to the 8 XCDs, and each XCD takes a contiguous range of a
// linear order that runs over z-segments outermost and, within a segment,
// over bands of kBandRows brick rows, column by column. The workgroups an
// XCD holds at once (32 CUs x 4) then form a compact patch of bricks, about
// 16 x 8, whose detector footprints overlap from brick to brick, so that its
// L2 serves most of their taps (a row of bricks across the volume did not).
constexpr uint32_t kBandRows = 8;
__device__ __forceinline__ void brick_index(const TileShape& ts, int32_t* bx, int32_t* by,
                                            int32_t* seg) {
  const uint32_t nwg = gridDim.x;
  uint32_t lin = blockIdx.x;
  if ((nwg & 7u) == 0) lin = (lin & 7u) * (nwg >> 3) + (lin >> 3);
  const uint32_t nbx = static_cast<uint32_t>(ts.nbx), nby = static_cast<uint32_t>(ts.nby);
  const uint32_t plane = nbx * nby;
  const uint32_t sg = lin / plane, r = lin - sg * plane;
  const uint32_t band = r / (kBandRows * nbx);
  const uint32_t rows = min(kBandRows, nby - band * kBandRows);
  const uint32_t rb = r - band * kBandRows * nbx;
  *bx = static_cast<int32_t>(rb / rows);
  *by = static_cast<int32_t>(band * kBandRows + rb % rows);
  *seg = static_cast<int32_t>(sg);
}

// across: groups of 16 threads run along y instead of x.
__device__ __forceinline__ BrickCoords brick_coords(const GeoConst& gc, const SliceRun& run,
                                                    const TileShape& ts, int32_t bz = kBrickZ,
                                                    bool across = false) {
  int32_t bx, by, seg;
  brick_index(ts, &bx, &by, &seg);
  BrickCoords bc;
  bc.i_lo = bx * kBrickX;
  bc.j_lo = by * kBrickY;
  bc.i_hi = min(bc.i_lo + kBrickX - 1, gc.nx - 1);
  bc.j_hi = min(bc.j_lo + kBrickY - 1, gc.ny - 1);
  static_assert(kBrickX == kBrickY, "threads run along x or y");
  const int32_t in = threadIdx.x % kBrickX, out = threadIdx.x / kBrickX;
  const int32_t tx0 = across ? out : in, ty0 = across ? in : out;
  bc.owner = (bc.i_lo + tx0 <= bc.i_hi) && (bc.j_lo + ty0 <= bc.j_hi);
  bc.i = min(bc.i_lo + tx0, bc.i_hi);
  bc.j = min(bc.j_lo + ty0, bc.j_hi);
  bc.txf = static_cast<float>(bc.i - bc.i_lo);
  bc.tyf = static_cast<float>(bc.j - bc.j_lo);
  bc.t0 = seg * bz;
  bc.kb = run.k_first + bc.t0;
  return bc;
}

}  // namespace
}  // namespace fdk
