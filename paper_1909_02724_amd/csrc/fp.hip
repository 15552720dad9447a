// Adjoint of the back-projection (forward projection) for gfx950: every
// voxel scatters scale * W * w_tap * vol into its four taps, with exactly the
// coordinates and weights of the matching back-projection variant (same
// brick setup, brick.h; FP32 columns for the tiled variant, FP64 columns for
// wide tiles and the direct one), so each is the transpose of its back-projector up to
// rounding.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "brick.h"

namespace fdk {
namespace {

// Tiled variant: per view, the brick's splats accumulate in LDS tiles with
// the back-projector's transposed layout (one more column, for the u + 1
// taps) as 32-bit fixed point, a row's and its mirror row's sums paired in
// one 64-bit word (FP32 for bricks that need it, one plane for main rows
// and one for mirror rows); the tiles are then added to the projection with
// one global atomic per non-zero pixel. Direct variant: global atomics per
// tap.

__device__ __forceinline__ void splat(float* __restrict__ qs, int32_t nu, int32_t nv, int32_t a,
                                      float du, int32_t ra, int32_t rb, float fr, float val) {
  const float wa = val * (1.0f - fr), wb = val * fr;
  const float w[4] = {wa * (1.0f - du), wa * du, wb * (1.0f - du), wb * du};
  const int32_t cols[4] = {a, a + 1, a, a + 1};
  const int32_t rows[4] = {ra, ra, rb, rb};
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (static_cast<uint32_t>(cols[m]) < static_cast<uint32_t>(nu) &&
        static_cast<uint32_t>(rows[m]) < static_cast<uint32_t>(nv))
      unsafeAtomicAdd(qs + static_cast<int64_t>(rows[m]) * nu + cols[m], w[m]);
  }
}

// Slot order of a lane in the adjoint. The LDS serves 64-bit adds 16 lanes and
// 32-bit ones 32 lanes at a time; lanes of such a group that add to one bank
// take turns, and to one address twice over (measured: m lanes on one
// address take 2m - 1 turns). Lanes along a ray share a detector column, so
// groups of 16 run across the rays (FpBatch), and each lane starts its
// 16 slots at another one, so that lanes that share a column all the same are
// on different rows: at (a in + b (out mod 4)) mod 16, with `in` the lane's
// place in its group and `out` the group's.
// The row walk (HALVES) knows two starts only, slot 0 and slot 8, by the
// parity of in + out. In a model of the addresses over all angles, at 0.75 to
// 1.33 pixels a voxel, its 64-bit adds then take 8.3 clocks a wave
// instruction (6.2 without a meeting; 40 to 100 with groups along the rays).
__device__ __forceinline__ uint32_t slot_rotation(const FpBatch& fb, bool halves) {
  const uint32_t in = threadIdx.x % kBrickX, out = threadIdx.x / kBrickX;
  if (halves) return ((in + out) & 1u) * (kBrickZ / 2);
  return (static_cast<uint32_t>(fb.rot_a) * in + static_cast<uint32_t>(fb.rot_b) * (out & 3u)) &
         (kBrickZ - 1);
}

// Voxel values of the thread's column, scaled, in the lane's slot order:
// x[t] is slot sl = (t + rot) mod 16; xm[t] is its mirror (mirrored runs)
// or slot 16 + sl (plain runs, whose bricks hold 32 slices).
template <bool MIRROR>
__device__ __forceinline__ void load_voxels(const GeoConst& gc, const SliceRun& run,
                                            const BrickCoords& bc, const float* __restrict__ vol,
                                            float scale, uint32_t rot, float* x, float* xm) {
  const int64_t slice = static_cast<int64_t>(gc.nx) * gc.ny;
  const int64_t col = static_cast<int64_t>(bc.j) * gc.nx + bc.i;
  // Every load is issued, at a slice clamped to the run, and what is not the
  // thread's is dropped: no branch, so all loads are in flight together.
  const int32_t top = run.n - 1 - bc.t0;
#pragma unroll
  for (int t = 0; t < kBrickZ; ++t) {
    const int32_t sl = static_cast<int32_t>((t + rot) & (kBrickZ - 1));
    const float v = vol[static_cast<int64_t>(run.loc_lo + bc.t0 + min(sl, top)) * slice + col];
    x[t] = bc.owner && sl <= top ? scale * v : 0.0f;
    const int32_t up = MIRROR ? min(sl, top) : min(kBrickZ + sl, top);
    const float m = vol[static_cast<int64_t>(MIRROR ? run.loc_hi - bc.t0 - up : run.loc_lo + bc.t0 + up) * slice + col];
    xm[t] = bc.owner && (MIRROR ? sl : kBrickZ + sl) <= top ? scale * m : 0.0f;
  }
}

// Accumulation for the tiled adjoint. LDS float atomics are serialised on
// gfx950: about 3 clocks per active lane per CU, 194 per full wave, against
// about 4.6 for a 32-bit integer add of a full wave and 6.4 for a 64-bit one
// (measured). A brick's splats therefore accumulate as 32-bit fixed point
// with integer LDS atomics (exact and independent of order within the
// workgroup), a tap's main and mirror sums in one 64-bit add, unless the
// brick spans a wide dynamic range: more than 1 % of its non-zero voxels
// lie below 2^-13 of its largest magnitude. Such a brick accumulates in
// 64-bit fixed point (the same scale rule with 2^63, one 64-bit add per
// tap), half a unit (about 2^-63 K M) per contribution: a voxel 2^-40 of
// the largest reaches a pixel through a full-weight tap at about 2^-24 K
// relative precision, so this serves bricks whose non-zero magnitudes span
// at most 2^40 (taps with weights near zero keep the absolute bound only).
// Two kinds take FP32 atomics (float tile, planar layout) instead:
//  - a brick with a NaN or an infinity, which integers cannot carry;
//  - a wide-range brick spanning more than 2^40, or one whose launch stages
//    a single view in 32 bits (its 64-bit tile would not fit).
// The wide kernel's tiles are sized for 64-bit sums and take them for every
// finite brick up to that range (with FDK_FIXED_SUMS, of any range).
// The FP32 path is slow (a workgroup on it can take longer than the rest of
// its launch), so it is kept for what fixed point cannot represent.
// On the FP32 path each pixel's sum carries FP32 rounding relative to its
// own contributions and non-finite values reach exactly the pixels they
// touch.
//
// Fixed-point scale, per brick and view, from a bound on what one pixel can
// receive:
//  - a column adds to the pixel columns floor(u) and floor(u) + 1, so pixel
//    column p hears only from columns with floor(u) in {p - 1, p};
//  - of a column's slices in the brick (16, or 32 for a plain run), those
//    with a tap on row r have v in [r - 1, r + 1): at most
//    floor(2 / (dv/dk)) + 2 of them (one spare for the rounding of v), and
//    never more than the brick's slice count;
//  - each contribution is at most M = max over columns of max|x| * W.
// K, the most contributions any pixel can receive, is bounded per brick and
// view from its corners (columns_at_pixel times slots_at_row, brick.h; on
// average 1.2 times the most any pixel does receive. A histogram of the
// columns' pixels gave the exact maximum, at two more barriers and column
// setups a stage and LDS atomics that all lanes send to a few addresses:
// 16.3 ms, of which 14.0 remained without it at 512^3 from 128 views).
// S = 2^31 / (1.01 K M) keeps every partial sum, rounding included, inside
// int32 (sum_scale; the voxels are scaled by a power of two to magnitudes below
// 1 first, so that it cannot overflow however small or large the values). A
// pixel's quantisation error is at most half a unit, about K M 2^-32, per
// contribution (one unit for splats above 2^23
// units, whose FP32 value is coarser than that anyway): relative to the
// brick's largest splat, not to the pixel's own sum, which is why
// wide-range bricks take 64 bits or FP32. (Rounded to a power of two, S wastes
// half a bit on average, and K's slack of 1.2 lost up to a bit more: a volume
// of one voxel in 500 at 1 and the rest at 2e-4 then projected with an error
// of 2.10e-6 against 64 bits, 2.01e-6 by the histogram's K, 1.84e-6 so.)
constexpr int kFpWideRangeLog2 = 13;        // "small" voxels: below 2^-13 of the brick's max
constexpr int kFpWideRangePct = 1;          // wide-range path above 1 % small voxels
constexpr int kFp64RangeLog2 = 40;          // 64-bit fixed point up to this magnitude range

// FP32 splat (FP32 path): taps (u, n), (u + 1, n), (u, n + 1),
// (u + 1, n + 1) of a tile with column pitch tvp.
__device__ __forceinline__ void splat_f32(float* p, int32_t tvp, float val, float fr, float du) {
  // (1 - fr) first: val - val fr would carry the rounding of val fr, up to
  // 2^-25 val, into a near-zero weight.
  const float fb = val * fr, fa = val * (1.0f - fr);
  const float du0 = 1.0f - du;
  atomicAdd(p, fa * du0);
  atomicAdd(p + tvp, fa * du);
  atomicAdd(p + 1, fb * du0);
  atomicAdd(p + tvp + 1, fb * du);
}

// Fixed point of x: floor(x + 0.5) in one conversion, exact below 2^23
// units and within one unit above (where the FP32 product feeding it is
// already coarser than a unit).
__device__ __forceinline__ int32_t fixed_round(float x) {
  int32_t r;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// Adds the fixed-point pair (a, b) to the 64-bit word at p, a into the low
// half and b into the high half: the addend is the 64-bit integer
// b 2^32 + a (a sign-extended), so every partial sum is exactly
// (sum b) 2^32 + (sum a), and both halves decode exactly while each sum
// stays inside int32. One 64-bit LDS add serves the row and its mirror.
__device__ __forceinline__ void add_pair(uint64_t* p, float a, float b) {
  const int32_t lo = fixed_round(a), hi = fixed_round(b);
  const uint64_t word = (static_cast<uint64_t>(static_cast<uint32_t>(hi + (lo >> 31))) << 32) |
                        static_cast<uint32_t>(lo);
  atomicAdd(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(word));
}

// Adds x, rounded to the nearest integer, to the 64-bit fixed-point sum at p.
__device__ __forceinline__ void add_fixed64(uint64_t* p, float x) {
  atomicAdd(reinterpret_cast<unsigned long long*>(p),
            static_cast<unsigned long long>(__float2ll_rn(x)));
}

// Largest of x over the wave, in lane 63: DPP moves within rows of 16 lanes,
// then row broadcasts.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#define FDK_DPP_MAX(ctrl, rows)                                                              \
  x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(                              \
                 0, static_cast<int>(x), ctrl, rows, 0xF, false)))
  FDK_DPP_MAX(0x111, 0xF);  // row_shr:1, 2, 4, 8
  FDK_DPP_MAX(0x112, 0xF);
  FDK_DPP_MAX(0x114, 0xF);
  FDK_DPP_MAX(0x118, 0xF);
  FDK_DPP_MAX(0x142, 0xA);  // row_bcast:15
  FDK_DPP_MAX(0x143, 0xC);  // row_bcast:31
#undef FDK_DPP_MAX
  return x;
}

// Row sums of kWalk slices of a column, the back-projector's row walk
// transposed. Where v drifts by less than a pixel against rows one apart over
// the slices, slice k has its taps in rows k, k + 1, k + 2 of the block's
// kWalk + 2 (weights 1 - a, a - b, b with a, b the clamped offsets), so each
// row is summed in a register and added to the tile once per pixel column: 40
// LDS adds per 16 slices (or pairs) instead of 64, at constant offsets, and
// 435 VALU instructions a wave and view instead of 600. The kernel stays
// bound by LDS adds (56 % of the cycles, 44 % of those for lanes that meet)
// beside VALU issue (44 % at the full rate). 512^3 from 128 views: 15.5 -> 9.4
// ms with the bounds, thread groups and tile pitch above; 215 x 190 x 171 at
// 1.2 pixels a voxel, which takes one slice at a time: 1.17 -> 0.69 ms.
//   emit(row, sum, sum of mirrors)
constexpr int kWalk = kBrickZ / 2;
template <bool MIRROR, class Emit>
__device__ __forceinline__ void walk_rows(float o, float eps, const float* x, const float* xm,
                                          Emit emit) {
  float c0 = 0.0f, c1 = 0.0f, m0 = 0.0f, m1 = 0.0f;  // pending sums of the next two rows
  const float o1 = o - 1.0f;
#pragma unroll
  for (int t = 0; t < kWalk; ++t) {
    const float a = __builtin_amdgcn_fmed3f(fmaf(static_cast<float>(t), eps, o), 0.0f, 1.0f);
    const float b = __builtin_amdgcn_fmed3f(fmaf(static_cast<float>(t), eps, o1), 0.0f, 1.0f);
    const float w0 = 1.0f - a, w1 = a - b;
    float msum = 0.0f;
    if constexpr (MIRROR) {
      msum = fmaf(xm[t], w0, m0);
      m0 = fmaf(xm[t], w1, m1);
      m1 = xm[t] * b;
    }
    emit(t, fmaf(x[t], w0, c0), msum);
    c0 = fmaf(x[t], w1, c1);
    c1 = x[t] * b;
    asm volatile("" ::: "memory");  // one step's values at a time in registers
  }
  emit(kWalk, c0, m0);
  emit(kWalk + 1, c1, m1);
}

// WIDE: tiles past the other kernels' stages (fp_tile_shape), with the direct
// kernel's FP64 columns (pixels up to 60 from the origin) and 64-bit sums,
// whose error is no larger than FP32 sums' (8.1e-7 against 8.4e-7 of FP64 at
// the size below; 32-bit ones, 30 % faster, have 9.1e-7). What was 8 global
// atomics a voxel and view, which bound the direct kernel, is one a pixel of
// the tile: 52 x 75 x 77 from 40 views at 1.33 pixels a voxel 1.69 -> 0.14 ms.
template <bool MIRROR, bool WALK, bool WIDE>
__device__ __forceinline__ void fp_tiled_body(const GeoConst& gc, const SliceRun& run,
                                              const FpBatch& fb, const TileShape& ts, const float* __restrict__ vol,
                                              float* __restrict__ q, int64_t vstride,
                                              float scale, int fixed_sums) {
  extern __shared__ __attribute__((aligned(16))) int atile[];
  // Of the chunk's views.
  __shared__ BrickView bvs[kFpMostViews];
  // 1.01 K times the largest W of the brick's columns; then the view's sum_scale,
  // and what a unit of its sums is worth.
  __shared__ float kw[kFpMostViews];
  __shared__ double units[kFpMostViews];
  __shared__ uint32_t amax_bits, amin_bits, n_nonzero, n_small, nonfinite;
  const int32_t tid = threadIdx.x;
  constexpr int BZ = MIRROR ? kBrickZ : kPlainBrickZ;  // slices per brick
  // blockIdx.y picks this workgroup's chunk of the launch's views.
  const ViewBatch& vb = fb.vb;
  const int32_t v_lo = fb.first[blockIdx.y], views = fb.first[blockIdx.y + 1] - v_lo;
  const BrickCoords bc = brick_coords(gc, run, ts, BZ,
                                      static_cast<int32_t>(blockIdx.y) >= fb.across_from);
  if (tid == 0) {
    amax_bits = n_nonzero = n_small = nonfinite = 0u;
    amin_bits = __float_as_uint(INFINITY);
  }
  const float kvf = static_cast<float>(gc.kv);
  if (tid < views) {
    const ViewGeo geo = view_geo(gc, vb.sn[v_lo + tid], vb.cs[v_lo + tid]);
    BrickView b = brick_setup(gc, geo, bc.i_lo, bc.i_hi, bc.j_lo,
                              bc.j_hi, bc.kb, 0, 0, BZ, MIRROR);
    // z is affine in (i, j): W, dv/dk and the drift of v are extremal at corners.
    float w = 0.0f, drift = 0.0f, dvk = INFINITY;
    for (int c = 0; c < 4; ++c) {
      const ColumnF32 col = column_f32(b, (c & 1) ? static_cast<float>(bc.i_hi - bc.i_lo) : 0.0f,
                                       (c & 2) ? static_cast<float>(bc.j_hi - bc.j_lo) : 0.0f, kvf);
      w = fmaxf(w, col.w);
      drift = fmaxf(drift, fabsf(col.eps));
      dvk = fminf(dvk, col.dvk);
    }
    kw[tid] = 1.01f * slots_at_row(dvk, BZ) *
              static_cast<float>(columns_at_pixel(gc, geo, bc.i_lo, bc.i_hi, bc.j_lo, bc.j_hi)) * w;
    b.inside = static_cast<float>(kWalk - 1) * drift <= static_cast<float>(kSpanDrift);  // the walk holds
    bvs[tid] = b;
  }
  const uint32_t rot = slot_rotation(fb, WALK);
  float x[kBrickZ], xm[kBrickZ];
  load_voxels<MIRROR>(gc, run, bc, vol, scale, rot, x, xm);
  // Brick statistics: largest and smallest non-zero magnitudes, non-finite
  // values (x - x is NaN exactly for those), then how many non-zero voxels
  // are small against the largest.
  float amax = 0.0f, amin = INFINITY;
  bool bad = false;
#pragma unroll
  for (int t = 0; t < kBrickZ; ++t) {
    amax = fmaxf(amax, fmaxf(fabsf(x[t]), fabsf(xm[t])));
    amin = fminf(amin, fminf(x[t] != 0.0f ? fabsf(x[t]) : INFINITY,
                             xm[t] != 0.0f ? fabsf(xm[t]) : INFINITY));
    bad = bad || ((x[t] - x[t]) != 0.0f) || ((xm[t] - xm[t]) != 0.0f);
  }
  __syncthreads();
  // One LDS atomic a wave (64 lanes on one address serialise). Non-negative
  // floats order as integers; the smallest is the largest complement.
  const bool last = (tid & (kWaveLanes - 1)) == kWaveLanes - 1;
  const uint32_t hi = wave_max(__float_as_uint(amax)), lo = ~wave_max(~__float_as_uint(amin));
  if (last) {
    atomicMax(&amax_bits, hi);
    atomicMin(&amin_bits, lo);
  }
  if (bad) nonfinite = 1u;
  __syncthreads();
  {
    const float small = ldexpf(__uint_as_float(amax_bits), -kFpWideRangeLog2);
    uint32_t nz = 0, ns = 0;
#pragma unroll
    for (int t = 0; t < kBrickZ; ++t) {
      nz += (x[t] != 0.0f) + (xm[t] != 0.0f);
      ns += (x[t] != 0.0f && fabsf(x[t]) < small) + (xm[t] != 0.0f && fabsf(xm[t]) < small);
    }
    // Sums over the wave bit by bit (a thread counts at most 32 voxels).
    uint32_t wnz = 0, wns = 0;
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      wnz += static_cast<uint32_t>(__popcll(__ballot((nz >> m) & 1u))) << m;
      wns += static_cast<uint32_t>(__popcll(__ballot((ns >> m) & 1u))) << m;
    }
    if (last) {
      atomicAdd(&n_nonzero, wnz);
      atomicAdd(&n_small, wns);
    }
  }
  __syncthreads();
  if (amax_bits == 0u && nonfinite == 0u) return;  // an all-zero brick adds nothing (uniform)
  // Accumulation of the brick (uniform): 32-bit fixed point; 64-bit fixed
  // point for a wide-range brick whose non-zero magnitudes span at most
  // 2^kFp64RangeLog2, with half the views per stage (its entries take twice
  // the bytes); FP32 for a brick with non-finite values, a wider range, or
  // when a stage holds a single view in 32 bits.
  // With fixed_sums every finite brick takes 32 bits. WIDE tiles hold 64-bit
  // sums of ts.vc views, and take them with fixed_sums whatever the range.
  const bool wide_range =
      WIDE || (!fixed_sums && 100u * n_small > static_cast<uint32_t>(kFpWideRangePct) * n_nonzero);
  const bool fixed64 = nonfinite == 0u && wide_range && (WIDE || ts.vc >= 2) &&
                       ((WIDE && fixed_sums) ||
                        __uint_as_float(amax_bits) <=
                            ldexpf(__uint_as_float(amin_bits), kFp64RangeLog2));
  const bool fp32_path = nonfinite != 0u || (wide_range && !fixed64);
  const int32_t vstep = fixed64 && !WIDE ? ts.vc / 2 : ts.vc;

  // Fixed point: the voxels are scaled by a power of two to magnitudes below
  // 1, so that neither their sums nor the scale of the sums leave FP32's
  // normal range whatever the volume's units are (the flush undoes it).
  int ex_max = 0;
  const float amax_1 = frexpf(__uint_as_float(amax_bits), &ex_max);
  if (!fp32_path) {
#pragma unroll
    for (int t = 0; t < kBrickZ; ++t) {
      x[t] = ldexpf(x[t], -ex_max);
      xm[t] = ldexpf(xm[t], -ex_max);
    }
    if (tid < views) {
      const float sum = sum_scale(kw[tid] * amax_1);
      int e;
      const float m = frexpf(sum, &e);
      double inv = rcp_f32(m);
      inv = fma(fma(-static_cast<double>(m), inv, 1.0), inv, inv);  // 1 / m to 2^-46
      units[tid] = sum > 0.0f ? ldexp(fixed64 ? 1.0 : inv, ex_max - e - (fixed64 ? 62 : 31)) : 0.0;
      kw[tid] = sum;
    }
  }
  const int32_t tuf = ts.tu + 1, tv = ts.tv, tvp = ts.tvp;
  const int32_t slot = tuf * tvp;
  const int32_t rstep = kThreads / tuf;
  const int32_t sr = tid / tuf, sc = tid - sr * tuf;
  // Tiles start at zero; the flush leaves them so for the next stage.
  for (int32_t e = tid; e < (MIRROR ? 2 : 1) * (WIDE ? 2 : 1) * ts.vc * slot; e += kThreads) atile[e] = 0;
  __syncthreads();
  int* const mtile = atile + ts.vc * slot;
  for (int32_t s0 = 0; s0 < views; s0 += vstep) {
    const int32_t nvc = min(vstep, views - s0);
    // Main rows in planes [0, vc) and mirror rows in planes [vc, 2 vc), one
    // 32-bit word per pixel: all LDS banks serve the adds (interleaved
    // (main, mirror) pairs reached only half of them and conflicted 10-way).
    // (The 32-bit fixed-point path of mirrored runs uses the same bytes as
    // 64-bit (main, mirror) words instead, the 64-bit one as 16-byte
    // (main, mirror) entries, and that of plain runs as 64-bit words.)
    if (bc.owner) {
      for (int32_t sl = 0; sl < nvc; ++sl) {
        const ColumnF32 c =
            WIDE ? column_f64(gc, view_geo(gc, vb.sn[v_lo + s0 + sl], vb.cs[v_lo + s0 + sl]), bvs[s0 + sl],
                              bc.i, bc.j, bc.kb)
                 : column_f32(bvs[s0 + sl], bc.txf, bc.tyf, kvf);
        const uint32_t nu = min(c.nu, static_cast<uint32_t>(ts.tu - 1));
        if (!fp32_path) {
          const float sum = kw[s0 + sl];
          if (!(sum > 0.0f)) continue;  // nothing reaches this view (uniform)
          const float du0 = 1.0f - c.du;
          if (WIDE || fixed64) {
            // S = 2^sh, at most 2^63 of that scale, applied to W x (at most M)
            // so that no intermediate overflows.
            int e;
            frexpf(sum, &e);
            const int sh = 62 + e;
            if constexpr (MIRROR) {
              uint64_t* const base =
                  reinterpret_cast<uint64_t*>(atile) + 2 * (sl * slot + nu * tvp + c.nvb);
              uint64_t* const base1 = base + 2 * tvp;  // pixel column u + 1
#pragma unroll
              for (int t = 0; t < kBrickZ; ++t) {
                uint32_t dn;
                float fr;
                voxel_row_off(c.fvb, c.dvk, static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn, &fr);
                const float val = ldexpf(c.w * x[t], sh), vm = ldexpf(c.w * xm[t], sh);
                const float wa = val * (1.0f - fr), wb = val * fr;
                const float ma = vm * (1.0f - fr), mb = vm * fr;
                uint64_t* const p = base + 2 * dn;
                uint64_t* const p1 = base1 + 2 * dn;
                add_fixed64(p, wa * du0);
                add_fixed64(p + 1, ma * du0);
                add_fixed64(p1, wa * c.du);
                add_fixed64(p1 + 1, ma * c.du);
                add_fixed64(p + 2, wb * du0);
                add_fixed64(p + 3, mb * du0);
                add_fixed64(p1 + 2, wb * c.du);
                add_fixed64(p1 + 3, mb * c.du);
              }
            } else {
              uint64_t* const base = reinterpret_cast<uint64_t*>(atile) + sl * slot + nu * tvp + c.nvb;
              uint64_t* const base1 = base + tvp;
#pragma unroll
              for (int t = 0; t < kBrickZ; ++t) {
                const int32_t tt = static_cast<int32_t>((t + rot) & (kBrickZ - 1));
                uint32_t dn, dn2;
                float fr, fr2;
                voxel_row_off(c.fvb, c.dvk, tt, &dn, &fr);
                voxel_row_off(c.fvb, c.dvk, kBrickZ + tt, &dn2, &fr2);
                const float val = ldexpf(c.w * x[t], sh), v2 = ldexpf(c.w * xm[t], sh);
                const float wa = val * (1.0f - fr), wb = val * fr;
                const float a2 = v2 * (1.0f - fr2), b2 = v2 * fr2;
                add_fixed64(base + dn, wa * du0);
                add_fixed64(base1 + dn, wa * c.du);
                add_fixed64(base + dn + 1, wb * du0);
                add_fixed64(base1 + dn + 1, wb * c.du);
                add_fixed64(base + dn2, a2 * du0);
                add_fixed64(base1 + dn2, a2 * c.du);
                add_fixed64(base + dn2 + 1, b2 * du0);
                add_fixed64(base1 + dn2 + 1, b2 * c.du);
              }
            }
            continue;
          }
          // W S, with the weights of the pixel columns u and u + 1.
          const float ws = c.w * sum * 0x1p31f, v0 = ws * du0, v1 = ws * c.du;
          if (WALK && __builtin_amdgcn_readfirstlane(bvs[s0 + sl].inside)) {
            // Blocks of kWalk slices, the lane's first one first.
            const float down = fminf(static_cast<float>(kWalk - 1) * c.eps, 0.0f);
#pragma unroll
            for (int p = 0; p < BZ / kWalk; ++p) {
              // First slice of block p of the column; its values are at kWalk (p mod 2).
              const int32_t k0 = (p & ~1) * kWalk + ((p & 1) ? kWalk - static_cast<int32_t>(rot)
                                                             : static_cast<int32_t>(rot));
              const float* const xs = (p < 2 ? x : xm) + (p & 1) * kWalk;
              const float o = fmaf(static_cast<float>(k0), c.eps, c.vl);
              const float n = floorf(o + down);
              const int32_t at = sl * slot + nu * tvp + k0 + static_cast<int32_t>(n);
              if constexpr (MIRROR) {
                uint64_t* const w = reinterpret_cast<uint64_t*>(atile) + at;
                uint64_t* const w1 = w + tvp;
                walk_rows<true>(o - n, c.eps, xs, xm + (p & 1) * kWalk,
                                [&](int r, float sum, float msum) {
                                  add_pair(w + r, sum * v0, msum * v0);
                                  add_pair(w1 + r, sum * v1, msum * v1);
                                });
              } else {
                int* const w = atile + at;
                int* const w1 = w + tvp;
                walk_rows<false>(o - n, c.eps, xs, nullptr, [&](int r, float sum, float) {
                  atomicAdd(w + r, fixed_round(sum * v0));
                  atomicAdd(w1 + r, fixed_round(sum * v1));
                });
              }
            }
            continue;
          }
          if constexpr (MIRROR) {
            // (main, mirror) pairs of 32-bit sums in 64-bit words.
            uint64_t* const base = reinterpret_cast<uint64_t*>(atile) + sl * slot + nu * tvp + c.nvb;
            uint64_t* const base1 = base + tvp;  // pixel column u + 1
#pragma unroll
            for (int t = 0; t < kBrickZ; ++t) {
              uint32_t dn;
              float fr;
              voxel_row_off(c.fvb, c.dvk, static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn, &fr);
              const float fa = 1.0f - fr;
              const float a0 = v0 * x[t], a1 = v1 * x[t], m0 = v0 * xm[t], m1 = v1 * xm[t];
              add_pair(base + dn, a0 * fa, m0 * fa);
              add_pair(base1 + dn, a1 * fa, m1 * fa);
              add_pair(base + dn + 1, a0 * fr, m0 * fr);
              add_pair(base1 + dn + 1, a1 * fr, m1 * fr);
            }
            continue;
          }
          int* const base = atile + sl * slot + nu * tvp + c.nvb;
          int* const base1 = base + tvp;  // pixel column u + 1
#pragma unroll
          for (int t = 0; t < kBrickZ; ++t) {
            uint32_t dn;
            float fr;
            voxel_row_off(c.fvb, c.dvk, static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn, &fr);
            const float fa = 1.0f - fr, a0 = v0 * x[t], a1 = v1 * x[t];
            atomicAdd(base + dn, fixed_round(a0 * fa));
            atomicAdd(base1 + dn, fixed_round(a1 * fa));
            atomicAdd(base + dn + 1, fixed_round(a0 * fr));
            atomicAdd(base1 + dn + 1, fixed_round(a1 * fr));
            {
              // The brick's upper 16 slices, into the same plane.
              uint32_t dn2;
              float fr2;
              voxel_row_off(c.fvb, c.dvk,
                            kBrickZ + static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn2, &fr2);
              const float fa2 = 1.0f - fr2, b0 = v0 * xm[t], b1 = v1 * xm[t];
              atomicAdd(base + dn2, fixed_round(b0 * fa2));
              atomicAdd(base1 + dn2, fixed_round(b1 * fa2));
              atomicAdd(base + dn2 + 1, fixed_round(b0 * fr2));
              atomicAdd(base1 + dn2 + 1, fixed_round(b1 * fr2));
            }
          }
        } else {
          float* const fbase = reinterpret_cast<float*>(atile) + sl * slot + nu * tvp + c.nvb;
          float* const fmbase = reinterpret_cast<float*>(mtile) + sl * slot + nu * tvp + c.nvb;
#pragma unroll
          for (int t = 0; t < kBrickZ; ++t) {
            uint32_t dn;
            float fr;
            voxel_row_off(c.fvb, c.dvk, static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn, &fr);
            splat_f32(fbase + dn, tvp, c.w * x[t], fr, c.du);
            if (MIRROR) {
              splat_f32(fmbase + dn, tvp, c.w * xm[t], fr, c.du);
            } else {
              uint32_t dn2;
              float fr2;
              voxel_row_off(c.fvb, c.dvk,
                            kBrickZ + static_cast<int32_t>((t + rot) & (kBrickZ - 1)), &dn2, &fr2);
              splat_f32(fbase + dn2, tvp, c.w * xm[t], fr2, c.du);
            }
          }
        }
      }
    }
    __syncthreads();
    // Flush: entry (r, c) holds pixel (org_u + c, org_v + r) and, for
    // mirrored runs, pixel (org_u + c, G - org_v - r).
    if (sr < rstep) {
      for (int32_t sl = 0; sl < nvc; ++sl) {
        const int32_t s = s0 + sl;
        const int32_t gu = bvs[s].org_u + sc;
        const bool on = static_cast<uint32_t>(gu) < static_cast<uint32_t>(gc.nu);
        // In FP64, so that a pixel's sum is rounded once (unused on the FP32 path).
        const double unit = units[s];
        float* qs = q + fb.idx[v_lo + s] * vstride + gu;
        for (int32_t r = sr; r < tv; r += rstep) {
          const int32_t at = sl * slot + sc * tvp + r;
          float ex, ey = 0.0f;
          if (fp32_path) {
            ex = __int_as_float(atile[at]);
            atile[at] = 0;
            if (MIRROR) {
              ey = __int_as_float(mtile[at]);
              mtile[at] = 0;
            }
          } else if (fixed64) {
            int64_t* const w = reinterpret_cast<int64_t*>(atile) + (MIRROR ? 2 * at : at);
            ex = static_cast<float>(static_cast<double>(w[0]) * unit);
            w[0] = 0;
            if (MIRROR) {
              ey = static_cast<float>(static_cast<double>(w[1]) * unit);
              w[1] = 0;
            }
          } else if (MIRROR) {
            // Word = (mirror sum) 2^32 + (main sum), both int32.
            uint64_t* const p = reinterpret_cast<uint64_t*>(atile) + at;
            const uint64_t w = *p;
            *p = 0;
            const int32_t lo = static_cast<int32_t>(static_cast<uint32_t>(w));
            const int32_t hi = static_cast<int32_t>((w - static_cast<uint64_t>(static_cast<int64_t>(lo))) >> 32);
            ex = static_cast<float>(lo * unit);
            ey = static_cast<float>(hi * unit);
          } else {
            ex = static_cast<float>(atile[at] * unit);
            atile[at] = 0;
          }
          const int32_t gr = bvs[s].org_v + r;
          if (on && ex != 0.0f && static_cast<uint32_t>(gr) < static_cast<uint32_t>(gc.nv))
            unsafeAtomicAdd(qs + static_cast<int64_t>(gr) * gc.nu, ex);
          if (MIRROR) {
            const int32_t gm = gc.mirror_g - gr;
            if (on && ey != 0.0f && static_cast<uint32_t>(gm) < static_cast<uint32_t>(gc.nv))
              unsafeAtomicAdd(qs + static_cast<int64_t>(gm) * gc.nu, ey);
          }
        }
      }
    }
    __syncthreads();
  }
}

// Mirrored runs that take one slice at a time: six 256-thread workgroups per CU
// (80 VGPRs). The 64-bit paths' code otherwise lifts the register count past
// it, and five workgroups cost 11 % at 2048^3. Those that walk: five (96
// VGPRs; six spill, 1 % faster at 512^3 and 5 to 24 % slower at 64^3 to 256^3).
// (Held to 80 registers, the plain variant spills inside its splat loops, so
// it keeps its count.)
template <bool WALK>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(WALK ? 5 : 6)))
void fp_mirror_kernel(GeoConst gc, SliceRun run, FpBatch fb, TileShape ts,
                      const float* __restrict__ vol, float* __restrict__ q, int64_t vstride,
                      float scale, int fixed_sums) {
  fp_tiled_body<true, WALK, false>(gc, run, fb, ts, vol, q, vstride, scale, fixed_sums);
}

template <bool WALK>
__global__ __launch_bounds__(kThreads)
void fp_plain_kernel(GeoConst gc, SliceRun run, FpBatch fb, TileShape ts,
                     const float* __restrict__ vol, float* __restrict__ q, int64_t vstride,
                     float scale, int fixed_sums) {
  fp_tiled_body<false, WALK, false>(gc, run, fb, ts, vol, q, vstride, scale, fixed_sums);
}

template <bool MIRROR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void fp_wide_kernel(GeoConst gc, SliceRun run, FpBatch fb, TileShape ts,
                    const float* __restrict__ vol, float* __restrict__ q, int64_t vstride,
                    float scale, int fixed_sums) {
  fp_tiled_body<MIRROR, false, true>(gc, run, fb, ts, vol, q, vstride, scale, fixed_sums);
}

template <bool MIRROR>
__global__ __launch_bounds__(kThreads) void fp_direct_kernel(GeoConst gc, SliceRun run,
                                                             FpBatch fb, TileShape ts,
                                                             const float* __restrict__ vol,
                                                             float* __restrict__ q,
                                                             int64_t vstride, float scale) {
  __shared__ BrickView bvs[kMaxViewsPerLaunch];
  const ViewBatch& vb = fb.vb;
  const int32_t tid = threadIdx.x;
  constexpr int BZ = MIRROR ? kBrickZ : kPlainBrickZ;  // slices per brick
  const BrickCoords bc = brick_coords(gc, run, ts, BZ);
  if (tid < vb.nviews)
    bvs[tid] = brick_setup(gc, view_geo(gc, vb.sn[tid], vb.cs[tid]), bc.i_lo, bc.i_hi, bc.j_lo, bc.j_hi, bc.kb, 0, 0, BZ,
                           MIRROR);
  const uint32_t rot = slot_rotation(fb, false);
  float x[kBrickZ], xm[kBrickZ];
  load_voxels<MIRROR>(gc, run, bc, vol, scale, rot, x, xm);
  __syncthreads();
  if (!bc.owner) return;
  for (int32_t s = 0; s < vb.nviews; ++s) {
    const ColumnF32 c = column_f64(gc, view_geo(gc, vb.sn[s], vb.cs[s]), bvs[s], bc.i, bc.j, bc.kb);
    float* qs = q + fb.idx[s] * vstride;
    const int32_t a = bvs[s].org_u + static_cast<int32_t>(c.nu);
    const int32_t nb = bvs[s].org_v + static_cast<int32_t>(c.nvb);
#pragma unroll
    for (int t = 0; t < kBrickZ; ++t) {
      const int32_t sl = static_cast<int32_t>((t + rot) & (kBrickZ - 1));
      if (bc.t0 + sl >= run.n) continue;
      uint32_t dn;
      float fr;
      voxel_row_off(c.fvb, c.dvk, sl, &dn, &fr);
      const int32_t n = nb + static_cast<int32_t>(dn);
      splat(qs, gc.nu, gc.nv, a, c.du, n, n + 1, fr, c.w * x[t]);
      if (MIRROR) {
        const int32_t m = gc.mirror_g - n;
        splat(qs, gc.nu, gc.nv, a, c.du, m, m - 1, fr, c.w * xm[t]);
      } else if (bc.t0 + kBrickZ + sl < run.n) {
        uint32_t dn2;
        float fr2;
        voxel_row_off(c.fvb, c.dvk, kBrickZ + sl, &dn2, &fr2);
        const int32_t n2 = nb + static_cast<int32_t>(dn2);
        splat(qs, gc.nu, gc.nv, a, c.du, n2, n2 + 1, fr2, c.w * xm[t]);
      }
    }
  }
}

__global__ void fill_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t m = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; m < n; m += stride)
    p[m] = 0.0f;
}

}  // namespace

int launch_forward_project(const GeoConst& gc, const SliceRun& run, const FpBatch& fb,
                           const TileShape& ts, const float* vol, float* q, int64_t vstride,
                           float scale, bool fixed_sums, void* stream) {
  const uint64_t nwg = static_cast<uint64_t>(ts.nbx) * ts.nby * ts.nseg;
  const dim3 block(kThreads);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ts.vc > 0) {
    const dim3 grid(static_cast<uint32_t>(nwg), static_cast<uint32_t>(fb.nchunks));
    const int32_t lds = fp_lds_bytes(ts, run.mirror != 0);
    const auto kernel =
        ts.wide ? (run.mirror ? &fp_wide_kernel<true> : &fp_wide_kernel<false>)
        : run.mirror ? (ts.span >= kWalk ? &fp_mirror_kernel<true> : &fp_mirror_kernel<false>)
                     : (ts.span >= kWalk ? &fp_plain_kernel<true> : &fp_plain_kernel<false>);
    if (lds > 65536 - 5 * 1024) {  // beside the static LDS; always the same limit (it is the kernel's, not the launch's)
      const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 kFpWideMostLdsBytes);
      if (err != hipSuccess) return static_cast<int>(err);
    }
    hipLaunchKernelGGL(kernel, grid, block, lds, st, gc, run, fb, ts, vol, q, vstride, scale,
                       static_cast<int>(fixed_sums));
  } else {
    const dim3 grid(static_cast<uint32_t>(nwg));
    if (run.mirror)
      hipLaunchKernelGGL((fp_direct_kernel<true>), grid, block, 0, st, gc, run, fb, ts, vol, q,
                         vstride, scale);
    else
      hipLaunchKernelGGL((fp_direct_kernel<false>), grid, block, 0, st, gc, run, fb, ts, vol, q,
                         vstride, scale);
  }
  return static_cast<int>(hipGetLastError());
}

int launch_fill_zero(float* p, int64_t n, void* stream) {
  if (n <= 0) return 0;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), p, n);
  return static_cast<int>(hipGetLastError());
}

}  // namespace fdk
