// The gfx950 pair kernel of libdisthist and its distance arithmetic.
// dh_pairs.hip instantiates it.
//
// The pair kernel is persistent: a grid of a few workgroups per CU drains a
// work list of (frame, histogram, bin window, i-block, j-range) items through
// an atomic counter. Its waves draw units of an item (64 R i-particles, R a
// lane in registers, against a piece of the j-range) from an LDS counter, so
// no barrier stands between units and a small frame's few items still keep
// every wave busy; j-particles arrive by buffer loads with a uniform offset,
// four ahead of the arithmetic. The wave that finds no unit left draws the
// workgroup's next item. Each pair's bin is counted with one ds_add_u32 into
// the workgroup's u32 LDS histogram (Sec. 2.4: groups of processing units
// share a private histogram; Sec. 3.2.3: partial histograms in on-chip
// memory). Lanes whose pair must not count (out of range, j <= i on a diagonal
// block, ragged i-block tail) are steered by a clamp to a per-lane discard
// slot past the bin window instead of a branch, so the atomic is issued
// without divergence and discarded pairs never collide on one address. When
// the histogram, window or frame changes, or before any u32 slot could wrap,
// the workgroup adds the counts to the uint64 output with global atomics
// (Sec. 3.1: u32 private histograms flushed into a u64 global one).
//
// Histograms too wide for LDS either run as bin windows (one LDS window per
// item, the shared-memory kernel's sweeps of Sec. 3.2.3) or, in the global
// mode, count every in-range pair with one uint64 atomic straight into the
// output (the global-memory kernel of Sec. 3.2.2); the host picks the mode.
#pragma once

#include "dh_internal.h"

#include <algorithm>
#include <type_traits>

namespace dh {
namespace {

template <typename T>
struct V4;
template <>
struct V4<float> { using type = float4; };
template <>
struct V4<double> { using type = double4; };

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// last word of a raw buffer resource (32-bit elements, no swizzle)
constexpr int kBufferFlags = 0x00020000;
using V4u = unsigned int __attribute__((ext_vector_type(4)));
using V2u = unsigned int __attribute__((ext_vector_type(2)));
// j-particles in flight ahead of the arithmetic, and the fewest j of a unit
constexpr int kJAhead = 4;
constexpr int kMinUnitJ = 8;
__device__ __forceinline__ float uni(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uni(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane(static_cast<int>(b & 0xffffffffll));
  const int hi = __builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              static_cast<unsigned int>(lo));
}
template <typename P>
__device__ __forceinline__ const P *uni(const P *p) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = static_cast<uint32_t>(uni(static_cast<int>(b & 0xffffffffu)));
  const uint32_t hi = static_cast<uint32_t>(uni(static_cast<int>(b >> 32)));
  return reinterpret_cast<const P *>((static_cast<uint64_t>(hi) << 32) | lo);
}

// --------------------------------------------------------------------------
// Distance arithmetic
// --------------------------------------------------------------------------

__device__ __forceinline__ float fmaT(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return fma(a, b, c); }

// binary64, canonical op sequence (Algorithm 1 with Eq. 5), no contraction.
struct Geo64 {
  double s, L0, L1, L2, iL0, iL1, iL2;
  double ax, bx, by, cx, cy, cz, h11, h12, h13, h22, h23, h33;
  const double (*shift)[3];
};

__device__ __forceinline__ Geo64 load_geo64(const FrameParams *F) {
  Geo64 g;
  g.s = uni(F->s);
  g.L0 = uni(F->L[0]); g.L1 = uni(F->L[1]); g.L2 = uni(F->L[2]);
  g.iL0 = uni(F->iL[0]); g.iL1 = uni(F->iL[1]); g.iL2 = uni(F->iL[2]);
  g.ax = uni(F->ax); g.bx = uni(F->bx); g.by = uni(F->by);
  g.cx = uni(F->cx); g.cy = uni(F->cy); g.cz = uni(F->cz);
  g.h11 = uni(F->h11); g.h12 = uni(F->h12); g.h13 = uni(F->h13);
  g.h22 = uni(F->h22); g.h23 = uni(F->h23); g.h33 = uni(F->h33);
  g.shift = F->shift64;
  return g;
}

// Fractional coordinates B^-1 x of a point (the rows of Eq. 5's reduction
// applied to a position instead of a difference).
__device__ __forceinline__ void frac64(double x, double y, double z, const Geo64 &g,
                                       double (&sg)[3]) {
  sg[0] = fma(z, g.h13, fma(y, g.h12, x * g.h11));
  sg[1] = fma(z, g.h23, y * g.h22);
  sg[2] = z * g.h33;
}

// Correctly rounded binary64 square root (IEEE-754 sqrt) for every
// argument. The candidate y comes from v_rsq_f64 refined by one Goldschmidt
// step and two Newton corrections with fused residuals, which leaves y within
// half an ulp plus a tiny fraction of sqrt(q): at most one ulp from the
// correctly rounded root. Tuckerman's rounding test then settles the last
// bit. With u = ulp(y) and the remainder r = q - y*y (one fma), sqrt(q) lies
// above the midpoint y + u/2 iff r > u*y, and below the midpoint under y iff
// r <= -u*y (-u*y/2 when y is a power of two, whose lower neighbour is only
// u/2 away): q and y*y are multiples of u*u, so r is too, and the midpoint
// conditions r < u*y + u*u/4 and r > -u*y + u*u/4 reduce to those
// thresholds. The thresholds and the next multiples of u*u beyond them are
// representable, so the comparisons are exact even where the fma rounds r.
// Arguments below 2^-767 are scaled by 2^1024 (exactly) so that the
// iteration and the remainder stay in the normal range, and the root is
// scaled back by 2^-512; 0, +inf and NaN are returned as IEEE sqrt returns
// them.
__device__ __forceinline__ double sqrt_cr(double q) {
  const bool tiny = q < 0x1p-767;
  const double qs = tiny ? ldexp(q, 1024) : q;
  const double y0 = __builtin_amdgcn_rsq(qs);
  double g = qs * y0;
  double h = 0.5 * y0;
  const double e = fma(-h, g, 0.5);
  h = fma(h, e, h);
  g = fma(g, e, g);
  double d = fma(-g, g, qs);
  g = fma(d, h, g);
  d = fma(-g, g, qs);
  double y = fma(d, h, g);
  const double r = fma(-y, y, qs);
  const uint64_t yb = static_cast<uint64_t>(__double_as_longlong(y));
  // y = f * 2^ex with f in [1/2, 1); y is normal here
  const int ex = static_cast<int>((yb >> 52) & 0x7ff) - 1022;
  const double uy = ldexp(y, ex - 53);  // ulp(y) * y, exact
  const bool pow2 = (yb & 0xFFFFFFFFFFFFFull) == 0;
  const double low = pow2 ? -0.5 * uy : -uy;
  const uint64_t step = r > uy ? 1ull : (r <= low ? ~0ull : 0ull);
  y = __longlong_as_double(static_cast<long long>(yb + step));
  if (tiny) y = ldexp(y, -512);
  if (qs > 0.0 && qs <= 0x1.fffffffffffffp+1023) return y;
  return q == 0.0 ? q : (q > 0.0 ? q : __builtin_nan(""));
}

// The bin bits (see kBinBits) of a binary64 pair from a binary32 root made
// exact by a binary64 residual. u is t^2 in units in which a bin is 2^-22
// wide, f = 2 + the binary32 root of u rounded to whole bins: m = f - 2 lies
// within 2/3 of a bin of the root for t < 2^20 (conversion and root are within
// 2^-22.5 relative), so floor(t) is m when u - m^2 >= 0 and one less
// otherwise. m^2 is exact and the residual one fma, so its sign is certain
// unless it is within the rounding of u and of the canonical t; the caller
// keeps the smallest |residual| of several pairs in `gap` (its upper word
// read as a float, monotone) and takes the canonical root for all of them when
// that is not above its threshold in some lane. Larger, infinite or NaN t
// give bits beyond every bin (2^20 - 2 bins at most). q = 0 has the residual
// 0. 12 instructions and one transcendental of 8 cycles, where a binary64
// root (v_rsq_f64 holds the SIMD for 16 cycles, then a Goldschmidt step) and
// its conversion took 13.
__device__ __forceinline__ uint32_t root_bits64(double u, float &gap);

// How a binary64 frame decides its bins: u = q scale, residuals up to `near`
// (in u) go to the canonical root. The scale's rounding, the product's and the
// canonical t's stay below 2^-49 of u together, and u <= (n_bins + 2)^2 2^-44
// where it matters. Frames with 2^20 - 2 bins or more, or whose scale is no
// normal number, take the canonical root for every pair (near = +inf).
// (60,000 points, 4,096 bins: without a box 1,165 us with the binary64 root,
// 948 us with this; in a cube 1,519 and 1,330 us, triclinic 1,842 and 1,649.)
struct Bins64 {
  double scale, s;
  float near;
};
__device__ __forceinline__ Bins64 bins64(const FrameParams *F) {
  Bins64 b;
  const int n_bins = uni(F->n_bins);
  b.s = uni(F->s);
  b.scale = (b.s * 0x1p-22) * (b.s * 0x1p-22);
  const double top = static_cast<double>(n_bins + 2) * 0x1p-22;
  const double thr = top * top * 0x1p-47;
  const bool fits = n_bins < (1 << 20) - 2 && b.s > 0x1p-400 && b.s < 0x1p400;
  b.near = uni(fits ? __int_as_float(static_cast<int>(__double_as_longlong(thr) >> 32) + 1)
                    : __builtin_inff());
  return b;
}
// u in the middle of a bin (2^19), for pairs that do not count: a particle
// against itself has the residual 0, which sent every j of a diagonal unit to
// the canonical root (1,000 points in a cube: 24.6 us, 15.5 with this; 10,000:
// 85 and 63 us; sorted, 100,000 points: 2,890 and 2,860 us).
// (Not in the unsorted image search, whose ballots are per pair: no change.)
constexpr double kFarU = 0x1.00002p-6;
// whether a lane of the wave has a residual too small to decide (a uniform
// answer; a NaN distance leaves gap alone: it counts nowhere)
__device__ __forceinline__ bool any_near(float gap, const Bins64 &b) {
  return __builtin_amdgcn_ballot_w64(!(gap > b.near)) != 0;
}
// the bits of a canonical t: floor(t), saturated beyond every bin (2^24 at
// most; a NaN t takes the other operand)
constexpr uint32_t kNoBits = (1u << 30) + (1u << 25);
__device__ __forceinline__ uint32_t canonical_bits(double q, double s);

// d = x_j - x_i reduced by the minimum-image rule of the box kind.
template <int BOX>
__device__ __forceinline__ void reduce64(double xi, double yi, double zi, double xj, double yj,
                                         double zj, const Geo64 &g, double &dx, double &dy,
                                         double &dz) {
  dx = xj - xi;
  dy = yj - yi;
  dz = zj - zi;
  if constexpr (BOX == kBoxOrtho || BOX == kBoxCube) {
    const double n0 = rint(dx * g.iL0), n1 = rint(dy * g.iL1), n2 = rint(dz * g.iL2);
    dx = fma(-g.L0, n0, dx);
    dy = fma(-g.L1, n1, dy);
    dz = fma(-g.L2, n2, dz);
  } else if constexpr (BOX == kBoxTric || BOX == kBoxTricSearch) {
    const double sc = dz * g.h33;
    const double sb = fma(dz, g.h23, dy * g.h22);
    const double sa = fma(dz, g.h13, fma(dy, g.h12, dx * g.h11));
    const double na = rint(sa), nb = rint(sb), nc = rint(sc);
    dz = fma(-g.cz, nc, dz);
    dy = fma(-g.cy, nc, fma(-g.by, nb, dy));
    dx = fma(-g.cx, nc, fma(-g.bx, nb, fma(-g.ax, na, dx)));
  }
}

// Minimum of q over the 27 images d + S (S = 0 gives q itself). Every q is
// a sum of squares (never -0), so fmin equals the select v < q ? v : q,
// NaN included (a NaN d makes every image NaN); the minimum of such values
// does not depend on the order, so three running minima give the chain
// more independent work.
__device__ __forceinline__ double search_q64(double dx, double dy, double dz, double q,
                                             const Geo64 &g) {
  double qa = q, qb = q, qc = q;
#pragma unroll
  for (int m = 0; m < kShifts; m += 3) {
    double v[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const double vx = dx + uni(g.shift[m + u][0]);
      const double vy = dy + uni(g.shift[m + u][1]);
      const double vz = dz + uni(g.shift[m + u][2]);
      v[u] = fma(vz, vz, fma(vy, vy, vx * vx));
    }
    qa = fmin(qa, v[0]);
    qb = fmin(qb, v[1]);
    qc = fmin(qc, v[2]);
  }
  return fmin(qa, fmin(qb, qc));
}

template <int BOX>
__device__ __forceinline__ double t64(double xi, double yi, double zi, double xj, double yj,
                                      double zj, const Geo64 &g) {
  double dx, dy, dz;
  reduce64<BOX>(xi, yi, zi, xj, yj, zj, g, dx, dy, dz);
  double q = fma(dz, dz, fma(dy, dy, dx * dx));
  if constexpr (BOX == kBoxTricSearch) q = search_q64(dx, dy, dz, q, g);
  return sqrt_cr(q) * g.s;
}

// q of the canonical sequence before the root (no image search)
template <int BOX>
__device__ __forceinline__ double q64(double xi, double yi, double zi, double xj, double yj,
                                      double zj, const Geo64 &g) {
  double dx, dy, dz;
  reduce64<BOX>(xi, yi, zi, xj, yj, zj, g, dx, dy, dz);
  return fma(dz, dz, fma(dy, dy, dx * dx));
}

// binary32. Without a box the staged coordinates are x * s, so the
// Euclidean length is already t. With a periodic cell they are 32-bit
// fixed-point fractional coordinates: the wrapped difference u_j - u_i read as
// a signed integer is 2^32 times the Eq. 5 reduced fractional difference, so
// the minimum image costs one integer subtraction per axis; converting it to
// float and applying the cell matrix scaled by s / 2^32 gives t units.
struct Geo32 {
  float kx, ky, kz;                 // orthorhombic: L_c * s / 2^32
  float ry, rz;                     // orthorhombic: (L_y / L_x)^2, (L_z / L_x)^2
  float ax, bx, by, cx, cy, cz;     // triclinic: cell matrix * s / 2^32
  float nbx, nby, ncx, ncy, ncz;    // triclinic: cell matrix / a_x
  const float (*shift)[3];          // image shifts * s
};

__device__ __forceinline__ Geo32 load_geo32(const FrameParams *F) {
  Geo32 g;
  g.kx = uni(F->k32[0]); g.ky = uni(F->k32[1]); g.kz = uni(F->k32[2]);
  g.ry = uni(F->ryz32[0]); g.rz = uni(F->ryz32[1]);
  g.ax = uni(F->Bk[0]); g.bx = uni(F->Bk[1]); g.by = uni(F->Bk[2]);
  g.cx = uni(F->Bk[3]); g.cy = uni(F->Bk[4]); g.cz = uni(F->Bk[5]);
  g.nbx = uni(F->Bn[0]); g.nby = uni(F->Bn[1]); g.ncx = uni(F->Bn[2]);
  g.ncy = uni(F->Bn[3]); g.ncz = uni(F->Bn[4]);
  g.shift = F->shift32;
  return g;
}

// reduced fractional difference, units of 2^-32 of the cell vector
__device__ __forceinline__ float frac_diff(float ui, float uj) {
  return static_cast<float>(static_cast<int32_t>(__float_as_uint(uj) - __float_as_uint(ui)));
}

template <int BOX>
__device__ __forceinline__ float t32_packed(uint64_t ab_j, uint64_t neg_ab_i, float zi, float zj,
                                            const Geo32 &g);
template <int BOX>
__device__ __forceinline__ float t32_packed_c(uint64_t ab_j, uint64_t neg_ab_i, float fc,
                                              const Geo32 &g);

// Binary32 bins without a float-to-integer conversion: t 2^-22 + (2 - 2^-23)
// rounded to nearest lies in [2, 4) for 1/2 <= t < 2^22, where the spacing is
// 2^-22, so its bits minus those of 2 are floor(t), except at an integer t:
// that is a tie, which goes to the even neighbour, so an odd integer t counts
// one bin lower (a pair at a bin edge, inside the binary32 tolerance). For
// t < 1/4 the difference is -1 (bin 0; the counting code maps it there); it
// grows monotonically with t and is at least 2^22 for t >= 2^22, +inf and NaN
// (read as unsigned). Binary32 histograms have at most 2^22 bins, so a pair
// counts iff the difference is below n_bins. The bits of 2 leave a 32-bit word
// when the bin is shifted to a byte offset, so the LDS address of a slot is
// one shift and the instruction's own offset.
constexpr float kBinScale = 0x1p-22f;
constexpr float kBinOffset = 0x1.fffffep+0f;  // 2 - 2^-23
// the offset of a lane that must not count: its bits are beyond every bin,
// and the clamp sends them to the lane's discard slot
constexpr float kNoBin = 3.5f;
constexpr uint32_t kBinBits = 0x40000000u;  // bits of 2
// LDS: the workgroup's control words, a guard whose last word is binary32 bin
// -1, then slot 0. The kernels have no other LDS variable, so the dynamic
// array starts at address 0 and slot 0 has a constant address, which the LDS
// instructions take as their immediate offset.
constexpr int kGuardBytes = 16;
constexpr uint32_t kSlot0 = kControlBytes + kGuardBytes;

__device__ __forceinline__ uint32_t bin_bits32(float t, float offset = kBinOffset) {
  return __float_as_uint(fmaf(t, kBinScale, offset));
}

// min(a, b) for an a that is an arithmetic result (never a signalling NaN):
// one v_min_f64, without the canonicalisation fmin adds for arbitrary input.
// A NaN a gives b, as fmin does.
__device__ __forceinline__ double min_arith(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

__device__ __forceinline__ uint32_t root_bits64(double u, float &gap) {
  const float f = __builtin_amdgcn_sqrtf(static_cast<float>(u)) + 2.f;
  const double m = static_cast<double>(f - 2.f);
  const double r = fma(-m, m, u);
  const int rh = static_cast<int>(__double_as_longlong(r) >> 32);
  gap = fminf(gap, fabsf(__int_as_float(rh)));
  return __float_as_uint(f) + static_cast<uint32_t>(rh >> 31);
}
__device__ __forceinline__ uint32_t canonical_bits(double q, double s) {
  return kBinBits + static_cast<uint32_t>(min_arith(sqrt_cr(q) * s, 0x1p25));
}



// Triclinic reduced vector (t units) from packed fractional words.
__device__ __forceinline__ void tric_vec32(uint64_t ab_j, uint64_t neg_ab_i, float zi, float zj,
                                           const Geo32 &g, float &dx, float &dy, float &dz) {
  const uint64_t dab = ab_j + neg_ab_i;
  const float fa = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab)));
  const float fb = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab >> 32)));
  const float fc = frac_diff(zi, zj);
  dx = fmaf(g.cx, fc, fmaf(g.bx, fb, g.ax * fa));
  dy = fmaf(g.cy, fc, g.by * fb);
  dz = g.cz * fc;
}

// Minimum of q over the 27 images (binary32, t units), three running minima.
__device__ __forceinline__ float search_q32(float dx, float dy, float dz, float q,
                                            const Geo32 &g) {
  float qa = q, qb = q, qc = q;
#pragma unroll
  for (int m = 0; m < kShifts; m += 3) {
    float v[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const float vx = dx + uni(g.shift[m + u][0]);
      const float vy = dy + uni(g.shift[m + u][1]);
      const float vz = dz + uni(g.shift[m + u][2]);
      v[u] = fmaf(vz, vz, fmaf(vy, vy, vx * vx));
    }
    qa = fminf(qa, v[0]);
    qb = fminf(qb, v[1]);
    qc = fminf(qc, v[2]);
  }
  return fminf(qa, fminf(qb, qc));
}

template <int BOX>
__device__ __forceinline__ float t32(float xi, float yi, float zi, float xj, float yj, float zj,
                                     const Geo32 &g) {
  if constexpr (BOX == kBoxNone) {
    const float dx = xj - xi, dy = yj - yi, dz = zj - zi;
    return __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));  // v_sqrt_f32
  } else {
    const uint64_t ai = (static_cast<uint64_t>(__float_as_uint(yi)) << 32) | __float_as_uint(xi);
    const uint64_t aj = (static_cast<uint64_t>(__float_as_uint(yj)) << 32) | __float_as_uint(xj);
    return t32_packed<BOX>(aj, 0ull - ai, zi, zj, g);
  }
}

// Periodic binary32 distance from packed fractional words: ab = (b << 32) | a
// of particle j and -(b << 32 | a) of particle i. One 64-bit addition gives
// both differences: the low word exactly, the high word lowered by one unit
// (2^-32 of a cell vector, far below binary32 rounding) when a borrows.
template <int BOX>
__device__ __forceinline__ float t32_packed(uint64_t ab_j, uint64_t neg_ab_i, float zi, float zj,
                                            const Geo32 &g) {
  return t32_packed_c<BOX>(ab_j, neg_ab_i, frac_diff(zi, zj), g);
}

// The same with the c difference given (as a float of fixed-point units).
template <int BOX>
__device__ __forceinline__ float t32_packed_c(uint64_t ab_j, uint64_t neg_ab_i, float fc,
                                              const Geo32 &g) {
  {
    const uint64_t dab = ab_j + neg_ab_i;
    const float fa = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab)));
    const float fb = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab >> 32)));
    if constexpr (BOX == kBoxCube) {
      return __builtin_amdgcn_sqrtf(fmaf(fc, fc, fmaf(fb, fb, fa * fa))) * g.kx;
    } else if constexpr (BOX == kBoxOrtho) {
      // q / kx^2, the y and z squares weighted by (L_y/L_x)^2 and (L_z/L_x)^2
      const float q = fmaf(fc * g.rz, fc, fmaf(fb * g.ry, fb, fa * fa));
      return __builtin_amdgcn_sqrtf(q) * g.kx;
    } else if constexpr (BOX == kBoxTric) {
      // d / (a_x s 2^-32): the cell matrix divided by a_x
      const float dx = fmaf(g.ncx, fc, fmaf(g.nbx, fb, fa));
      const float dy = fmaf(g.ncy, fc, g.nby * fb);
      const float dz = g.ncz * fc;
      return __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx))) * g.ax;
    } else {
      const float dx = fmaf(g.cx, fc, fmaf(g.bx, fb, g.ax * fa));
      const float dy = fmaf(g.cy, fc, g.by * fb);
      const float dz = g.cz * fc;
      float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
      if constexpr (BOX == kBoxTricSearch) q = search_q32(dx, dy, dz, q, g);
      return __builtin_amdgcn_sqrtf(q);
    }
  }
}

// Bin bits (see bin_bits32) of the same distance; without the image search
// the scale (L_x or a_x times s / 2^32) and the offset are one fused
// multiply-add on the root.
template <int BOX>
__device__ __forceinline__ uint32_t bits32_packed_c(uint64_t ab_j, uint64_t neg_ab_i, float fc,
                                                    const Geo32 &g, float offset) {
  if constexpr (BOX == kBoxCube || BOX == kBoxOrtho || BOX == kBoxTric) {
    const uint64_t dab = ab_j + neg_ab_i;
    const float fa = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab)));
    const float fb = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(dab >> 32)));
    float q, k;
    if constexpr (BOX == kBoxCube) {
      q = fmaf(fc, fc, fmaf(fb, fb, fa * fa));
      k = g.kx * kBinScale;
    } else if constexpr (BOX == kBoxOrtho) {
      q = fmaf(fc * g.rz, fc, fmaf(fb * g.ry, fb, fa * fa));
      k = g.kx * kBinScale;
    } else {
      const float dx = fmaf(g.ncx, fc, fmaf(g.nbx, fb, fa));
      const float dy = fmaf(g.ncy, fc, g.nby * fb);
      const float dz = g.ncz * fc;
      q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
      k = g.ax * kBinScale;
    }
    return __float_as_uint(fmaf(__builtin_amdgcn_sqrtf(q), k, offset));
  } else {
    return bin_bits32(t32_packed_c<BOX>(ab_j, neg_ab_i, fc, g), offset);
  }
}

// Counts pairs from their bin bits (see bin_bits32, root_bits64). The clamp is an
// upper one only: bin -1 is the guard word below the histogram, added to bin 0
// on flush, and a lane whose pair must not count passes bits beyond every bin
// (kNoBin). Two-operand instructions throughout: v_min_u32, v_lshlrev_b32 and
// v_sub_u32 take about 2.7 cycles of a SIMD, the three-operand v_med3_u32 and
// v_lshl_add_u32 about 4.5.
template <int MODE>
struct Count {
  using LdsU32 = __attribute__((address_space(3))) uint32_t;
  using GlobalU64 = __attribute__((address_space(1))) unsigned long long;
  uint32_t top;     // the lane's discard slot (LDS: in bin bits; windows: as a slot)
  uint32_t base;    // bin bits of slot 0 of a window: the bin below its first
  uint32_t n_bins;
  GlobalU64 *out;

  __device__ __forceinline__ Count(const FrameParams *F, const WorkItem &w, int lane) {
    const uint32_t win = static_cast<uint32_t>(uni(F->win));
    const uint32_t b_lo = static_cast<uint32_t>(w.sweep) * win;
    n_bins = static_cast<uint32_t>(uni(F->n_bins));
    top = win + static_cast<uint32_t>(lane) + (MODE == kModeSweep ? 1u : kBinBits);
    base = kBinBits + b_lo - 1u;
    // global memory, said so that the atomics are global_atomic_* (a generic
    // pointer would give flat atomics, which also count as LDS operations)
    out = (GlobalU64 *)(F->out + static_cast<size_t>(w.hist) * n_bins);
  }
  // CLAMP = false: every t is known to lie below the LDS stride.
  template <bool CLAMP>
  __device__ __forceinline__ void add(uint32_t b) const {
    if constexpr (MODE == kModeGlobal) {
      const uint32_t k = max(b, kBinBits) - kBinBits;
      if (k < n_bins)
        __hip_atomic_fetch_add(out + k, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    // windows: slot 0 is the guard word (bin -1 of window 0; what other
    // windows leave there is dropped on flush); bins below wrap to large
    // values and are discarded with those above
    const uint32_t m = MODE == kModeSweep ? min(b - base, top) : CLAMP ? min(b, top) : b;
    const uint32_t at = (m << 2) + (MODE == kModeSweep ? kSlot0 - 4u : kSlot0);
    __hip_atomic_fetch_add((LdsU32 *)(uintptr_t)at, 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// min(a, b) of two arithmetic results (never signalling NaNs), without the
// canonicalisation fmin adds; a NaN operand gives the other, as fmin does.
__device__ __forceinline__ float min_arith(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Minimum of q over the images in the search table from `base` (an octant
// row, or the 27 shift vectors), n of them (uniform), three running minima.
// Rows are padded with the zero shift, and a run past a row's end reads
// further table entries, which are images too, so the minimum is unchanged;
// images
// left out of an octant row cannot be nearer (see octant_images on the
// host), so it equals the one over all 27 images.
template <typename T>
__device__ __forceinline__ T search_oct(T dx, T dy, T dz, T q, int base, int n,
                                        const typename V4<T>::type *__restrict__ tab) {
  T qa = q, qb = q, qc = q;
  const typename V4<T>::type *row = tab + base;
  auto image = [&](int k) {
    const typename V4<T>::type S = row[k];
    const T vx = dx + S.x;
    const T vy = dy + S.y;
    const T vz = dz + S.z;
    return fmaT(vz, vz, fmaT(vy, vy, vx * vx));
  };
  int k = 0;
  for (; k + 2 < n; k += 3) {
    const T v0 = image(k), v1 = image(k + 1), v2 = image(k + 2);
    qa = min_arith(qa, v0);
    qb = min_arith(qb, v1);
    qc = min_arith(qc, v2);
  }
  for (; k < n; ++k) qa = min_arith(qa, image(k));
  return min_arith(qa, min_arith(qb, qc));
}

// Image shifts of the seven neighbours towards a reduced vector whose
// third fractional component is not negative (c always shifted by -1), for
// either sign of the first two (the table's values).
template <typename T>
struct Seven {
  T xa;                // ( 1, 0, 0)
  T xb, yb;            // ( 0, 1, 0)
  T xs, xd;            // ( 1, 1, 0), (-1, 1, 0)
  T xc, yc, zc;        // ( 0, 0,-1)
  T xca[2];            // (-1, 0,-1), ( 1, 0,-1)
  T xcb[2], ycb[2];    // ( 0,-1,-1), ( 0, 1,-1)
  T xcab[2][2];        // [b][a]
};
template <typename T>
__device__ __forceinline__ Seven<T> load_seven(const FrameParams *F) {
  auto at = [&](int i, int j, int k, int c) {
    const int m = 9 * (i + 1) + 3 * (j + 1) + (k + 1);
    if constexpr (sizeof(T) == 4)
      return uni(F->shift32[m][c]);
    else
      return uni(F->shift64[m][c]);
  };
  Seven<T> s;
  s.xa = at(1, 0, 0, 0);
  s.xb = at(0, 1, 0, 0); s.yb = at(0, 1, 0, 1);
  s.xs = at(1, 1, 0, 0); s.xd = at(-1, 1, 0, 0);
  s.xc = at(0, 0, -1, 0); s.yc = at(0, 0, -1, 1); s.zc = at(0, 0, -1, 2);
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    s.xca[p] = at(2 * p - 1, 0, -1, 0);
    s.xcb[p] = at(0, 2 * p - 1, -1, 0);
    s.ycb[p] = at(0, 2 * p - 1, -1, 1);
#pragma unroll
    for (int v = 0; v < 2; ++v) s.xcab[p][v] = at(2 * v - 1, 2 * p - 1, -1, 0);
  }
  return s;
}

// The minimum of search_oct where every octant's list is its seven images
// towards the vector, without the table: the vector is turned into the half
// space c >= 0 (an image and its opposite differ in sign alone, and so do the
// table's entries), which leaves two signs to choose the shifts by; images
// share their y and z. Every image's q is the one of the table's entry.
// The table's rows, read per lane, were what bounded the search: seven 16-byte
// LDS reads are 56 cycles of a CU per 64 vectors whatever rows the lanes take.
// 200,000 points in a sheared triclinic cell, 48 % of the pairs searched:
// 54.5 ms with the table, 30.5 ms with this, 27.9 ms with ring positions that
// wrap by a mask and the octant from three shifts besides; now bound by
// vector issue. Binary64, 60,000 and 20,000 points: 7.40 and 5.78 ms, 975 and
// 842 us.
__device__ __forceinline__ float flip_sign(float v, uint32_t sign) {
  return __uint_as_float(__float_as_uint(v) ^ sign);
}
__device__ __forceinline__ double flip_sign(double v, uint32_t sign) {
  return __longlong_as_double(__double_as_longlong(v) ^
                              static_cast<long long>(static_cast<uint64_t>(sign) << 32));
}
template <typename T>
__device__ __forceinline__ T search_seven(T dx, T dy, T dz, T q, int code, const Seven<T> &s) {
  const uint32_t turn = (static_cast<uint32_t>(code) << 29) & 0x80000000u;
  dx = flip_sign(dx, turn); dy = flip_sign(dy, turn); dz = flip_sign(dz, turn);
  // the signs of the first two components after the turn: a set bit means
  // negative, where the image nearer to the vector is the positive one
  const uint32_t ta = static_cast<uint32_t>(code) ^ (static_cast<uint32_t>(code) >> 2);
  const uint32_t tb = (static_cast<uint32_t>(code) >> 1) ^ (static_cast<uint32_t>(code) >> 2);
  const bool a = (ta & 1u) != 0, b = (tb & 1u) != 0, same = ((ta ^ tb) & 1u) == 0;
  const uint32_t sa = (~ta) << 31, sb = (~tb) << 31;
  const T yb = dy + flip_sign(s.yb, sb), yc = dy + s.yc, zc = dz + s.zc;
  const T ycb = dy + (b ? s.ycb[1] : s.ycb[0]);
  auto len = [](T x, T y, T z) { return fmaT(z, z, fmaT(y, y, x * x)); };
  const T q1 = len(dx + flip_sign(s.xa, sa), dy, dz);
  const T q2 = len(dx + flip_sign(s.xb, sb), yb, dz);
  const T q3 = len(dx + flip_sign(same ? s.xs : s.xd, sb), yb, dz);
  const T q4 = len(dx + s.xc, yc, zc);
  const T q5 = len(dx + (a ? s.xca[1] : s.xca[0]), yc, zc);
  const T q6 = len(dx + (b ? s.xcb[1] : s.xcb[0]), ycb, zc);
  const T u = a ? s.xcab[0][1] : s.xcab[0][0], v = a ? s.xcab[1][1] : s.xcab[1][0];
  const T q7 = len(dx + (b ? v : u), ycb, zc);
  q = min_arith(min_arith(q, q1), min_arith(q2, q3));
  return min_arith(q, min_arith(min_arith(q4, q5), min_arith(q6, q7)));
}

// A wave's share of its item's searched pairs and images evaluated, into the
// workgroup's sums: one thread adds those to the frame's two counts, where every
// addition takes its turn (about 10 ns each; 1,000 points of 32 species, 528
// items of four waves: 74 us with an addition per wave, 36 us with one per item).
__device__ __forceinline__ void add_searched(unsigned long long *s_search, int lane,
                                             uint64_t pairs, uint64_t images) {
  if (lane == 0 && (pairs | images) != 0) {
    atomicAdd(s_search, static_cast<unsigned long long>(pairs));
    atomicAdd(s_search + 1, static_cast<unsigned long long>(images));
  }
}

// Octant of a reduced binary64 vector: bit k when fractional component k is
// negative; 8 (the full list) when a component lies outside the octant boxes
// of the host (|f| beyond 1/2 plus half their slack, or NaN).
__device__ __forceinline__ int octant64(double dx, double dy, double dz, const Geo64 &g) {
  double f[3];
  frac64(dx, dy, dz, g, f);
  int code = 0;
  bool inside = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    code |= f[k] < 0.0 ? 1 << k : 0;
    inside = inside && fabs(f[k]) <= 0.5 + 0.5 * kOctSlack;
  }
  return inside ? code : 8;
}

// Octant of a reduced binary32 vector from its wrapped fixed-point
// differences (exact, within [-1/2, 1/2) of a cell vector).
__device__ __forceinline__ int octant32(uint64_t ab_j, uint64_t neg_ab_i, float zi, float zj) {
  const uint64_t dab = ab_j + neg_ab_i;
  // (each step shifts the next sign in from the right)
  uint32_t code = (__float_as_uint(zj) - __float_as_uint(zi)) >> 31;
  code = __builtin_amdgcn_alignbit(code, static_cast<uint32_t>(dab >> 32), 31);
  code = __builtin_amdgcn_alignbit(code, static_cast<uint32_t>(dab), 31);
  return static_cast<int>(code);
}

template <typename T>
struct Geo;
template <>
struct Geo<float> {
  using type = Geo32;
  static __device__ __forceinline__ Geo32 load(const FrameParams *F) { return load_geo32(F); }
};
template <>
struct Geo<double> {
  using type = Geo64;
  static __device__ __forceinline__ Geo64 load(const FrameParams *F) { return load_geo64(F); }
};

template <typename T, int BOX>
__device__ __forceinline__ T pair_t(T xi, T yi, T zi, T xj, T yj, T zj,
                                    const typename Geo<T>::type &g) {
  if constexpr (sizeof(T) == 4)
    return t32<BOX>(xi, yi, zi, xj, yj, zj, g);
  else
    return t64<BOX>(xi, yi, zi, xj, yj, zj, g);
}

// --------------------------------------------------------------------------
// Pair kernel
// --------------------------------------------------------------------------

// Adds the LDS counts of bins [0, count) into out[] and clears every slot;
// ends with a barrier. The out-of-range count of the histogram is its pair
// count less every flushed count: the waves sum theirs in LDS (s_sum, zero
// between calls) and one thread subtracts the total, since every subtraction
// goes to the same address and takes its turn there (about 10 ns each: with
// one per wave, 256 workgroups of 16 waves ran a 5,000-point frame in 92 us).
__device__ __forceinline__ void flush_hist(uint32_t *hist, const PairKernelArgs &a,
                                           const FrameParams *F, int hist_idx, int sweep,
                                           unsigned long long *s_sum) {
  const int n_bins = uni(F->n_bins);
  const int win = uni(F->win);
  const int b_lo = sweep * win;
  const int count = min(win, n_bins - b_lo);
  uint64_t *out = F->out + static_cast<size_t>(hist_idx) * n_bins + b_lo;
  // the whole stride: slots past the window may hold counts of out-of-range
  // pairs of unclamped units, and the next frame may use a wider window
  const int clear = a.stride;
  uint64_t in_range = 0;
  for (int b = threadIdx.x; b < clear; b += blockDim.x) {
    uint64_t v = hist[b];
    hist[b] = 0u;
    if (b == 0) {
      // the guard word: binary32 bin -1 (see Count)
      if (sweep == 0) v += hist[-1];
      hist[-1] = 0u;
    }
    if (b < count && v != 0) {
      atomicAdd(reinterpret_cast<unsigned long long *>(out + b),
                static_cast<unsigned long long>(v));
      in_range += v;
    }
  }
  const bool oor = uni(F->oor_by_flush) != 0;
  if (oor) {
    for (int o = 32; o > 0; o >>= 1) in_range += __shfl_xor(in_range, o);
    if ((threadIdx.x & 63) == 0 && in_range != 0)
      atomicAdd(s_sum, static_cast<unsigned long long>(in_range));
  }
  __syncthreads();
  if (oor && threadIdx.x == 0 && *s_sum != 0) {
    atomicAdd(reinterpret_cast<unsigned long long *>(F->oor + hist_idx), 0ull - *s_sum);
    *s_sum = 0;
  }
}

}  // namespace
}  // namespace dh

#include "dh_sorted.h"

namespace dh {
namespace {

// One work item of an unsorted frame: the workgroup's waves draw its units
// from a counter in LDS, a unit being one slice of 64 R i-particles (held in
// registers, lane l the particles wbase + 64 r + l) against one piece of the
// item's j-range. Every wave streams its j straight from the staged frame:
// all lanes load one address, the cache hands the point to the whole wave,
// and four j are in flight ahead of the arithmetic, so no tile is staged, no
// barrier stands inside an item and LDS holds nothing but the histogram. An
// item can be any number of slices by any j-range and still keep every wave
// busy, and only the units that touch the diagonal of an intra-species
// histogram pay for the mask. Bound by vector-unit issue in large frames
// (100,000 points in a cube, binary32, 10,000 bins: 1,410 us with the j-tiles
// in LDS and a barrier per tile, 1,285 us now), by latency in small ones,
// whose block on the diagonal used to run as one serial item (5,000 points,
// binary64: 634 us, now 23 us; 1,000 points, binary32: 113 and 16 us).
//
// Units whose lanes all hold a particle run without the clamp where the host
// proved that every t of the frame is below the LDS stride (out-of-range
// pairs land in slots [n_bins, stride) that are never flushed).
//
// BOX = kBoxTricSearch: the 27-image search only runs for pairs whose reduced
// vector is not provably the nearest image (q0 >= qskip: at least half the
// shortest lattice vector long). Those pairs are queued per wave in LDS and
// searched 64 at a time by the whole wave, so the search never runs for a
// wave with only a few lanes needing it; the others are counted directly.
template <typename T, int R, int BOX, int MODE>
__device__ __forceinline__ void run_units(const PairKernelArgs &a, const WorkItem &w,
                                          const FrameParams *F, uint32_t *__restrict__ my,
                                          typename V4<T>::type *__restrict__ queue,
                                          typename V4<T>::type *__restrict__ sh, int *s_unit,
                                          int *s_item, unsigned long long *s_search) {
  using V = typename V4<T>::type;
  using G = typename Geo<T>::type;
  constexpr bool SEARCH = BOX == kBoxTricSearch;
  const V *__restrict__ X = uni(static_cast<const V *>(F->coords));
  const G g = Geo<T>::load(F);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const Count<MODE> count(F, w, lane);
  // binary32 frames whose every t is below the LDS stride need no clamp;
  // binary64 reads raw device coordinates and keeps it for non-finite ones
  const bool noclamp = MODE == kModeLds && !SEARCH && sizeof(T) == 4 && uni(F->noclamp) != 0;
  [[maybe_unused]] const Bins64 bins = sizeof(T) == 8 ? bins64(F) : Bins64{};

  // bin bits of one binary64 pair (its own ballot)
  [[maybe_unused]] auto bits_of = [&](double q) {
    float gap = __builtin_inff();
    const uint32_t b = root_bits64(q * bins.scale, gap);
    return __builtin_expect(any_near(gap, bins), 0) ? canonical_bits(q, bins.s) : b;
  };

  // image-search ring of this wave: qn entries from head (wave-uniform)
  constexpr int cap = queue_cap(R);
  static_assert((cap & (cap - 1)) == 0, "ring positions wrap by a mask");
  V *const wq = queue + wave * cap;
  int head = 0, qn = 0;
  [[maybe_unused]] uint64_t n_searched = 0;  // pairs this wave searched in this item
  [[maybe_unused]] uint64_t n_images = 0;    // images it evaluated for them
  [[maybe_unused]] T qskip;
  if constexpr (sizeof(T) == 4)
    qskip = uni(F->qskip32);
  else
    qskip = uni(F->qskip64);
  [[maybe_unused]] uint32_t oct_full = 0;
  [[maybe_unused]] int oct_n = 0;
  [[maybe_unused]] bool oct_seven = false;
  [[maybe_unused]] Seven<T> seven;
  if constexpr (SEARCH) {
    oct_seven = uni(static_cast<int>(F->oct_seven)) != 0;
    seven = load_seven<T>(F);
  }
  if constexpr (SEARCH) {
    oct_full = static_cast<uint32_t>(uni(static_cast<int>(F->oct_full)));
    oct_n = uni(static_cast<int>(F->oct_n));
    // this frame's search table: the 8 octant rows, then all 27 shift vectors
    for (int k = tid; k < kSearchTable; k += blockDim.x) {
      const int m = k < 8 * kOctCap ? F->oct_shift[k / kOctCap][k % kOctCap] : k - 8 * kOctCap;
      V S;
      if constexpr (sizeof(T) == 4) {
        S.x = F->shift32[m][0]; S.y = F->shift32[m][1]; S.z = F->shift32[m][2];
      } else {
        S.x = F->shift64[m][0]; S.y = F->shift64[m][1]; S.z = F->shift64[m][2];
      }
      S.w = T(0);
      sh[k] = S;
    }
    __syncthreads();
  }
  using Yes = std::true_type;
  using No = std::false_type;
  // searches and counts the `cnt` (<= 64) oldest queued vectors
  auto drain = [&](int cnt) {
    if constexpr (SEARCH) {
      __builtin_amdgcn_wave_barrier();
      const bool v = lane < cnt;
      const V e = wq[(head + (v ? lane : 0)) & (cap - 1)];
      T q = fmaT(e.z, e.z, fmaT(e.y, e.y, e.x * e.x));
      // the vector's octant (8: outside the octant boxes), 8 as well when its
      // list is the full one; the wave runs the full list when any of its
      // vectors needs it
      int code;
      if constexpr (sizeof(T) == 4)
        code = __float_as_int(e.w);
      else
        code = octant64(e.x, e.y, e.z, g);
      if (oct_seven && (sizeof(T) == 4 || __builtin_amdgcn_ballot_w64(code == 8) == 0)) {
        q = search_seven<T>(e.x, e.y, e.z, q, code, seven);
        n_images += static_cast<uint64_t>(cnt) * 7u;
      } else {
        if ((oct_full >> code) & 1u) code = 8;
        const int n = __builtin_amdgcn_ballot_w64(code == 8) != 0 ? kShifts : oct_n;
        q = search_oct<T>(e.x, e.y, e.z, q, code == 8 ? 8 * kOctCap : code * kOctCap, n, sh);
        n_images += static_cast<uint64_t>(cnt) * static_cast<uint64_t>(n);
      }
      if constexpr (sizeof(T) == 4)
        count.template add<true>(
            bin_bits32(__builtin_amdgcn_sqrtf(q), v ? kBinOffset : kNoBin));
      else
      {
        const uint32_t b = bits_of(q);
        count.template add<true>(v ? b : kNoBits);
      }
      n_searched += cnt;  // wave-uniform; added to the frame's count once per item
      head = (head + cnt) & (cap - 1);
      qn -= cnt;
      __builtin_amdgcn_wave_barrier();
    }
  };

  // the i-particles of the current slice
  int wbase = -1;
  T xi[R], yi[R], zi[R];
  // a lane past the end of the item: its bin offset is beyond every bin
  // (binary32); in binary64 its particle is at infinity, where every distance
  // is infinite or NaN
  [[maybe_unused]] float off[R];
  // -(b:a) of each i-particle for the packed periodic binary32 difference;
  // -(c' : c) of i-particles 2k and 2k+1: one 64-bit addition to j's (c : c)
  // gives both c differences, the second lowered by one unit when the first
  // borrows (as for b)
  static_assert(R % 2 == 0, "i-particles are paired for the c difference");
  uint64_t nab[R], nzz[R / 2];
  auto load_i = [&]() {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = wbase + r * 64 + lane;
      const bool ok = i < w.i1;
      const V p = X[ok ? i : w.i0];
      xi[r] = sizeof(T) == 8 && !ok ? static_cast<T>(__builtin_inf()) : p.x;
      yi[r] = p.y; zi[r] = p.z;
      off[r] = ok ? kBinOffset : kNoBin;
      if constexpr (sizeof(T) == 4)
        nab[r] = 0ull - ((static_cast<uint64_t>(__float_as_uint(yi[r])) << 32) |
                         __float_as_uint(xi[r]));
      else
        nab[r] = 0ull;
    }
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      if constexpr (sizeof(T) == 4)
        nzz[k] = 0ull - ((static_cast<uint64_t>(__float_as_uint(zi[2 * k + 1])) << 32) |
                         __float_as_uint(zi[2 * k]));
      else
        nzz[k] = 0ull;
    }
  };

  // periodic binary32: j as its packed (b:a) and (c:c) words (see t32_packed
  // and the staging)
  constexpr bool kPacked = sizeof(T) == 4 && BOX != kBoxNone;
  struct JPacked {
    uint64_t ab;
    uint64_t cc;
  };
  using J = typename std::conditional<kPacked, JPacked, V>::type;

  // R pairs of one j: distance, bin, one atomic each
  auto pairs_of = [&](auto diag_c, auto clamp_c, const J &pj, int j) {
    constexpr bool DIAG = decltype(diag_c)::value;
    if constexpr (sizeof(T) == 8 && !SEARCH) {
      // binary64: one ballot for all R pairs (see root_bits64)
      double q[R];
      uint32_t b[R];
      float gap = __builtin_inff();
#pragma unroll
      for (int r = 0; r < R; ++r) {
        q[r] = q64<BOX>(xi[r], yi[r], zi[r], pj.x, pj.y, pj.z, g);
        double u = q[r] * bins.scale;
        if constexpr (DIAG) u = j <= wbase + r * 64 + lane ? kFarU : u;
        b[r] = root_bits64(u, gap);
      }
      if (__builtin_expect(any_near(gap, bins), 0))
#pragma unroll
        for (int r = 0; r < R; ++r) b[r] = canonical_bits(q[r], bins.s);
#pragma unroll
      for (int r = 0; r < R; ++r)
        count.template add<true>(DIAG && j <= wbase + r * 64 + lane ? kNoBits : b[r]);
      return;
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        [[maybe_unused]] float o = off[r];
        if constexpr (DIAG) o = j > wbase + r * 64 + lane ? o : kNoBin;
        if constexpr (SEARCH) {
          T dx, dy, dz;
          if constexpr (kPacked)
            tric_vec32(pj.ab, nab[r], zi[r], __uint_as_float(static_cast<uint32_t>(pj.cc)), g,
                       dx, dy, dz);
          else
            reduce64<BOX>(xi[r], yi[r], zi[r], pj.x, pj.y, pj.z, g, dx, dy, dz);
          const T q0 = fmaT(dz, dz, fmaT(dy, dy, dx * dx));
          // valid pairs at least half the shortest lattice vector long
          // are searched later; they must not count now
          const bool need = o == kBinOffset && q0 >= qskip;
          if constexpr (sizeof(T) == 4) {
            count.template add<true>(
                bin_bits32(__builtin_amdgcn_sqrtf(q0), need ? kNoBin : o));
          } else {
            const uint32_t b = bits_of(q0);
            count.template add<true>(need || o != kBinOffset ? kNoBits : b);
          }
          const uint64_t m = __builtin_amdgcn_ballot_w64(need);
          if (m != 0) {
            const int end = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                static_cast<uint32_t>(m >> 32),
                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m),
                                          static_cast<uint32_t>(head + qn))));
            if (need) {
              const int pos = end & (cap - 1);
              // binary32: the octant from the exact signs of the
              // fixed-point differences, as the bits of w; binary64 takes
              // it in the drain from the vector itself
              V e;
              e.x = dx; e.y = dy; e.z = dz;
              if constexpr (kPacked)
                e.w = __int_as_float(octant32(pj.ab, nab[r], zi[r],
                                              __uint_as_float(static_cast<uint32_t>(pj.cc))));
              else
                e.w = T(0);
              wq[pos] = e;
            }
            qn += __builtin_popcountll(m);
            if (qn >= 64) drain(64);
          }
        } else if constexpr (kPacked) {
          // c differences of i-particles r and r+1 from one 64-bit add
          const uint64_t dcc = pj.cc + nzz[r / 2];
          const float fc = static_cast<float>(static_cast<int32_t>(
              static_cast<uint32_t>(r % 2 == 0 ? dcc : dcc >> 32)));
          count.template add<decltype(clamp_c)::value>(
              bits32_packed_c<BOX>(pj.ab, nab[r], fc, g, o));
        } else {
          count.template add<decltype(clamp_c)::value>(
              bin_bits32(pair_t<T, BOX>(xi[r], yi[r], zi[r], pj.x, pj.y, pj.z, g), o));
        }
      }
    }
  };
  // The slice against j in [jb, je), kJAhead of them in flight: the load of
  // j + kJAhead follows the pairs of j. Buffer loads with a uniform
  // offset: they count in vmcnt (scalar loads would share lgkmcnt with the LDS
  // atomics and, returning out of order, wait for all of them), need no
  // address arithmetic in the vector unit, and a read ahead past the end of
  // the unit is out of the buffer's range and returns zeros, never used.
  auto stream = [&](auto diag_c, auto clamp_c, int jb, int je) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<V *>(X + jb), 0, (je - jb) * static_cast<int>(sizeof(V)), kBufferFlags);
    int at = 0;
    auto load_j = [&](int k) -> J {
      union {
        V4u w[sizeof(V) / 16];
        J j;
      } e;
#pragma unroll
      for (int h = 0; h < static_cast<int>(sizeof(V) / 16); ++h)
        e.w[h] = __builtin_amdgcn_raw_buffer_load_b128(
            rsrc, k * static_cast<int>(sizeof(V)) + 16 * h, at, 0);
      return e.j;
    };
    J p[kJAhead];
#pragma unroll
    for (int k = 0; k < kJAhead; ++k) p[k] = load_j(k);
    int j = jb;
    for (; j + kJAhead <= je; j += kJAhead) {
      at += kJAhead * static_cast<int>(sizeof(V));
#pragma unroll
      for (int k = 0; k < kJAhead; ++k) {
        pairs_of(diag_c, clamp_c, p[k], j + k);
        // into the registers the pairs have just freed
        p[k] = load_j(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int k = 0; k < kJAhead - 1; ++k)
      if (j + k < je) pairs_of(diag_c, clamp_c, p[k], j + k);
  };

  const int span = 64 * R;
  const int n_slice = (w.i1 - w.i0 + span - 1) / span;
  const int n_wave = static_cast<int>(blockDim.x) / 64;
  // j per unit: a power of two that gives every wave about four units
  int sub = a.tj;
  while (sub > kMinUnitJ && n_slice * ((w.j1 - w.j0 + sub - 1) / sub) < 4 * n_wave) sub >>= 1;
  const int n_unit = n_slice * ((w.j1 - w.j0 + sub - 1) / sub);
  // the wave that runs out of units first draws the workgroup's next item
  // while the others finish theirs
  if (wave == n_unit && lane == 0)
    *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  for (int u = wave; u < n_unit;) {
    const int slice = u % n_slice, piece = u / n_slice;
    const int wb = w.i0 + slice * span;
    int jb = w.j0 + piece * sub;
    const int je = min(jb + sub, w.j1);
    const bool diag = (w.flags & kItemDiag) != 0 && jb < wb + span;
    if (diag) jb = max(jb, wb + 1);
    if (jb < je) {
      if (wb != wbase) {
        wbase = wb;
        load_i();
      }
      if (diag)
        stream(Yes{}, Yes{}, jb, je);
      else if (noclamp && wb + span <= w.i1)
        stream(No{}, No{}, jb, je);
      else
        stream(No{}, Yes{}, jb, je);
    }
    int nu = 0;
    if (lane == 0) nu = atomicAdd(s_unit, 1);
    u = uni(nu);
    if (u == n_unit && lane == 0)
      *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  }
  if constexpr (SEARCH) {
    if (qn > 0) drain(qn);
    add_searched(s_search, lane, n_searched, n_images);
  }
}

// Workgroups of up to 1024 threads share one LDS histogram (more waves per
// CU when a wide histogram leaves room for one workgroup only). The image
// search keeps many more live values and is limited to 256 threads.
template <int BOX>
constexpr int max_threads() {
  return BOX == kBoxTricSearch ? 256 : 1024;
}

// Waves per SIMD the registers have to allow: eight for the binary32 kernels
// without image search and with four particles per lane, so that two
// workgroups of 1,024 threads share a CU where their histograms fit. A loop of
// the short path's instructions takes 41 cycles per pair of a wave with four
// waves per SIMD and 37 with eight (the root alone 14); 1M clustered points:
// 89.3 and 85.7 ms; 24 orthorhombic frames: 21.9 and 21.4 ms. Four for the
// binary64 search, which lies at the 128 registers of four waves (eight frames of
// 8,000 to 29,000 points in a batch: 4.92 ms at 126 registers, 5.17 at 129).
template <typename T, int R, int BOX>
constexpr int min_waves() {
  if (BOX == kBoxTricSearch) return sizeof(T) == 8 && R == 4 ? 4 : 1;
  return sizeof(T) == 4 && R == 4 ? 8 : 1;
}

template <typename T, int R, int BOX, int MODE>
__global__ __launch_bounds__(max_threads<BOX>(), (min_waves<T, R, BOX>())) void pairs_kernel(PairKernelArgs a) {
  using V = typename V4<T>::type;
  extern __shared__ __align__(32) unsigned char smem[];
  // control words: in-range counts of a flush, next item, next unit, and the
  // item's searched pairs and images
  unsigned long long &s_sum = *reinterpret_cast<unsigned long long *>(smem);
  int &s_item = *reinterpret_cast<int *>(smem + 8), &s_unit = *reinterpret_cast<int *>(smem + 12);
  unsigned long long *const s_search = reinterpret_cast<unsigned long long *>(smem + 16);
  // the histogram follows a guard of kGuardBytes: one word per copy for
  // binary32 bin -1 (t < 1/4), added to bin 0 on flush
  uint32_t *hist = reinterpret_cast<uint32_t *>(smem + kSlot0);
  const int tid = threadIdx.x;
  // image-search queues after the histogram, 32-byte aligned
  const size_t q_off = (kSlot0 + static_cast<size_t>(a.stride) * 4 + 31) / 32 * 32;
  V *queue = reinterpret_cast<V *>(smem + q_off);
  V *shifts = queue + (blockDim.x / 64) * queue_cap(R);

  constexpr bool GLOBAL = MODE == kModeGlobal;
  if constexpr (!GLOBAL)
    for (int k = tid - 1; k < a.stride; k += blockDim.x) hist[k] = 0u;

  if (tid == 0) s_sum = s_search[0] = s_search[1] = 0;
  int cur_frame = -1, cur_hist = -1, cur_sweep = -1;
  uint64_t acc = 0;
  // the first item of a workgroup is its own index, the others come from the
  // counter
  int it = blockIdx.x;
  while (it < a.n_items) {
    if (tid == 0) s_unit = static_cast<int>(blockDim.x) / 64;
    WorkItem w;
    {
      const WorkItem *p = a.items + it;
      w.frame = uni(p->frame); w.hist = uni(p->hist); w.sweep = uni(p->sweep);
      w.flags = uni(p->flags); w.i0 = uni(p->i0); w.i1 = uni(p->i1);
      w.j0 = uni(p->j0); w.j1 = uni(p->j1);
    }
    if constexpr (!GLOBAL) {
      const uint64_t npairs =
          static_cast<uint64_t>(w.i1 - w.i0) * static_cast<uint64_t>(w.j1 - w.j0);
      if (w.frame != cur_frame || w.hist != cur_hist || w.sweep != cur_sweep ||
          acc + npairs > 0xffffffffull) {
        if (cur_frame >= 0) flush_hist(hist, a, a.frames + cur_frame, cur_hist, cur_sweep, &s_sum);
        cur_frame = w.frame; cur_hist = w.hist; cur_sweep = w.sweep;
        acc = 0;
      }
      acc += npairs;
    }
    // the histogram is clear, the unit counter set
    __syncthreads();
    const FrameParams *F = a.frames + w.frame;
    if constexpr (sizeof(T) == 8 && (BOX == kBoxTricSorted || BOX == kBoxSearchSorted)) {
      run_sorted64<MODE, BOX == kBoxSearchSorted>(a, w, F, &s_unit, &s_item, s_search);
    } else if constexpr (BOX == kBoxTricSorted) {
      run_sorted<MODE>(a, w, F, &s_unit, &s_item);
    } else {
      run_units<T, R, BOX, MODE>(a, w, F, hist, queue, shifts, &s_unit, &s_item, s_search);
    }
    // every wave has counted the item, and the next one is known
    __syncthreads();
    it = uni(s_item);
    if constexpr (BOX == kBoxTricSearch || BOX == kBoxSearchSorted) {
      // (the next item's waves add after the barrier at its start)
      if (tid == 0 && F->searched != nullptr && (s_search[0] | s_search[1]) != 0) {
        atomicAdd(F->searched, s_search[0]);
        atomicAdd(F->searched + 1, s_search[1]);
        s_search[0] = s_search[1] = 0;
      }
    }
  }
  if constexpr (!GLOBAL)
    if (cur_frame >= 0) flush_hist(hist, a, a.frames + cur_frame, cur_hist, cur_sweep, &s_sum);
}

template <typename T, int R, int SW>
PairFn pick_box(int box) {
  switch (box) {
    case kBoxNone: return pairs_kernel<T, R, kBoxNone, SW>;
    case kBoxOrtho: return pairs_kernel<T, R, kBoxOrtho, SW>;
    case kBoxTric: return pairs_kernel<T, R, kBoxTric, SW>;
    case kBoxCube:
      if constexpr (sizeof(T) == 4) return pairs_kernel<T, R, kBoxCube, SW>;
      return pairs_kernel<T, R, kBoxOrtho, SW>;
    // (units of a sorted frame are the same for every R)
    case kBoxTricSorted: return pairs_kernel<T, 4, kBoxTricSorted, SW>;
    case kBoxSearchSorted:  // binary64 only
      if constexpr (sizeof(T) == 8) return pairs_kernel<T, 4, kBoxSearchSorted, SW>;
      return nullptr;
    default: return pairs_kernel<T, R, kBoxTricSearch, SW>;
  }
}

}  // namespace
}  // namespace dh
