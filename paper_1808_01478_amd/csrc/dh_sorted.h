// The pair kernel's work on spatially sorted frames (kBoxTricSorted and
// kBoxSearchSorted).
//
// The unit of work is a wave's: eight slices of 64 i-particles against eight
// groups of 64 j-particles. Each lane takes one (slice, group) pair of the 64
// and, from the two groups' bounding boxes, decides two things about all
// their pairs at once: which minimum-image arithmetic they take, and whether
// any of their distances can fall in the histogram at all. Group pairs beyond
// the cut-off (or outside the bin window) are never computed: their pairs
// are out of range, and the out-of-range count of a histogram is its pair
// count less what was counted. The others run group by group, the wave
// streaming the group's 64 j against as many slices as take the same path.
//
// Bound by vector-unit issue, so what is not computed is what counts: of the
// 1,000,000-point clustered triclinic frame (cut-off 22 in cells of 50) 41 %
// of the pairs are in range and 75 % are computed, 59 % of them all on the
// short path. With every pair computed, j-tiles in LDS and a barrier per tile
// the frame took 147 ms in binary32; skipping them in independent units
// took 90 ms, at eight waves per SIMD (half the registers) it takes 85 ms.
// Binary64 (run_sorted64): 371 and 162 ms.
#pragma once

#include "dh_internal.h"

namespace dh {
namespace {

constexpr int kUnitSlices = 8;  // i-slices of 64 per unit
constexpr int kUnitGroups = 8;  // j-groups of 64 per unit
static_assert(kUnitSlices * kUnitGroups == 64, "one (slice, group) pair per lane");
static_assert(kUnitPoints == 64 * kUnitSlices, "i-span of a unit");

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

template <int N>
using Int = std::integral_constant<int, N>;

// What the boxes of slice r and group g of a unit say about all their pairs
// (the lane's own pair; see run_sorted).
struct GroupPair {
  int kind;        // kFast, kFix + axis, kSlow, or kSkip
  bool diag;       // the same group: pairs j > i only
  bool in_window;  // every t below the LDS stride (no clamp needed)
  float sx, sy, sz;  // binary32: lattice shift B n of the lower-end wraps
  int n[3];          // binary64: the shared wraps
};
constexpr int kSkip = 0, kFast = 1, kFix = 2, kSlow = 5;  // kFix + axis: 2, 3, 4
// binary64 only: groups whose coordinates are too large for the bounds (or
// not finite)
constexpr int kExact = 6;

// Along an axis the fixed-point differences of the pairs lie in
// [jlo - ihi, jhi - ilo], and the wrap of u_j - u_i, floor((u_j - u_i + 2^31)
// / 2^32), is one of -1, 0, 1; it is shared by all pairs iff both ends give
// the same one. If every axis is shared, the pairs are `fast`: the Cartesian
// difference to the i-point shifted by B n. If exactly one axis is ambiguous
// and its two ends differ by one, they are `fix`: the shift of the lower
// ends, or one more cell vector B_K when the pair's fractional coordinate
// along K exceeds 1/2. Otherwise `slow`: the fixed-point words wrap per pair.
// The distance bounds take the Cartesian boxes under every wrap the pairs can
// have (a box spanning more than two wraps gives no bound).
//
// binary64 (F64): the intervals are widened by kWrapMargin, far more than the
// rounding of any fractional coordinate; `fix` and `slow` pairs round their
// one ambiguous axis, or all three, whatever its span, so the shift leaves
// out the ambiguous axes.
constexpr int64_t kWrapMargin = 1024;  // 2^-22 of a cell vector
template <bool F64>
__device__ __forceinline__ GroupPair classify(const GroupBox &I, const GroupBox &J,
                                              const float (&cell)[6], float r_lo, float r_hi,
                                              float r_in) {
  GroupPair p;
  int nl[3], nh[3];
  uint32_t amb = 0;
  bool wide = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if constexpr (F64) {
      const int64_t lo = static_cast<int64_t>(J.ulo[k]) - static_cast<int64_t>(I.uhi[k]);
      const int64_t hi = static_cast<int64_t>(J.uhi[k]) - static_cast<int64_t>(I.ulo[k]);
      nl[k] = static_cast<int>((lo - kWrapMargin + 0x80000000ll) >> 32);
      nh[k] = static_cast<int>((hi + kWrapMargin + 0x80000000ll) >> 32);
    } else {
      nl[k] = static_cast<int>(J.ulo[k] - I.uhi[k] >= 0x80000000u) -
              static_cast<int>(J.ulo[k] < I.uhi[k]);
      nh[k] = static_cast<int>(J.uhi[k] - I.ulo[k] >= 0x80000000u) -
              static_cast<int>(J.uhi[k] < I.ulo[k]);
    }
    amb |= nl[k] != nh[k] ? 1u << k : 0u;
    wide = wide || nh[k] - nl[k] > 1;
  }
  p.kind = amb == 0u ? kFast
                     : ((amb & (amb - 1u)) == 0u && (F64 || !wide) ? kFix + (amb == 1u ? 0 : amb == 2u ? 1 : 2)
                                                          : kSlow);
  auto shift = [&](int na, int nb, int nc, float &x, float &y, float &z) {
    const float fa = static_cast<float>(na), fb = static_cast<float>(nb),
                fc = static_cast<float>(nc);
    x = (fa * cell[0] + fb * cell[1]) + fc * cell[3];
    y = fb * cell[2] + fc * cell[4];
    z = fc * cell[5];
  };
  float lo2 = __builtin_inff(), hi2 = 0.f;
  auto bound = [&](int na, int nb, int nc) {
    float x, y, z;
    shift(na, nb, nc, x, y, z);
    // the difference d = j - (i + S) along each Cartesian axis
    const float ax = J.clo[0] - (I.chi[0] + x), bx = J.chi[0] - (I.clo[0] + x);
    const float ay = J.clo[1] - (I.chi[1] + y), by = J.chi[1] - (I.clo[1] + y);
    const float az = J.clo[2] - (I.chi[2] + z), bz = J.chi[2] - (I.clo[2] + z);
    const float gx = fmaxf(fmaxf(ax, -bx), 0.f), gy = fmaxf(fmaxf(ay, -by), 0.f),
                gz = fmaxf(fmaxf(az, -bz), 0.f);
    const float fx = fmaxf(-ax, bx), fy = fmaxf(-ay, by), fz = fmaxf(-az, bz);
    lo2 = fminf(lo2, gx * gx + gy * gy + gz * gz);
    hi2 = fmaxf(hi2, fx * fx + fy * fy + fz * fz);
  };
  bound(nl[0], nl[1], nl[2]);
  if (__builtin_amdgcn_ballot_w64(amb != 0u) != 0)
    for (int c = 1; c < 8; ++c)
      bound(c & 1 ? nh[0] : nl[0], c & 2 ? nh[1] : nl[1], c & 4 ? nh[2] : nl[2]);
  // (comparisons of this form keep a pair of groups whose bounds are NaN)
  const bool out = lo2 > r_hi * r_hi || hi2 < r_lo * r_lo;
  if (out && !wide) p.kind = kSkip;
  p.in_window = !wide && hi2 < r_in * r_in;
  p.diag = false;
  if constexpr (F64) {
#pragma unroll
    for (int k = 0; k < 3; ++k) p.n[k] = nl[k] == nh[k] ? nl[k] : 0;
  } else {
    shift(nl[0], nl[1], nl[2], p.sx, p.sy, p.sz);
  }
  return p;
}

// Distance bounds of a bin window in length units, widened by far more than
// the rounding of any pair's distance: a pair outside [lo, hi] cannot count,
// one inside `in` needs no clamp (its t is below the LDS stride; slots past
// the window are never flushed).
struct WindowBounds {
  float lo, hi, in;
  float slack;  // the absolute part of the widening
};
__device__ __forceinline__ WindowBounds window_bounds(const FrameParams *F, int b_lo, int win,
                                                      int stride) {
  float size = 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) size += fabsf(uni(F->cell32[k]));
  const float eps = size * 0x1p-16f, s = uni(F->s32);
  WindowBounds b;
  b.slack = eps;
  b.lo = b_lo > 0 ? fmaxf(static_cast<float>(b_lo) / s * (1.f - 0x1p-12f) - eps, 0.f) : 0.f;
  b.hi = static_cast<float>(b_lo + win) / s * (1.f + 0x1p-12f) + eps;
  b.in = fmaxf(static_cast<float>(stride - 2) / s * (1.f - 0x1p-12f) - eps, 0.f);
  if (!bounds_decide(size)) {
    b.lo = b.in = 0.f;
    b.hi = __builtin_inff();
  }
  return b;
}

// One work item of a spatially sorted binary32 frame, in units drawn from the
// LDS counter s_unit as for unsorted frames. A pair's path and arithmetic
// depend only on its two groups (species-aligned blocks of 64 points), not on
// the unit, the item or the other slices of the wave, so every launch shape,
// batch and server path gives the same counts.
template <int MODE>
__device__ __forceinline__ void run_sorted(const PairKernelArgs &a, const WorkItem &w,
                                           const FrameParams *F, int *s_unit, int *s_item) {
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const char *const staged = uni(static_cast<const char *>(F->coords));
  const int64_t n_pad = uni(static_cast<int>(F->n_pad));
  const float4 *const C = reinterpret_cast<const float4 *>(staged);
  const uint32_t *const W = reinterpret_cast<const uint32_t *>(staged + 16 * n_pad);
  const GroupBox *const boxes = reinterpret_cast<const GroupBox *>(staged + 28 * n_pad);
  const Geo32 g32 = load_geo32(F);
  float cell[6], h[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    cell[k] = uni(F->cell32[k]);
    h[k] = uni(F->hinv32[k]);
  }
  const float s32 = uni(F->s32) * kBinScale;
  const int win = uni(F->win);
  const WindowBounds wb = window_bounds(F, w.sweep * win, win, a.stride);
  const bool noclamp = MODE == kModeLds && uni(F->noclamp) != 0;
  const Count<MODE> count(F, w, lane);
  using Yes = std::true_type;
  using No = std::false_type;

  // the unit: its first i and j, and this lane's group pair
  int ib = 0, jb = 0;
  GroupPair gp;
  // row K of B^-1 applied to a point: its fractional coordinate along K
  // (up to the constant of the cell centre)
  auto proj = [&](auto axis_c, float x, float y, float z) {
    constexpr int K = decltype(axis_c)::value;
    if constexpr (K == 0)
      return fmaf(z, h[2], fmaf(y, h[1], x * h[0]));
    else if constexpr (K == 1)
      return fmaf(z, h[4], y * h[3]);
    else
      return z * h[5];
  };
  // Runs body(j, its entry) over the group's j, AHEAD of them in flight.
  auto run_j = [&](auto ahead_c, auto words_c, int j0, auto &&body) {
    constexpr int AHEAD = decltype(ahead_c)::value;
    constexpr int STRIDE = decltype(words_c)::value ? 12 : 16;
    const int j1 = min(j0 + 64, w.j1);
    const void *first = decltype(words_c)::value ? static_cast<const void *>(W + first_word(j0))
                                                 : static_cast<const void *>(C + j0);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(first), 0, (j1 - j0) * STRIDE + (16 - STRIDE), kBufferFlags);
    int off = 0;
    auto load = [&](int k) {
      // (a read of three words takes the next one along, unused: after the
      // last point's words come the group boxes)
      const V4u v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, k * STRIDE, off, 0);
      return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                         __uint_as_float(v.w));
    };
    float4 p[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) p[k] = load(k);
    int j = j0;
    for (; j + AHEAD <= j1; j += AHEAD) {
      off += AHEAD * STRIDE;
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        body(p[k], j + k);
        p[k] = load(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int k = 0; k < AHEAD - 1; ++k)
      if (j + k < j1) body(p[k], j + k);
  };
  // One group against M slices (four bits each in rs) of one kind.
  auto pass = [&](auto kind_c, auto m_c, auto clamp_c, auto diag_c, uint32_t rs, int g) {
    constexpr int KIND = decltype(kind_c)::value, M = decltype(m_c)::value;
    constexpr bool DIAG = decltype(diag_c)::value;
    const int j0 = jb + 64 * g;
    if constexpr (KIND == kSlow) {
      // -(b:a) of the i-points and -(c:c'), c' the c of the point 64 before an
      // odd slice's and 0 otherwise: the upper word of one 64-bit addition to
      // j's (c:c) is the c difference, an odd slice's lowered by one unit when
      // the even one borrows, as in unsorted frames
      uint64_t nab[M], nzz[M];
      float off[M];
      [[maybe_unused]] int i0 = 0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int r = static_cast<int>((rs >> (4 * k)) & 15u);
        const int i = ib + 64 * r + lane;
        const bool ok = i < w.i1;
        const uint32_t *const wi = W + first_word(ok ? i : ib);
        const uint32_t zb = r & 1 ? W[first_word(ok ? i - 64 : ib) + 2] : 0u;
        nab[k] = 0ull - ((static_cast<uint64_t>(wi[1]) << 32) | wi[0]);
        nzz[k] = 0ull - ((static_cast<uint64_t>(wi[2]) << 32) | zb);
        off[k] = ok ? kBinOffset : kNoBin;
        if constexpr (DIAG) i0 = i;
      }
      run_j(Int<4>{}, Yes{}, j0, [&](const float4 &e, int j) {
        const uint64_t ab =
            (static_cast<uint64_t>(__float_as_uint(e.y)) << 32) | __float_as_uint(e.x);
        const uint64_t cc =
            (static_cast<uint64_t>(__float_as_uint(e.z)) << 32) | __float_as_uint(e.z);
#pragma unroll
        for (int k = 0; k < M; ++k) {
          const float fc = static_cast<float>(
              static_cast<int32_t>(static_cast<uint32_t>((cc + nzz[k]) >> 32)));
          count.template add<true>(bits32_packed_c<kBoxTric>(
              ab, nab[k], fc, g32, DIAG && j <= i0 ? kNoBin : off[k]));
        }
      });
    } else {
      // A lane past the end of the item holds an i-point at infinity: its q is
      // +inf, which the clamp discards.
      float sx[M], sy[M], sz[M];
      // fix: the threshold j's projection must exceed and the i-point shifted
      // by one more cell vector B_K
      [[maybe_unused]] float th[M], ux[M], uy[M], uz[M];
      constexpr int K = KIND >= kFix ? KIND - kFix : 0;
      [[maybe_unused]] int i0 = 0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int r = static_cast<int>((rs >> (4 * k)) & 15u);
        const int i = ib + 64 * r + lane;
        const bool ok = i < w.i1;
        const float4 c = C[ok ? i : ib];
        const int src = g * kUnitSlices + r;
        const float inf = __builtin_inff();
        sx[k] = (ok ? c.x : inf) + lane_value(gp.sx, src);
        sy[k] = (ok ? c.y : inf) + lane_value(gp.sy, src);
        sz[k] = (ok ? c.z : inf) + lane_value(gp.sz, src);
        if constexpr (DIAG) i0 = i;
        if constexpr (KIND >= kFix) {
          th[k] = proj(Int<K>{}, sx[k], sy[k], sz[k]) + 0.5f;
          ux[k] = sx[k] + (K == 0 ? cell[0] : K == 1 ? cell[1] : cell[3]);
          uy[k] = K == 0 ? sy[k] : sy[k] + (K == 1 ? cell[2] : cell[4]);
          uz[k] = K == 2 ? sz[k] + cell[5] : sz[k];
        }
      }
      run_j(Int<(M >= 8 ? 2 : 4)>{}, No{}, j0, [&](const float4 &c, int j) {
        [[maybe_unused]] float pj = 0.f;
        if constexpr (KIND >= kFix) pj = proj(Int<K>{}, c.x, c.y, c.z);
#pragma unroll
        for (int k = 0; k < M; ++k) {
          float x = sx[k], y = sy[k], z = sz[k];
          if constexpr (KIND >= kFix) {
            const bool up = pj > th[k];
            x = up ? ux[k] : x;
            if constexpr (K >= 1) y = up ? uy[k] : y;
            if constexpr (K == 2) z = up ? uz[k] : z;
          }
          const float dx = c.x - x, dy = c.y - y, dz = c.z - z;
          const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
          const float o = DIAG && j <= i0 ? kNoBin : kBinOffset;
          count.template add<decltype(clamp_c)::value>(
              __float_as_uint(fmaf(__builtin_amdgcn_sqrtf(q), s32, o)));
        }
      });
    }
  };
  // the slices in `m` (bit r) against group g, in passes of as many as fit
  auto passes = [&](auto kind_c, auto clamp_c, uint32_t m, int g) {
    auto take = [&](int n) {
      uint32_t rs = 0;
      for (int k = 0; k < n; ++k) {
        rs |= static_cast<uint32_t>(__builtin_ctz(m)) << (4 * k);
        m &= m - 1u;
      }
      return rs;
    };
    if constexpr (decltype(kind_c)::value == kFast)
      if (__builtin_popcount(m) >= 8) pass(kind_c, Int<8>{}, clamp_c, No{}, take(8), g);
    while (__builtin_popcount(m) >= 4) pass(kind_c, Int<4>{}, clamp_c, No{}, take(4), g);
    if (__builtin_popcount(m) >= 2) pass(kind_c, Int<2>{}, clamp_c, No{}, take(2), g);
    if (m != 0u) pass(kind_c, Int<1>{}, clamp_c, No{}, take(1), g);
  };

  const int n_ib = (w.i1 - w.i0 + kUnitPoints - 1) / kUnitPoints;
  // groups per unit: as many as leave every wave about four units
  const int n_wave = static_cast<int>(blockDim.x) / 64;
  int gpu = kUnitGroups;
  while (gpu > 1 && n_ib * ((w.j1 - w.j0 + 64 * gpu - 1) / (64 * gpu)) < 4 * n_wave) gpu >>= 1;
  const int n_unit = n_ib * ((w.j1 - w.j0 + 64 * gpu - 1) / (64 * gpu));
  if (wave == n_unit && lane == 0)
    *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  for (int u = wave; u < n_unit;) {
    ib = w.i0 + (u % n_ib) * kUnitPoints;
    jb = w.j0 + (u / n_ib) * 64 * gpu;
    {
      const int r = lane % kUnitSlices, gr = lane / kUnitSlices;
      const int gi = (ib >> 6) + r, gj = (jb >> 6) + gr;
      const bool valid = ib + 64 * r < w.i1 && gr < gpu && jb + 64 * gr < w.j1 &&
                         !((w.flags & kItemDiag) && gj < gi);
      gp = classify<false>(boxes[valid ? gi : ib >> 6], boxes[valid ? gj : jb >> 6], cell, wb.lo, wb.hi,
                    wb.in);
      gp.diag = (w.flags & kItemDiag) && gj == gi;
      gp.in_window = (gp.in_window || noclamp) && ib + 64 * r + 64 <= w.i1;
      if (!valid) gp.kind = kSkip;
    }
    const uint64_t m_fast = __builtin_amdgcn_ballot_w64(gp.kind == kFast && !gp.diag);
    const uint64_t m_in = __builtin_amdgcn_ballot_w64(gp.in_window);
    const uint64_t m_fix0 = __builtin_amdgcn_ballot_w64(gp.kind == kFix && !gp.diag);
    const uint64_t m_fix1 = __builtin_amdgcn_ballot_w64(gp.kind == kFix + 1 && !gp.diag);
    const uint64_t m_fix2 = __builtin_amdgcn_ballot_w64(gp.kind == kFix + 2 && !gp.diag);
    const uint64_t m_slow = __builtin_amdgcn_ballot_w64(gp.kind == kSlow && !gp.diag);
    const uint64_t m_diag = __builtin_amdgcn_ballot_w64(gp.kind != kSkip && gp.diag);
    for (int g = 0; g < gpu; ++g) {
      auto bits = [&](uint64_t m) {
        return static_cast<uint32_t>(m >> (g * kUnitSlices)) & ((1u << kUnitSlices) - 1u);
      };
      const uint32_t fast = bits(m_fast);
      if (MODE == kModeLds && (fast & ~bits(m_in)) == 0u)
        passes(Int<kFast>{}, No{}, fast, g);
      else
        passes(Int<kFast>{}, Yes{}, fast, g);
      passes(Int<kFix>{}, Yes{}, bits(m_fix0), g);
      passes(Int<kFix + 1>{}, Yes{}, bits(m_fix1), g);
      passes(Int<kFix + 2>{}, Yes{}, bits(m_fix2), g);
      passes(Int<kSlow>{}, Yes{}, bits(m_slow), g);
      if (const uint32_t m = bits(m_diag)) {
        // at most one slice of the unit is the group itself
        const uint32_t r = static_cast<uint32_t>(__builtin_ctz(m));
        switch (__builtin_amdgcn_readlane(gp.kind, g * kUnitSlices + static_cast<int>(r))) {
          case kFast: pass(Int<kFast>{}, Int<1>{}, Yes{}, Yes{}, r, g); break;
          case kFix: pass(Int<kFix>{}, Int<1>{}, Yes{}, Yes{}, r, g); break;
          case kFix + 1: pass(Int<kFix + 1>{}, Int<1>{}, Yes{}, Yes{}, r, g); break;
          case kFix + 2: pass(Int<kFix + 2>{}, Int<1>{}, Yes{}, Yes{}, r, g); break;
          default: pass(Int<kSlow>{}, Int<1>{}, Yes{}, Yes{}, r, g); break;
        }
      }
    }
    int nu = 0;
    if (lane == 0) nu = atomicAdd(s_unit, 1);
    u = uni(nu);
    if (u == n_unit && lane == 0)
      *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  }
}

// The images of a pair of groups of a frame with image search (binary64): the
// lattice shifts N under which some pair of the two groups can be nearest and
// within the window, as an ordered list of at most kListed, from the distance
// bounds of the groups' boxes under every N that a pair can need (its Eq. 5
// wrap and one more step either way). A shift whose lower bound exceeds the
// smallest upper bound is never the nearest; one beyond the window's end can
// be the nearest only of pairs that are out of range, whose other images are
// farther still. Frames come here only when no image outside the 27 of the
// canonical search is ever nearest (see staged_kind), so the canonical minimum
// over a pair's 27 images is the minimum over this list.
constexpr int kListed = 8;
struct Images {
  uint64_t list;  // eight bits each: (a + 2) + 5 (b + 2) + 25 (c + 2)
  int n;          // entries; kListed + 1: more than fit
  float far2;     // square of an upper bound of every pair's distance
};
__device__ __forceinline__ Images group_images(const GroupBox &I, const GroupBox &J,
                                               const float (&cell)[6], float r_hi, float slack) {
  int n_lo[3], n_hi[3];
  float dc[3], hw[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int64_t lo = static_cast<int64_t>(J.ulo[k]) - static_cast<int64_t>(I.uhi[k]);
    const int64_t hi = static_cast<int64_t>(J.uhi[k]) - static_cast<int64_t>(I.ulo[k]);
    n_lo[k] = static_cast<int>((lo - kWrapMargin + 0x80000000ll) >> 32) - 1;
    n_hi[k] = static_cast<int>((hi + kWrapMargin + 0x80000000ll) >> 32) + 1;
    // centre and half width of the interval of j - i
    dc[k] = 0.5f * ((J.clo[k] + J.chi[k]) - (I.clo[k] + I.chi[k]));
    hw[k] = 0.5f * ((J.chi[k] - J.clo[k]) + (I.chi[k] - I.clo[k]));
  }
  // squares of the least and largest distance of a pair under each shift
  auto scan = [&](auto &&visit) {
    for (int c = -2; c <= 2; ++c) {
      const float fc = static_cast<float>(c), tz = fabsf(dc[2] - fc * cell[5]);
      const float gz = fmaxf(tz - hw[2], 0.f), fz = tz + hw[2];
      for (int b = -2; b <= 2; ++b) {
        const float fb = static_cast<float>(b), ty = fabsf(dc[1] - (fb * cell[2] + fc * cell[4]));
        const float gy = fmaxf(ty - hw[1], 0.f), fy = ty + hw[1];
        const float g2 = gz * gz + gy * gy, f2 = fz * fz + fy * fy;
        const bool in = c >= n_lo[2] && c <= n_hi[2] && b >= n_lo[1] && b <= n_hi[1];
        for (int a = -2; a <= 2; ++a) {
          const float tx = fabsf(dc[0] - (static_cast<float>(a) * cell[0] + fb * cell[1] +
                                          fc * cell[3]));
          const float gx = fmaxf(tx - hw[0], 0.f), fx = tx + hw[0];
          visit(in && a >= n_lo[0] && a <= n_hi[0], g2 + gx * gx, f2 + fx * fx,
                (a + 2) + 5 * (b + 2) + 25 * (c + 2));
        }
      }
    }
  };
  Images m;
  m.far2 = __builtin_inff();
  scan([&](bool in, float, float f2, int) { m.far2 = in ? fminf(m.far2, f2) : m.far2; });
  // widened by far more than the rounding of the bounds and of any distance
  const float lim = fminf(__builtin_sqrtf(m.far2) * (1.f + 0x1p-12f) + slack, r_hi);
  m.list = 0;
  m.n = 0;
  scan([&](bool in, float g2, float, int id) {
    if (in && g2 <= lim * lim) {
      if (m.n < kListed) m.list |= static_cast<uint64_t>(id) << (8 * m.n);
      m.n = m.n <= kListed ? m.n + 1 : m.n;
    }
  });
  return m;
}

// Pairs gathered in the lanes of a wave, from whatever i and j, for arithmetic that
// few of them need: lane q < n holds the word of one.
struct LaneQueue {
  int held = 0, n = 0;
  // takes in the words of the lanes that say so; a full wave of them goes to drain
  template <typename F>
  __device__ __forceinline__ void push(bool take, int word, F &&drain) {
    const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63, cnt = __builtin_popcountll(mask);
    const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
        static_cast<uint32_t>(mask >> 32),
        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
    // the lanes taken to n, n + 1, ... (round the wave), the others after them
    const int to = n + (take ? below : cnt + lane - below);
    const int got = __builtin_amdgcn_ds_permute((to & 63) << 2, word);
    held = lane >= n ? got : held;
    n += cnt;
    if (n >= 64) {
      drain(held, 64);
      held = got;
      n -= 64;
    }
  }
  template <typename F>
  __device__ __forceinline__ void finish(F &&drain) {
    if (n > 0) drain(held, n);
    n = 0;
  }
};

// Pairs of a sorted binary64 frame next to a bin edge. A pass leaves its pairs
// of two j here as soon as one of them is too close to an edge (see
// run_sorted64): each pair's bin is taken again from the staged positions, the
// pairs near an edge of the window are gathered in lanes, from whatever i and
// j, and 64 at a time go through the canonical sequence on their input points.
// With random points about one pass in 10^5 leaves anything; where distances
// repeat at whole bins (a crystal, the bin a fraction of its spacing) all of
// them leave everything, some per cent of it near an edge. 103,823 points of a
// cubic lattice (spacing 3.61, cut-off 70, 7,000 bins): 11.9 ms with the
// canonical sequence for every pair left, 10.3 ms unsorted with a binary64
// root per pair, 6.7 ms with this; random points of the same frame 2.7 ms.
// Groups without a rounding bound (kExact) are taken from the input throughout,
// as an unsorted frame's: 100,000 points of a cube, all too far out for a bound,
// 7.3 ms (19.1 with the canonical sequence for each pair).
//
// The first m slices in rs (four bits each) of the unit at ib against the j of
// [j0, j1) in `left` (bit b: j0 + 2b and the next). SEARCH: the images of slice
// r and the group are those of lane src + r; without, its shift.
constexpr int kSettleDiag = 1, kSettleExact = 2, kSettleFast = 4;
template <int MODE, bool SEARCH>
__device__ __attribute__((noinline)) void settle_pairs(const FrameParams *frame, WorkItem w, int ib_,
                                                       int j0_, int j1_, uint32_t rs_, int m_,
                                                       uint32_t left_, int flags_, int src_,
                                                       float near_, double shx, double shy,
                                                       double shz, Images img) {
  const FrameParams *const F = uni(frame);
  const int ib = uni(ib_), i1 = uni(w.i1), j0 = uni(j0_), j1 = uni(j1_), m = uni(m_);
  const int flags = uni(flags_), src = uni(src_);
  const uint32_t rs = static_cast<uint32_t>(uni(static_cast<int>(rs_)));
  const float near_hi = uni(near_);
  w.hist = uni(w.hist);
  w.sweep = uni(w.sweep);
  const int lane = threadIdx.x & 63;
  const int64_t n_pad = F->n_pad;
  const double *const P = static_cast<const double *>(F->coords);
  const uint32_t *const index =
      reinterpret_cast<const uint32_t *>(static_cast<const char *>(F->coords) + 24 * n_pad);
  const double *const in = F->in;
  const Geo64 g = load_geo64(F);
  // (as in run_sorted64)
  const double s = g.s * 0x1p-22, is = 1.0 / s;
  const double ax = g.ax * s, bx = g.bx * s, by = g.by * s;
  const double cx = g.cx * s, cy = g.cy * s, cz = g.cz * s;
  const Count<MODE> count(F, w, lane);
  const int b_lo = w.sweep * uni(F->win), b_hi = b_lo + uni(F->win);

  // pairs for the canonical sequence, as the offsets of i from ib and j from j0
  LaneQueue queue;
  auto drain = [&](int word, int cnt) {
    const bool v = lane < cnt;
    const int64_t p = 3 * static_cast<int64_t>(index[v ? ib + (word & 511) : ib]);
    const int64_t q = 3 * static_cast<int64_t>(index[v ? j0 + (word >> 9) : j0]);
    const double t = t64<SEARCH ? kBoxTricSearch : kBoxTric>(in[p], in[p + 1], in[p + 2], in[q],
                                                             in[q + 1], in[q + 2], g);
    // (a NaN t takes the other operand: out of range)
    const uint32_t b = kBinBits + static_cast<uint32_t>(min_arith(t, 0x1p25));
    count.template add<true>(v ? b : kNoBits);
  };

  // the staged or, for groups without a rounding bound, the input points;
  // lane l holds the group's point l
  const bool exact = (flags & kSettleExact) != 0;
  auto point = [&](int at) {
    return exact ? in + 3 * static_cast<int64_t>(index[at]) : P + 3 * static_cast<int64_t>(at);
  };
  const double *const pj = point(j0 + lane < j1 ? j0 + lane : j0);
  const double jx = pj[0], jy = pj[1], jz = pj[2];
  const Bins64 bins = bins64(F);
  auto frac = [&](double x, double y, double z, double (&f)[3]) {
    f[0] = fma(z, g.h13 * is, fma(y, g.h12 * is, x * (g.h11 * is)));
    f[1] = fma(z, g.h23 * is, y * (g.h22 * is));
    f[2] = z * (g.h33 * is);
  };
  for (int k = 0; k < m; ++k) {
    const int r = static_cast<int>((rs >> (4 * k)) & 15u), at = src + r;
    const int i = ib + 64 * r + lane;
    const double *const pi = point(i < i1 ? i : ib);
    double x = pi[0], y = pi[1], z = pi[2];
    [[maybe_unused]] uint64_t list = 0;
    [[maybe_unused]] int n_img = 0;
    [[maybe_unused]] double fi[3];
    if constexpr (SEARCH) {
      list = static_cast<uint64_t>(static_cast<uint32_t>(
                 __builtin_amdgcn_readlane(static_cast<int>(img.list), at))) |
             static_cast<uint64_t>(static_cast<uint32_t>(
                 __builtin_amdgcn_readlane(static_cast<int>(img.list >> 32), at)))
                 << 32;
      n_img = __builtin_amdgcn_readlane(img.n, at);
    } else if (!exact) {
      x += lane_value(shx, at);
      y += lane_value(shy, at);
      z += lane_value(shz, at);
      frac(x, y, z, fi);
    }
    for (uint32_t left = static_cast<uint32_t>(uni(static_cast<int>(left_))); left != 0u;
         left &= left - 1u)
      for (int h = 0; h < 2; ++h) {
        const int o = 2 * __builtin_ctz(left) + h, j = j0 + o;
        if (j >= j1) continue;
        const bool counts = i < i1 && (!(flags & kSettleDiag) || j > i);
        if (exact) {
          // as an unsorted frame's pair
          double dx, dy, dz;
          reduce64<kBoxTric>(x, y, z, lane_value(jx, o), lane_value(jy, o), lane_value(jz, o), g,
                             dx, dy, dz);
          double q = fma(dz, dz, fma(dy, dy, dx * dx));
          if constexpr (SEARCH) q = search_q64(dx, dy, dz, q, g);
          float gap = __builtin_inff();
          uint32_t b = root_bits64(q * bins.scale, gap);
          if (__builtin_expect(any_near(gap, bins), 0)) b = canonical_bits(q, bins.s);
          count.template add<true>(counts ? b : kNoBits);
          continue;
        }
        double dx = lane_value(jx, o) - x, dy = lane_value(jy, o) - y, dz = lane_value(jz, o) - z;
        double u = 0.0;
        if constexpr (SEARCH) {
          for (int e = 0; e < n_img; ++e) {
            const int id = static_cast<int>((list >> (8 * e)) & 255u);
            const double na = id % 5 - 2, nb = id / 5 % 5 - 2, nc = id / 25 - 2;
            const double vx = dx - ((na * ax + nb * bx) + nc * cx), vy = dy - (nb * by + nc * cy),
                         vz = dz - nc * cz;
            const double v = fma(vz, vz, fma(vy, vy, vx * vx));
            u = e == 0 ? v : min_arith(u, v);
          }
        } else {
          if (!(flags & kSettleFast)) {
            double fj[3];
            frac(lane_value(jx, o), lane_value(jy, o), lane_value(jz, o), fj);
            const double na = rint(fj[0] - fi[0]), nb = rint(fj[1] - fi[1]),
                         nc = rint(fj[2] - fi[2]);
            dz = fma(-cz, nc, dz);
            dy = fma(-cy, nc, fma(-by, nb, dy));
            dx = fma(-cx, nc, fma(-bx, nb, fma(-ax, na, dx)));
          }
          u = fma(dz, dz, fma(dy, dy, dx * dx));
        }
        float gap = __builtin_inff();
        const uint32_t b = root_bits64(u, gap);
        // the pair's bin is b or a neighbour: settled when it is not near an
        // edge, when it is within half a bin of 0 (coincident points), or when
        // none of the three is in the window
        const int bin = static_cast<int>(b - kBinBits);
        const bool open =
            counts && gap <= near_hi && u >= 0x1p-46 && bin >= b_lo - 1 && bin <= b_hi;
        count.template add<true>(counts && !open ? b : kNoBits);
        queue.push(open, (i - ib) | (j - j0) << 9, drain);
      }
  }
  queue.finish(drain);
}

// Rounding between the inputs and a coordinate difference of a pair of two
// groups (binary64), here and in the canonical sequence: each of the dozen steps
// rounds something no larger than the two points' |x| + |y| + |z| plus the cell,
// so 2^-48 of that covers them; dt is that times s, in scaled units. Whether the
// groups' coordinates are small enough for it to decide anything (false for a
// group that is not finite); hm is the largest entry of B^-1. Up to 2^24 cells
// out, a pair's fractional differences here and in the canonical sequence (each
// some eight roundings of 2^-53 of hm mag) agree to 2^-25, well within
// kWrapMargin; where they round to different wraps the pair is out of range
// under both (see staged_kind).
__device__ __forceinline__ bool rounding_bound(const GroupBox &I, const GroupBox &J,
                                               const float (&cell)[6], double s, double hm,
                                               double &dt) {
  const double size = static_cast<double>(fabsf(cell[0]) + fabsf(cell[1]) + fabsf(cell[2]) +
                                          fabsf(cell[3]) + fabsf(cell[4]) + fabsf(cell[5]));
  const double mag = static_cast<double>(I.mag) + static_cast<double>(J.mag) + size;
  dt = 0x1p-48 * mag * s;
  return dt < 0x1p-25 && hm * mag < 0x1p24;
}

// The pairs of a unit of a sorted frame with image search that the search is
// defined for: Eq. 5 vector of the canonical sequence at least half the
// shortest lattice vector long (q >= qskip64), whatever the images evaluated.
// Pairs of groups whose boxes lie on one side of that sphere count without a
// look at their pairs. The others are looked at in binary32, groups with one
// shared wrap by their shifted positions, the others wrapped as 32-bit fixed-point
// fractions (see dh_pairs.h), and where its rounding could decide, of the length
// or of a wrap, by the canonical sequence on the input.
// The frame of 70,001 points takes 4.6 ms with the count and 4.0 without (7.1
// with it in binary64, a slice at a time; 10.6 before such frames were sorted);
// 74,088 points of a grid, whose wraps tie, 5.0 ms, 6.3 with the canonical
// sequence for all pairs of a tie's slice.
__device__ __attribute__((noinline)) uint64_t searched_pairs(const FrameParams *frame, WorkItem w,
                                                             int ib_, int jb_, int gpu_) {
  const FrameParams *const F = uni(frame);
  const int ib = uni(ib_), jb = uni(jb_), gpu = uni(gpu_), i1 = uni(w.i1), j1 = uni(w.j1);
  const bool diag_item = (uni(w.flags) & kItemDiag) != 0;
  const int lane = threadIdx.x & 63;
  const int64_t n_pad = F->n_pad;
  const char *const staged = static_cast<const char *>(F->coords);
  const double *const P = reinterpret_cast<const double *>(staged);
  const uint32_t *const index = reinterpret_cast<const uint32_t *>(staged + 24 * n_pad);
  const GroupBox *const boxes = reinterpret_cast<const GroupBox *>(staged + 28 * n_pad);
  const double *const in = F->in;
  float cell[6], size = 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    cell[k] = uni(F->cell32[k]);
    size += fabsf(cell[k]);
  }
  const Geo64 geo = load_geo64(F);
  const Geo32 g32 = load_geo32(F);
  const double qskip = uni(F->qskip64);
  const float radius = static_cast<float>(sqrt_cr(qskip)), slack = size * 0x1p-16f;

  const int r = lane % kUnitSlices, gr = lane / kUnitSlices;
  const int gi = (ib >> 6) + r, gj = (jb >> 6) + gr;
  const bool valid =
      ib + 64 * r < i1 && gr < gpu && jb + 64 * gr < j1 && !(diag_item && gj < gi);
  const bool diag = diag_item && gj == gi;
  const GroupBox &bi = boxes[valid ? gi : ib >> 6], &bj = boxes[valid ? gj : jb >> 6];
  // (widened as the distance bounds of a window)
  const GroupPair gp = classify<true>(bi, bj, cell, 0.f, radius * (1.f + 0x1p-12f) + slack,
                                      fmaxf(radius * (1.f - 0x1p-12f) - slack, 0.f));
  double dt;
  const double hm = fmax(fmax(fabs(geo.h11), fabs(geo.h12)),
                         fmax(fmax(fabs(geo.h13), fabs(geo.h22)),
                              fmax(fabs(geo.h23), fabs(geo.h33))));
  const bool bounded = rounding_bound(bi, bj, cell, geo.s * 0x1p-22, hm, dt);
  const bool longer = bounded && gp.kind == kSkip, shorter = bounded && gp.in_window && !longer;
  const int n_i = min(64, i1 - (ib + 64 * r)), n_j = min(64, j1 - (jb + 64 * gr));
  int sum = !valid || shorter ? 0 : diag ? n_j * (n_j - 1) / 2 : n_i * n_j;
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  int below = 0;  // pairs under qskip among those looked at
  const bool look = valid && !longer && !shorter;
  const uint64_t m_look = __builtin_amdgcn_ballot_w64(look);
  const uint64_t m_exact = __builtin_amdgcn_ballot_w64(look && !bounded);
  const uint64_t m_wrap = __builtin_amdgcn_ballot_w64(look && gp.kind != kFast);

  // Groups with one shared wrap: binary32 positions with its shift, lengths in
  // units of the cell; the others: fixed-point fractions, in units of 2^-32 of
  // a_x. A component of either vector is off by less than 2^-21 of the sum of the
  // cell's entries.
  const float off = size * 0x1p-20f, unit = 0x1p32f / cell[0];
  const float r_lo = fmaxf(radius - off, 0.f), r_hi = radius + off;
  const double shx = gp.n[0] * geo.ax + gp.n[1] * geo.bx + gp.n[2] * geo.cx,
               shy = gp.n[1] * geo.by + gp.n[2] * geo.cy, shz = gp.n[2] * geo.cz;
  const double len = 1.0 / (geo.s * 0x1p-22), to = len * 0x1p32;
  const double h11 = geo.h11 * to, h12 = geo.h12 * to, h13 = geo.h13 * to;
  const double h22 = geo.h22 * to, h23 = geo.h23 * to, h33 = geo.h33 * to;
  // a staged point as three words: its fractions, or its position plus S
  auto words = [&](auto wrap_c, int at, double Sx, double Sy, double Sz, int (&u)[3]) {
    const double *const p = P + 3 * static_cast<int64_t>(at);
    const double x = p[0], y = p[1], z = p[2];
    if constexpr (decltype(wrap_c)::value) {
      auto whole = [](double v) {
        return static_cast<int>(fmin(fmax(v, -0x1p31), 0x1p31 - 1.0));
      };
      u[0] = whole(fma(z, h13, fma(y, h12, x * h11)));
      u[1] = whole(fma(z, h23, y * h22));
      u[2] = whole(z * h33);
    } else {
      u[0] = __float_as_int(static_cast<float>(x * len + Sx));
      u[1] = __float_as_int(static_cast<float>(y * len + Sy));
      u[2] = __float_as_int(static_cast<float>(z * len + Sz));
    }
  };
  // pairs for the canonical sequence, as the offsets of i from ib and j from jb
  LaneQueue queue;
  auto drain = [&](int word, int cnt) {
    const bool v = lane < cnt;
    const int64_t a = 3 * static_cast<int64_t>(index[v ? ib + (word & 511) : ib]);
    const int64_t b = 3 * static_cast<int64_t>(index[v ? jb + (word >> 9) : jb]);
    const double q0 =
        q64<kBoxTric>(in[a], in[a + 1], in[a + 2], in[b], in[b + 1], in[b + 2], geo);
    below += __builtin_popcountll(__builtin_amdgcn_ballot_w64(v && !(q0 >= qskip)));
  };
  for (int g = 0; g < gpu; ++g) {
    const int ja = jb + 64 * g, n = min(64, j1 - ja);
    auto bits = [&](uint64_t m) {
      return static_cast<uint32_t>(m >> (g * kUnitSlices)) & ((1u << kUnitSlices) - 1u);
    };
    if (bits(m_look) == 0u) continue;
    for (uint32_t m = bits(m_exact); m != 0u; m &= m - 1u) {
      const int i = ib + 64 * __builtin_ctz(m) + lane;
      for (int j = ja; j < ja + n; ++j)
        queue.push(i < i1 && (!diag_item || (i >> 6) != (ja >> 6) || j > i),
                   (i - ib) | (j - jb) << 9, drain);
    }
    // (mask_c: not all of the slices' and the group's pairs belong to the item)
    auto slices = [&](auto wrap_c, auto m_c, auto mask_c, uint32_t rs, const int (&uj)[3]) {
      constexpr int M = decltype(m_c)::value;
      constexpr bool WRAP = decltype(wrap_c)::value, MASK = decltype(mask_c)::value;
      const float far = WRAP ? unit : 1.f;
      const float q_lo = r_lo * far * (r_lo * far), q_hi = r_hi * far * (r_hi * far);
      int ui[M][3];
      [[maybe_unused]] int after[M];  // the lane's pairs are those with j from here on
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int r_k = static_cast<int>((rs >> (4 * k)) & 15u), at = g * kUnitSlices + r_k;
        const int i = ib + 64 * r_k + lane;
        words(wrap_c, i < i1 ? i : ib, lane_value(shx, at), lane_value(shy, at),
              lane_value(shz, at), ui[k]);
        after[k] = i >= i1 ? 64 : diag_item && (i >> 6) == (ja >> 6) ? lane + 1 : 0;
      }
      for (int j = 0; j < n; ++j) {
        const int ua = __builtin_amdgcn_readlane(uj[0], j), ub = __builtin_amdgcn_readlane(uj[1], j),
                  uc = __builtin_amdgcn_readlane(uj[2], j);
        int found = 0;
        uint64_t open[M], any = 0;
#pragma unroll
        for (int k = 0; k < M; ++k) {
          float dx, dy, dz;
          bool tie = false;
          if constexpr (WRAP) {
            auto diff = [](int a, int b) {
              return static_cast<float>(
                  static_cast<int>(static_cast<uint32_t>(a) - static_cast<uint32_t>(b)));
            };
            const float fa = diff(ua, ui[k][0]), fb = diff(ub, ui[k][1]), fc = diff(uc, ui[k][2]);
            dx = fmaf(g32.ncx, fc, fmaf(g32.nbx, fb, fa));
            dy = fmaf(g32.ncy, fc, g32.nby * fb);
            dz = g32.ncz * fc;
            tie = fmaxf(fabsf(fa), fmaxf(fabsf(fb), fabsf(fc))) > 0x1p31f * (1.f - 0x1p-21f);
            if constexpr (MASK) tie = tie && j >= after[k];
          } else {
            dx = __int_as_float(ua) - __int_as_float(ui[k][0]);
            dy = __int_as_float(ub) - __int_as_float(ui[k][1]);
            dz = __int_as_float(uc) - __int_as_float(ui[k][2]);
          }
          float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
          if constexpr (MASK) q = j >= after[k] ? q : __builtin_inff();
          const uint64_t in_lo = __builtin_amdgcn_ballot_w64(q < q_lo);
          open[k] = __builtin_amdgcn_ballot_w64(q < q_hi) ^ in_lo;
          if constexpr (WRAP) open[k] |= __builtin_amdgcn_ballot_w64(tie);
          any |= open[k];
          found += __builtin_popcountll(in_lo & ~open[k]);
        }
        below += found;
        if (__builtin_expect(any != 0, 0))
          for (int k = 0; k < M; ++k)
            queue.push((open[k] >> lane & 1u) != 0,
                       (64 * static_cast<int>((rs >> (4 * k)) & 15u) + lane) | (ja - jb + j) << 9,
                       drain);
      }
    };
    auto group = [&](auto wrap_c, uint32_t m) {
      if (m == 0u) return;
      int uj[3];  // lane l holds the group's point l
      words(wrap_c, ja + (lane < n ? lane : 0), 0.0, 0.0, 0.0, uj);
      using Yes = std::true_type;
      using No = std::false_type;
      // the group itself, and the slice at the end of the item, by themselves
      const int own = (ja - ib) >> 6, last = (i1 - ib) >> 6;
      uint32_t part = 0;
      if (diag_item && own >= 0 && own < kUnitSlices) part |= 1u << own;
      if (last < kUnitSlices && ((i1 - ib) & 63) != 0) part |= 1u << last;
      for (uint32_t b = m & part; b != 0u; b &= b - 1u)
        slices(wrap_c, Int<1>{}, Yes{}, static_cast<uint32_t>(__builtin_ctz(b)), uj);
      m &= ~part;
      while (__builtin_popcount(m) >= 4) {
        uint32_t rs = 0;
        for (int k = 0; k < 4; ++k) {
          rs |= static_cast<uint32_t>(__builtin_ctz(m)) << (4 * k);
          m &= m - 1u;
        }
        slices(wrap_c, Int<4>{}, No{}, rs, uj);
      }
      for (; m != 0u; m &= m - 1u)
        slices(wrap_c, Int<1>{}, No{}, static_cast<uint32_t>(__builtin_ctz(m)), uj);
    };
    group(std::false_type{}, bits(m_look & ~m_exact & ~m_wrap));
    group(std::true_type{}, bits(m_look & ~m_exact & m_wrap));
  }
  queue.finish(drain);
  return static_cast<uint64_t>(uni(sum) - uni(below));
}

// One work item of a spatially sorted binary64 frame. binary64 counts follow
// the canonical sequence bit for bit, but a pair's bin needs that sequence
// only when its distance lies next to a bin edge. The pairs here work on
// positions of the wrapped points relative to the cell centre, scaled to
// units in which a bin is 2^-22 wide, so with one shared shift per pair of
// groups a pair takes three differences and u = t^2 in binary64, and its bin
// from root_bits64. Here the threshold of the residuals bounds every rounding
// between the inputs and u and between the inputs and the canonical t; one
// ballot serves the pairs of two j, and when it fires the wave leaves them to
// settle_pairs (about one such group in 10^5 on the 1M-point frame).
//
// Bound by vector-unit issue: 15 instructions per pair on the short path (17
// with the clamp) against 22 over the frame with a binary64 root per pair
// (v_rsq_f64 alone holds a SIMD for 16 cycles, v_sqrt_f32 for 8). The
// 1,000,000-point clustered triclinic frame (20,000 bins) took 371 ms with
// every pair computed and that root, 178 ms in Morton order, and takes 162 ms;
// 100,000 points in a cube (cut-off half the edge, so little is skipped) 4.34,
// 3.49 and 2.87 ms.
template <int MODE, bool SEARCH>
__device__ __forceinline__ void run_sorted64(const PairKernelArgs &a, const WorkItem &w,
                                             const FrameParams *F, int *s_unit, int *s_item,
                                             unsigned long long *s_search) {
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const char *const staged = uni(static_cast<const char *>(F->coords));
  const int64_t n_pad = uni(static_cast<int>(F->n_pad));
  const double *const P = reinterpret_cast<const double *>(staged);
  const GroupBox *const boxes = reinterpret_cast<const GroupBox *>(staged + 28 * n_pad);
  float cell[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) cell[k] = uni(F->cell32[k]);
  // cell rows in scaled units, entries of B^-1 per scaled unit
  const double s = uni(F->s) * 0x1p-22, is = 1.0 / s;
  const double ax = uni(F->ax) * s, bx = uni(F->bx) * s, by = uni(F->by) * s;
  const double cx = uni(F->cx) * s, cy = uni(F->cy) * s, cz = uni(F->cz) * s;
  const double h11 = uni(F->h11) * is, h12 = uni(F->h12) * is, h13 = uni(F->h13) * is;
  const double h22 = uni(F->h22) * is, h23 = uni(F->h23) * is, h33 = uni(F->h33) * is;
  const int win = uni(F->win);
  const WindowBounds wb = window_bounds(F, w.sweep * win, win, a.stride);
  const bool noclamp = MODE == kModeLds && !SEARCH && uni(F->noclamp) != 0;
  const Count<MODE> count(F, w, lane);
  using Yes = std::true_type;
  using No = std::false_type;

  int ib = 0, jb = 0;
  GroupPair gp;
  double shx = 0.0, shy = 0.0, shz = 0.0;  // the lane's shift B n
  float near_hi = 0.f;  // thr's upper word, as a float (see below)
  [[maybe_unused]] Images img{};
  // image search: pairs it is defined for (see searched_pairs; counted in the
  // first bin window), and the images evaluated
  [[maybe_unused]] uint64_t n_searched = 0, n_images = 0;
  [[maybe_unused]] const bool tell = SEARCH && F->searched != nullptr && w.sweep == 0;

  auto frac = [&](auto axis_c, double x, double y, double z) {
    constexpr int K = decltype(axis_c)::value;
    if constexpr (K == 0)
      return fma(z, h13, fma(y, h12, x * h11));
    else if constexpr (K == 1)
      return fma(z, h23, y * h22);
    else
      return z * h33;
  };
  // One group against M slices (four bits each in rs) of one kind.
  // IMAGES: shifts tried per pair (1 without image search, whose shift is gp's).
  auto pass = [&](auto kind_c, auto images_c, auto m_c, auto clamp_c, auto diag_c, uint32_t rs,
                  int g) {
    constexpr int KIND = decltype(kind_c)::value, M = decltype(m_c)::value;
    constexpr int IMAGES = decltype(images_c)::value;
    constexpr bool DIAG = decltype(diag_c)::value;
    const int j0 = jb + 64 * g, j1 = min(j0 + 64, w.j1);
    auto slice = [&](int k) { return ib + 64 * static_cast<int>((rs >> (4 * k)) & 15u) + lane; };
    // j pairs (bit b: j0 + 2b and the next) left to the canonical sequence
    uint32_t left = 0;
    if constexpr (KIND == kExact) {
      left = ~0u;
    } else {
      // (a lane past the end of the item holds a point at infinity: q = +inf,
      // beyond every bin)
      double sx[M * IMAGES], sy[M * IMAGES], sz[M * IMAGES];
      [[maybe_unused]] double fi[3][M];
      constexpr int K = KIND >= kFix && KIND < kSlow ? KIND - kFix : 0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int i = slice(k);
        const bool ok = i < w.i1;
        const double *const p = P + 3 * static_cast<int64_t>(ok ? i : ib);
        const int src = g * kUnitSlices + static_cast<int>((rs >> (4 * k)) & 15u);
        if constexpr (SEARCH) {
          const uint32_t lo = static_cast<uint32_t>(
              __builtin_amdgcn_readlane(static_cast<int>(img.list), src));
          const uint32_t hi = static_cast<uint32_t>(
              __builtin_amdgcn_readlane(static_cast<int>(img.list >> 32), src));
          const int n = __builtin_amdgcn_readlane(img.n, src);
#pragma unroll
          for (int e = 0; e < IMAGES; ++e) {
            // (a list shorter than IMAGES repeats its first entry)
            const int at = e < n ? e : 0;
            const int id = static_cast<int>((at < 4 ? lo >> (8 * at) : hi >> (8 * at - 32)) & 255u);
            const double na = id % 5 - 2, nb = id / 5 % 5 - 2, nc = id / 25 - 2;
            sx[k * IMAGES + e] = (ok ? p[0] : __builtin_inf()) + ((na * ax + nb * bx) + nc * cx);
            sy[k * IMAGES + e] = p[1] + (nb * by + nc * cy);
            sz[k * IMAGES + e] = p[2] + nc * cz;
          }
          continue;
        }
        sx[k] = p[0] + lane_value(shx, src);
        sy[k] = p[1] + lane_value(shy, src);
        sz[k] = p[2] + lane_value(shz, src);
        if constexpr (KIND == kSlow) {
          fi[0][k] = frac(Int<0>{}, sx[k], sy[k], sz[k]);
          fi[1][k] = frac(Int<1>{}, sx[k], sy[k], sz[k]);
          fi[2][k] = frac(Int<2>{}, sx[k], sy[k], sz[k]);
        } else if constexpr (KIND >= kFix) {
          fi[0][k] = frac(Int<K>{}, sx[k], sy[k], sz[k]);
        }
        sx[k] = ok ? sx[k] : __builtin_inf();
      }
      struct J {
        double x, y, z;
      };
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<double *>(P + 3 * static_cast<int64_t>(j0)), 0, (j1 - j0) * 24,
          kBufferFlags);
      int at = 0;
      auto load = [&](int k) {
        union {
          struct {
            V4u a;
            V2u b;
          } w;
          J j;
        } e;
        e.w.a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 24 * k, at, 0);
        e.w.b = __builtin_amdgcn_raw_buffer_load_b64(rsrc, 24 * k + 16, at, 0);
        return e.j;
      };
      // bin bits and the smallest |residual| of the pairs of one j
      auto bits_of = [&](const J &p, int j, uint32_t *b, float &gap) {
        [[maybe_unused]] double fj[3];
        if constexpr (KIND == kSlow) {
          fj[0] = frac(Int<0>{}, p.x, p.y, p.z);
          fj[1] = frac(Int<1>{}, p.x, p.y, p.z);
          fj[2] = frac(Int<2>{}, p.x, p.y, p.z);
        } else if constexpr (KIND >= kFix) {
          fj[0] = frac(Int<K>{}, p.x, p.y, p.z);
        }
#pragma unroll
        for (int k = 0; k < M; ++k) {
          if constexpr (SEARCH) {
            double u = 0.0;
#pragma unroll
            for (int e = 0; e < IMAGES; ++e) {
              const double dx = p.x - sx[k * IMAGES + e], dy = p.y - sy[k * IMAGES + e],
                           dz = p.z - sz[k * IMAGES + e];
              const double v = fma(dz, dz, fma(dy, dy, dx * dx));
              u = e == 0 ? v : min_arith(u, v);
            }
            if constexpr (DIAG) u = j <= slice(k) ? kFarU : u;
            b[k] = root_bits64(u, gap);
            continue;
          }
          double dx = p.x - sx[k], dy = p.y - sy[k], dz = p.z - sz[k];
          if constexpr (KIND == kSlow) {
            const double na = rint(fj[0] - fi[0][k]), nb = rint(fj[1] - fi[1][k]),
                         nc = rint(fj[2] - fi[2][k]);
            dz = fma(-cz, nc, dz);
            dy = fma(-cy, nc, fma(-by, nb, dy));
            dx = fma(-cx, nc, fma(-bx, nb, fma(-ax, na, dx)));
          } else if constexpr (KIND >= kFix) {
            const double n = rint(fj[0] - fi[0][k]);
            if constexpr (K == 2) dz = fma(-cz, n, dz);
            if constexpr (K >= 1) dy = fma(K == 1 ? -by : -cy, n, dy);
            dx = fma(K == 0 ? -ax : K == 1 ? -bx : -cx, n, dx);
          }
          double u = fma(dz, dz, fma(dy, dy, dx * dx));
          if constexpr (DIAG) u = j <= slice(k) ? kFarU : u;
          b[k] = root_bits64(u, gap);
        }
      };
      auto tally = [&](const uint32_t *b, int j) {
#pragma unroll
        for (int k = 0; k < M; ++k)
          count.template add<decltype(clamp_c)::value>(
              DIAG && j <= slice(k) ? kNoBits : b[k]);
      };
      J pa = load(0), pb = load(1);
      int j = j0, je = j1;
      for (; j + 1 < je; j += 2) {
        at += 48;
        uint32_t b[2 * M];
        float gap = __builtin_inff();
        bits_of(pa, j, b, gap);
        pa = load(0);
        bits_of(pb, j + 1, b + M, gap);
        pb = load(1);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(gap <= near_hi) != 0, 0)) {
          left |= 1u << ((j - j0) >> 1);
          // (all of the first eight j: distances repeat at bin edges here)
          if (left == 15u) {
            left = ~0u;
            je = j0;
          }
          continue;
        }
        tally(b, j);
        tally(b + M, j + 1);
      }
      if (j < je) {
        uint32_t b[M];
        float gap = __builtin_inff();
        bits_of(pa, j, b, gap);
        if (__builtin_amdgcn_ballot_w64(gap <= near_hi) != 0)
          left |= 1u << ((j - j0) >> 1);
        else
          tally(b, j);
      }
    }
    if (__builtin_expect(left != 0u, 0))
      settle_pairs<MODE, SEARCH>(F, w, ib, j0, j1, rs, M, left,
                                 (DIAG ? kSettleDiag : 0) | (KIND == kExact ? kSettleExact : 0) |
                                     (KIND == kFast ? kSettleFast : 0),
                                 g * kUnitSlices, near_hi, shx, shy, shz, img);
    if constexpr (SEARCH && IMAGES != 1) {
      const uint64_t n = static_cast<uint64_t>(j1 - j0);
      uint64_t pairs = DIAG ? n * (n - 1) / 2 : 0;
      for (int k = 0; k < M && !DIAG; ++k)
        pairs += n * static_cast<uint64_t>(max(0, min(64, w.i1 - (slice(k) - lane))));
      n_images += pairs * (KIND == kExact ? kShifts : IMAGES);
    }
  };
  // the slices in `m` (bit r) against group g, in passes of as many as fit
  auto passes = [&](auto kind_c, auto images_c, auto clamp_c, uint32_t m, int g) {
    constexpr int IMAGES = decltype(images_c)::value;
    auto take = [&](int n) {
      uint32_t rs = 0;
      for (int k = 0; k < n; ++k) {
        rs |= static_cast<uint32_t>(__builtin_ctz(m)) << (4 * k);
        m &= m - 1u;
      }
      return rs;
    };
    if constexpr (IMAGES == 1)
      while (__builtin_popcount(m) >= 4)
        pass(kind_c, images_c, Int<4>{}, clamp_c, No{}, take(4), g);
    if constexpr (IMAGES <= 2)
      while (__builtin_popcount(m) >= 2)
        pass(kind_c, images_c, Int<2>{}, clamp_c, No{}, take(2), g);
    while (m != 0u) pass(kind_c, images_c, Int<1>{}, clamp_c, No{}, take(1), g);
  };

  const int n_ib = (w.i1 - w.i0 + kUnitPoints - 1) / kUnitPoints;
  const int n_wave = static_cast<int>(blockDim.x) / 64;
  int gpu = kUnitGroups;
  while (gpu > 1 && n_ib * ((w.j1 - w.j0 + 64 * gpu - 1) / (64 * gpu)) < (SEARCH ? 2 : 4) * n_wave)
    gpu >>= 1;
  const int n_unit = n_ib * ((w.j1 - w.j0 + 64 * gpu - 1) / (64 * gpu));
  if (wave == n_unit && lane == 0)
    *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  for (int u = wave; u < n_unit;) {
    ib = w.i0 + (u % n_ib) * kUnitPoints;
    jb = w.j0 + (u / n_ib) * 64 * gpu;
    {
      const int r = lane % kUnitSlices, gr = lane / kUnitSlices;
      const int gi = (ib >> 6) + r, gj = (jb >> 6) + gr;
      const bool valid = ib + 64 * r < w.i1 && gr < gpu && jb + 64 * gr < w.j1 &&
                         !((w.flags & kItemDiag) && gj < gi);
      const GroupBox &bi = boxes[valid ? gi : ib >> 6], &bj = boxes[valid ? gj : jb >> 6];
      if constexpr (SEARCH) {
        if (tell) n_searched += searched_pairs(F, w, ib, jb, gpu);
        img = group_images(bi, bj, cell, wb.hi, wb.slack);
        gp.kind = img.n == 0 || img.far2 < wb.lo * wb.lo ? kSkip
                  : img.n == 1                           ? kFast
                  : img.n == 2                           ? kFix
                  : img.n <= 4                           ? kFix + 1
                  : img.n <= kListed                     ? kFix + 2
                                                         : kExact;
        // (the nearest image's shift is in the list when it is within the window)
        gp.in_window = img.far2 < fminf(wb.in * wb.in, wb.hi * wb.hi);
        gp.n[0] = gp.n[1] = gp.n[2] = 0;
      } else {
        gp = classify<true>(bi, bj, cell, wb.lo, wb.hi, wb.in);
      }
      shx = (gp.n[0] * ax + gp.n[1] * bx) + gp.n[2] * cx;
      shy = gp.n[1] * by + gp.n[2] * cy;
      shz = gp.n[2] * cz;
      // A residual is off by at most 2 t dt + 2^-48 t^2, t <= n_bins + 2
      // (beyond that the pair is out of range either way).
      double dt;
      const double top = static_cast<double>(count.n_bins + 2u) * 0x1p-22;
      const double hm = fmax(fmax(fabs(h11), fabs(h12)), fmax(fmax(fabs(h13), fabs(h22)),
                                                              fmax(fabs(h23), fabs(h33)))) * s;
      const bool bounded = rounding_bound(bi, bj, cell, s, hm, dt);
      if (!bounded) {
        gp.kind = kExact;
        gp.in_window = false;
      }
      gp.diag = (w.flags & kItemDiag) && gj == gi;
      gp.in_window = (gp.in_window || (noclamp && bounded)) && ib + 64 * r + 64 <= w.i1;
      if (!valid) gp.kind = kSkip;
      // the unit's largest threshold, as the upper word of a binary64 number
      // read as a float (monotone for non-negative numbers), rounded up
      double thr = gp.kind == kSkip || gp.kind == kExact ? 0.0 : 2.0 * top * dt + 0x1p-48 * top * top;
      for (int o = 32; o > 0; o >>= 1) thr = fmax(thr, __shfl_xor(thr, o));
      near_hi = uni(__int_as_float(static_cast<int>(__double_as_longlong(thr) >> 32) + 1));
    }
    const uint64_t m_fast = __builtin_amdgcn_ballot_w64(gp.kind == kFast && !gp.diag);
    const uint64_t m_in = __builtin_amdgcn_ballot_w64(gp.in_window);
    const uint64_t m_fix0 = __builtin_amdgcn_ballot_w64(gp.kind == kFix && !gp.diag);
    const uint64_t m_fix1 = __builtin_amdgcn_ballot_w64(gp.kind == kFix + 1 && !gp.diag);
    const uint64_t m_fix2 = __builtin_amdgcn_ballot_w64(gp.kind == kFix + 2 && !gp.diag);
    const uint64_t m_slow = __builtin_amdgcn_ballot_w64(gp.kind == kSlow && !gp.diag);
    const uint64_t m_exact = __builtin_amdgcn_ballot_w64(gp.kind == kExact && !gp.diag);
    const uint64_t m_diag = __builtin_amdgcn_ballot_w64(gp.kind != kSkip && gp.diag);
    for (int g = 0; g < gpu; ++g) {
      auto bits = [&](uint64_t m) {
        return static_cast<uint32_t>(m >> (g * kUnitSlices)) & ((1u << kUnitSlices) - 1u);
      };
      const uint32_t fast = bits(m_fast);
      const bool inside = MODE == kModeLds && (fast & ~bits(m_in)) == 0u;
      if (inside)
        passes(Int<kFast>{}, Int<1>{}, No{}, fast, g);
      else
        passes(Int<kFast>{}, Int<1>{}, Yes{}, fast, g);
      if constexpr (SEARCH) {
        passes(Int<kFast>{}, Int<2>{}, Yes{}, bits(m_fix0), g);
        passes(Int<kFast>{}, Int<4>{}, Yes{}, bits(m_fix1), g);
        passes(Int<kFast>{}, Int<kListed>{}, Yes{}, bits(m_fix2), g);
      } else {
        passes(Int<kFix>{}, Int<1>{}, Yes{}, bits(m_fix0), g);
        passes(Int<kFix + 1>{}, Int<1>{}, Yes{}, bits(m_fix1), g);
        passes(Int<kFix + 2>{}, Int<1>{}, Yes{}, bits(m_fix2), g);
        passes(Int<kSlow>{}, Int<1>{}, Yes{}, bits(m_slow), g);
      }
      for (uint32_t m = bits(m_exact); m != 0u; m &= m - 1u)
        pass(Int<kExact>{}, Int<0>{}, Int<1>{}, Yes{}, No{},
             static_cast<uint32_t>(__builtin_ctz(m)), g);
      if (const uint32_t m = bits(m_diag)) {
        // at most one slice of the unit is the group itself
        const uint32_t r = static_cast<uint32_t>(__builtin_ctz(m));
        const int kind = __builtin_amdgcn_readlane(gp.kind, g * kUnitSlices + static_cast<int>(r));
        if (kind == kFast)
          pass(Int<kFast>{}, Int<1>{}, Int<1>{}, Yes{}, Yes{}, r, g);
        else if (kind == kExact)
          pass(Int<kExact>{}, Int<0>{}, Int<1>{}, Yes{}, Yes{}, r, g);
        else if constexpr (SEARCH)
          pass(Int<kFast>{}, Int<kListed>{}, Int<1>{}, Yes{}, Yes{}, r, g);
        else
          pass(Int<kSlow>{}, Int<1>{}, Int<1>{}, Yes{}, Yes{}, r, g);
      }
    }
    int nu = 0;
    if (lane == 0) nu = atomicAdd(s_unit, 1);
    u = uni(nu);
    if (u == n_unit && lane == 0)
      *s_item = static_cast<int>(gridDim.x) + atomicAdd(a.counter, 1);
  }
  if constexpr (SEARCH) {
    // (the unsorted search counts them in every bin window, and once where it
    // takes one pass of atomics instead)
    const int windows = uni(F->n_sweeps);
    add_searched(s_search, lane,
                 n_searched * static_cast<uint64_t>(windows < kWideDefault64 ? windows : 1),
                 n_images);
  }
}

}  // namespace
}  // namespace dh
