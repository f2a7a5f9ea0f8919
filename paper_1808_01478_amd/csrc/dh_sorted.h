// The pair kernel's work on spatially sorted frames (kBoxTricSorted).
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
// takes 90 ms.
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

template <int N>
using Int = std::integral_constant<int, N>;

// What the boxes of slice r and group g of a unit say about all their pairs
// (the lane's own pair; see run_sorted).
struct GroupPair {
  int kind;        // kFast, kFix + axis, kSlow, or kSkip
  bool diag;       // the same group: pairs j > i only
  bool in_window;  // every t below the LDS stride (no clamp needed)
  float sx, sy, sz;  // lattice shift B n of the lower-end wraps
};
constexpr int kSkip = 0, kFast = 1, kFix = 2, kSlow = 5;  // kFix + axis: 2, 3, 4

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
__device__ __forceinline__ GroupPair classify(const GroupBox &I, const GroupBox &J,
                                              const float (&cell)[6], float r_lo, float r_hi,
                                              float r_in) {
  GroupPair p;
  int nl[3], nh[3];
  uint32_t amb = 0;
  bool wide = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    nl[k] = static_cast<int>(J.ulo[k] - I.uhi[k] >= 0x80000000u) -
            static_cast<int>(J.ulo[k] < I.uhi[k]);
    nh[k] = static_cast<int>(J.uhi[k] - I.ulo[k] >= 0x80000000u) -
            static_cast<int>(J.uhi[k] < I.ulo[k]);
    amb |= nl[k] != nh[k] ? 1u << k : 0u;
    wide = wide || nh[k] - nl[k] > 1;
  }
  p.kind = amb == 0u ? kFast
                     : ((amb & (amb - 1u)) == 0u && !wide ? kFix + (amb == 1u ? 0 : amb == 2u ? 1 : 2)
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
  shift(nl[0], nl[1], nl[2], p.sx, p.sy, p.sz);
  return p;
}

// Distance bounds of a bin window in length units, widened by far more than
// the rounding of any pair's distance: a pair outside [lo, hi] cannot count,
// one inside `in` needs no clamp (its t is below the LDS stride; slots past
// the window are never flushed).
struct WindowBounds {
  float lo, hi, in;
};
__device__ __forceinline__ WindowBounds window_bounds(const FrameParams *F, int b_lo, int win,
                                                      int stride) {
  float size = 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) size += fabsf(uni(F->cell32[k]));
  const float eps = size * 0x1p-16f, s = uni(F->s32);
  WindowBounds b;
  b.lo = b_lo > 0 ? fmaxf(static_cast<float>(b_lo) / s * (1.f - 0x1p-12f) - eps, 0.f) : 0.f;
  b.hi = static_cast<float>(b_lo + win) / s * (1.f + 0x1p-12f) + eps;
  b.in = fmaxf(static_cast<float>(stride - 2) / s * (1.f - 0x1p-12f) - eps, 0.f);
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
  const Count32<MODE> count(F, w, lane);
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
    const void *first = decltype(words_c)::value ? static_cast<const void *>(W + 3 * j0)
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
      static_assert(M == 1, "fixed-point passes take one slice");
      // -(b:a) of the i-point and -(c':c), c' the c of the point 64 before an
      // odd slice's (one 64-bit addition to j's (c:c) gives both c
      // differences, an odd slice's lowered by one unit when the even one
      // borrows, as in unsorted frames)
      const int r = static_cast<int>(rs & 15u);
      const int i = ib + 64 * r + lane;
      const bool ok = i < w.i1;
      const int ic = ok ? i : ib;
      const uint32_t za = W[3 * ic + 2];
      const uint32_t zb = r & 1 ? W[3 * (ok ? i - 64 : ib) + 2] : 0u;
      const uint64_t nab =
          0ull - ((static_cast<uint64_t>(W[3 * ic + 1]) << 32) | W[3 * ic]);
      const uint64_t nzz = r & 1 ? 0ull - ((static_cast<uint64_t>(za) << 32) | zb)
                                 : 0ull - static_cast<uint64_t>(za);
      const bool odd = (r & 1) != 0;
      run_j(Int<4>{}, Yes{}, j0, [&](const float4 &e, int j) {
        const uint64_t ab =
            (static_cast<uint64_t>(__float_as_uint(e.y)) << 32) | __float_as_uint(e.x);
        const uint64_t cc =
            (static_cast<uint64_t>(__float_as_uint(e.z)) << 32) | __float_as_uint(e.z);
        const uint64_t dcc = cc + nzz;
        const float fc = static_cast<float>(
            static_cast<int32_t>(static_cast<uint32_t>(odd ? dcc >> 32 : dcc)));
        count.template add<true>(bits32_packed_c<kBoxTric>(
            ab, nab, fc, g32, ok && (!DIAG || j > i) ? kBinOffset : kNoBin));
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
      gp = classify(boxes[valid ? gi : ib >> 6], boxes[valid ? gj : jb >> 6], cell, wb.lo, wb.hi,
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
      for (uint32_t m = bits(m_slow); m != 0u; m &= m - 1u)
        pass(Int<kSlow>{}, Int<1>{}, Yes{}, No{}, static_cast<uint32_t>(__builtin_ctz(m)), g);
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

}  // namespace
}  // namespace dh
