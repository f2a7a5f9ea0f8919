// gfx950 kernels of libdisthist around the pair kernel (dh_pairs.h): staging,
// output zeroing, out-of-range counts and the per-pair probe, with the
// launchers of all of them.
#include "dh_pairs.h"

namespace dh {
namespace {

// --------------------------------------------------------------------------
// Staging: binary64 [N][3] -> padded float4 / double4
// --------------------------------------------------------------------------

// The share of one thread of a grid in clearing a call's output (see ZeroArgs).
__device__ __forceinline__ void zero_part(const ZeroArgs &z) {
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  for (int64_t i = i0; i < z.n_counters; i += step) z.counters[i] = 0;
  if (z.oor)
    for (int64_t i = i0; i < z.n_hist; i += step) z.oor[i] = z.pairs[i];
  for (int64_t i = i0; i < z.n_words; i += step) z.out[i] = 0ull;
}

// Unsorted frames are staged and their output cleared by one launch: a small
// frame is a chain of launches, about 2.5 us of host time and a gap on the
// device each (1,000 points, binary32: 21.6 us a call with two launches, 16.1 us
// with one and no image lists for frames without a search).
__global__ void stage64_kernel(const double *__restrict__ in, double4 *__restrict__ out,
                               int64_t n, ZeroArgs z) {
  zero_part(z);
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += step)
    out[i] = make_double4(in[3 * i], in[3 * i + 1], in[3 * i + 2], 0.0);
}

// 32-bit fixed-point image of a fractional coordinate: floor(2^32 * (f mod 1))
__device__ __forceinline__ float fixfrac(double f) {
  const double w = f - floor(f);
  const uint64_t u = static_cast<uint64_t>(w * 4294967296.0);
  return __uint_as_float(static_cast<uint32_t>(u));
}

// One staged binary32 point (see FrameParams for the formats).
template <int BOX>
__device__ __forceinline__ float4 stage_point32(double x, double y, double z,
                                                const FrameParams &p) {
  if constexpr (BOX == kBoxNone) {
    return make_float4(static_cast<float>(x * p.s), static_cast<float>(y * p.s),
                       static_cast<float>(z * p.s), 0.f);
  } else if constexpr (BOX == kBoxOrtho) {
    // c twice: the pair kernel reads (c : c) as one 64-bit word
    const float c = fixfrac(z * p.iL[2]);
    return make_float4(fixfrac(x * p.iL[0]), fixfrac(y * p.iL[1]), c, c);
  } else {
    const double fa = fma(z, p.h13, fma(y, p.h12, x * p.h11));
    const double fb = fma(z, p.h23, y * p.h22);
    const double fc = z * p.h33;
    const float c = fixfrac(fc);
    return make_float4(fixfrac(fa), fixfrac(fb), c, c);
  }
}

template <int BOX>
__global__ void stage32_kernel(const double *__restrict__ in, float4 *__restrict__ out, int64_t n,
                               FrameParams p, ZeroArgs z) {
  zero_part(z);
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += step)
    out[i] = stage_point32<BOX>(in[3 * i], in[3 * i + 1], in[3 * i + 2], p);
}

// --------------------------------------------------------------------------
// Spatially sorted staging
// --------------------------------------------------------------------------
//
// The points of every species are put in the order of a Morton curve over
// their wrapped fractional coordinates (9 bits per axis), ties by input
// index, so that 64 consecutive points are close together in the cell. The
// pair kernel then finds, for most pairs of such groups, one lattice shift
// that is the Eq. 5 wrap of every pair of the two groups (see run_sorted), or
// that all their pairs are out of range. Binary64 frames are put into tighter
// groups still (see refine_order_kernel).
// The order is a permutation within each species, so the histograms are
// those of the input; the sort is a bitonic network on 64-bit keys
// (species : Morton code : input index), which makes the order unique.

struct SpeciesOffsets {
  int64_t v[kMaxSpeciesStage + 1];
};

// Morton code of three 9-bit integers: bit b of axis a goes to bit 3b + a.
__device__ __forceinline__ uint64_t morton9(uint32_t a, uint32_t b, uint32_t c) {
  uint64_t m = 0;
#pragma unroll
  for (int bit = 0; bit < 9; ++bit)
    m |= (static_cast<uint64_t>((a >> bit) & 1u) << (3 * bit)) |
         (static_cast<uint64_t>((b >> bit) & 1u) << (3 * bit + 1)) |
         (static_cast<uint64_t>((c >> bit) & 1u) << (3 * bit + 2));
  return m;
}

// wrapped fractional coordinate as 32-bit fixed point (as fixfrac)
__device__ __forceinline__ uint32_t fix32(double f) {
  const double w = f - floor(f);
  return static_cast<uint32_t>(static_cast<uint64_t>(w * 4294967296.0));
}

__global__ void sort_keys_kernel(const double *__restrict__ in, int64_t n, int64_t npad,
                                 SpeciesOffsets off, int32_t k, FrameParams p,
                                 uint64_t *__restrict__ keys) {
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < npad;
       i += step) {
    if (i >= n) {
      keys[i] = ~0ull;
      continue;
    }
    int s = 0;
    while (s + 1 < k && off.v[s + 1] <= i) ++s;
    const double x = in[3 * i], y = in[3 * i + 1], z = in[3 * i + 2];
    const uint32_t ua = fix32(fma(z, p.h13, fma(y, p.h12, x * p.h11)));
    const uint32_t ub = fix32(fma(z, p.h23, y * p.h22));
    const uint32_t uc = fix32(z * p.h33);
    const uint64_t m = morton9(ua >> 23, ub >> 23, uc >> 23);
    keys[i] = (static_cast<uint64_t>(s) << 58) | (m << 31) | static_cast<uint64_t>(i);
  }
}

constexpr int kBitonicBlock = 8192;  // keys sorted in LDS by one workgroup of 1024

template <typename K>
__device__ __forceinline__ void bitonic_cas(K &a, K &b, bool ascending) {
  if ((a > b) == ascending) {
    const K t = a;
    a = b;
    b = t;
  }
}

// Index of the lower element of compare-exchange t of a step j (a power of
// two): t with a zero inserted at the bit of j.
__device__ __forceinline__ int cas_index(int t, int j) {
  return ((t & ~(j - 1)) << 1) | (t & (j - 1));
}

// The step j of stage kk on a block of keys in LDS (1,024 threads). The 128
// elements of a wave's 64 exchanges are the same in every step below 128, so
// only steps of 64 and more need a barrier; the others need the wave's own LDS
// order, which the hardware keeps.
__device__ __forceinline__ void bitonic_step(uint64_t *key, int j, int64_t kk, int64_t base) {
  if (j >= 64)
    __syncthreads();
  else
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int t = threadIdx.x; t < kBitonicBlock / 2; t += 1024) {
    const int at = cas_index(t, j);
    bitonic_cas(key[at], key[at + j], ((base + at) & kk) == 0);
  }
}

// (The whole sort of 100,000 points, 131,072 keys: 5 launches here at 22 us and
// 6 over the whole array at 5 us. With blocks of 2,048 keys, divisions for the
// index, a barrier per step and one step per global launch there were 7 and 21
// launches.)
// All stages k <= kBitonicBlock of each block (first == true), or the steps
// j < kBitonicBlock of stage k (first == false), in LDS.
__global__ __launch_bounds__(1024) void bitonic_local_kernel(uint64_t *__restrict__ keys,
                                                             int64_t k_stage, int first) {
  __shared__ uint64_t sk[kBitonicBlock];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kBitonicBlock;
  for (int t = threadIdx.x; t < kBitonicBlock; t += 1024) sk[t] = keys[base + t];
  __syncthreads();
  const int64_t k_lo = first ? 2 : k_stage, k_hi = first ? kBitonicBlock : k_stage;
  for (int64_t kk = k_lo; kk <= k_hi; kk <<= 1)
    for (int j = kk / 2 < kBitonicBlock / 2 ? static_cast<int>(kk / 2) : kBitonicBlock / 2;
         j > 0; j >>= 1)
      bitonic_step(sk, j, kk, base);
  __syncthreads();
  for (int t = threadIdx.x; t < kBitonicBlock; t += 1024) keys[base + t] = sk[t];
}

// The step j >= kBitonicBlock of stage k over the whole array, with TWO the
// step j / 2 as well (half the passes over memory and half the launches).
template <bool TWO>
__global__ void bitonic_global_kernel(uint64_t *__restrict__ keys, int64_t npad, int64_t j,
                                      int64_t k_stage) {
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t h = TWO ? j / 2 : j;
  for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
       t < npad / (TWO ? 4 : 2); t += step) {
    const int64_t at = ((t & ~(h - 1)) << (TWO ? 2 : 1)) | (t & (h - 1));
    const bool asc = (at & k_stage) == 0;
    if constexpr (TWO) {
      uint64_t a = keys[at], b = keys[at + h], c = keys[at + j], e = keys[at + j + h];
      bitonic_cas(a, c, asc);
      bitonic_cas(b, e, asc);
      bitonic_cas(a, b, asc);
      bitonic_cas(c, e, asc);
      keys[at] = a;
      keys[at + h] = b;
      keys[at + j] = c;
      keys[at + j + h] = e;
    } else {
      uint64_t a = keys[at], b = keys[at + j];
      bitonic_cas(a, b, asc);
      keys[at] = a;
      keys[at + j] = b;
    }
  }
}

// Minimum and maximum over the 64 lanes of a wave.
template <typename V>
__device__ __forceinline__ V wave_min(V v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
template <typename V>
__device__ __forceinline__ V wave_max(V v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

// binary32 staging of a sorted frame at padded indices (see padded_frame),
// one group of 64 points per wave: the fixed-point fractional words as for
// unsorted triclinic frames, the Cartesian position of the same wrapped point
// relative to the cell centre, B (u - 1/2) with u the fixed-point fraction
// read back exactly, so the two formats describe one point, and the group's
// boxes.
__global__ void stage_sorted_kernel(const double *__restrict__ in,
                                    const uint64_t *__restrict__ keys, SpeciesOffsets off,
                                    int32_t k, FrameParams p, char *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t group = blockIdx.x * static_cast<int64_t>(blockDim.x / 64) + threadIdx.x / 64;
  if (64 * group >= p.n_pad) return;
  int64_t g0 = 0;
  int s = 0;
  for (; s + 1 < k; ++s) {
    const int64_t ng = (off.v[s + 1] - off.v[s] + 63) / 64;
    if (group < g0 + ng) break;
    g0 += ng;
  }
  const int64_t q = off.v[s] + 64 * (group - g0) + lane;
  const bool ok = q < off.v[s + 1];
  uint32_t u[3] = {0u, 0u, 0u};
  float c[3] = {0.f, 0.f, 0.f};
  if (ok) {
    const int64_t i = static_cast<int64_t>(keys[q] & 0x7FFFFFFFull);
    const double x = in[3 * i], y = in[3 * i + 1], z = in[3 * i + 2];
    u[0] = fix32(fma(z, p.h13, fma(y, p.h12, x * p.h11)));
    u[1] = fix32(fma(z, p.h23, y * p.h22));
    u[2] = fix32(z * p.h33);
    const double va = u[0] * 0x1p-32 - 0.5, vb = u[1] * 0x1p-32 - 0.5, vc = u[2] * 0x1p-32 - 0.5;
    c[0] = static_cast<float>(fma(p.cx, vc, fma(p.bx, vb, p.ax * va)));
    c[1] = static_cast<float>(fma(p.cy, vc, p.by * vb));
    c[2] = static_cast<float>(p.cz * vc);
  }
  const int64_t at = 64 * group + lane;
  reinterpret_cast<float4 *>(out)[at] = make_float4(c[0], c[1], c[2], 0.f);
  uint32_t *const words = reinterpret_cast<uint32_t *>(out + 16 * static_cast<int64_t>(p.n_pad)) + 3 * at;
  GroupBox b;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    words[ax] = u[ax];
    b.ulo[ax] = wave_min(ok ? u[ax] : 0xFFFFFFFFu);
    b.uhi[ax] = wave_max(ok ? u[ax] : 0u);
    b.clo[ax] = wave_min(ok ? c[ax] : __builtin_inff());
    b.chi[ax] = wave_max(ok ? c[ax] : -__builtin_inff());
  }
  b.mag = 0.f;
  for (uint32_t &v : b.unused) v = 0u;
  if (lane == 0) reinterpret_cast<GroupBox *>(out + 28 * static_cast<int64_t>(p.n_pad))[group] = b;
}

// Morton order alone leaves loose groups: 64 consecutive points straddle the
// curve's jumps (mean box 8.3 x 6.2 x 4.6 where 64 points fill a cube of 4.5),
// and everything decided per pair of groups weakens with that. So each run of
// kRefine points of the curve is halved six times, along the axis in which its
// points spread most, down to the groups of 64 (mean box 4.7 x 4.7 x 4.5).
// Binary64 against the Morton order alone: 1,000,000 clustered triclinic points
// 176 and 160 ms, image search of 70,001 points 7.33 and 4.20 ms.
//
// One workgroup per run: 16-bit fractional coordinates in LDS, a 32-bit key
// (coordinate : place in the run) per point, four consecutive keys per thread
// in registers. A level sorts its segments by the bitonic network (308 steps
// in all): steps of 1 and 2 stay in a thread, those up to 128 in a wave
// (shuffles), only the 20 wider ones go through LDS with a barrier (100,000
// points: 141 us a launch with all steps in LDS, 99 us so). Runs of 2,048 are
// quicker to halve and worse (66 us; image search of 70,001 points 5.0 against
// 4.2 ms).
constexpr int kRefine = 4096;

__global__ __launch_bounds__(1024) void refine_order_kernel(const double *__restrict__ in,
                                                            uint64_t *__restrict__ keys,
                                                            SpeciesOffsets off, int32_t k,
                                                            FrameParams p) {
  __shared__ uint16_t co[3][kRefine];
  __shared__ uint4 key[kRefine / 4];
  __shared__ uint32_t own[kRefine];
  __shared__ uint32_t lo[kRefine / 128][3], hi[kRefine / 128][3];
  const int tid = threadIdx.x, lane = tid & 63;
  int64_t b0 = 0;
  int s = 0;
  for (; s + 1 < k; ++s) {
    const int64_t nb = (off.v[s + 1] - off.v[s] + kRefine - 1) / kRefine;
    if (blockIdx.x < b0 + nb) break;
    b0 += nb;
  }
  const int64_t first = off.v[s] + (blockIdx.x - b0) * kRefine;
  const int count = static_cast<int>(min(static_cast<int64_t>(kRefine), off.v[s + 1] - first));
  for (int q = tid; q < count; q += 1024) {
    own[q] = static_cast<uint32_t>(keys[first + q] & 0x7FFFFFFFull);
    const int64_t i = 3 * static_cast<int64_t>(own[q]);
    const double x = in[i], y = in[i + 1], z = in[i + 2];
    co[0][q] = static_cast<uint16_t>(fix32(fma(z, p.h13, fma(y, p.h12, x * p.h11))) >> 16);
    co[1][q] = static_cast<uint16_t>(fix32(fma(z, p.h23, y * p.h22)) >> 16);
    co[2][q] = static_cast<uint16_t>(fix32(z * p.h33) >> 16);
  }
  // lengths of the cell vectors: the spread along an axis in length units
  const float len[3] = {static_cast<float>(p.ax),
                        sqrtf(static_cast<float>(p.bx * p.bx + p.by * p.by)),
                        sqrtf(static_cast<float>(p.cx * p.cx + p.cy * p.cy + p.cz * p.cz))};
  // the thread's four consecutive places: keys at 4 tid .. 4 tid + 3
  uint32_t v[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = static_cast<uint32_t>(4 * tid + r);
  for (int m = kRefine; m > 64; m >>= 1) {
    const int g = 4 * tid / m;
    if (tid < kRefine / 128 * 3) {
      lo[tid / 3][tid % 3] = 0xFFFFFFFFu;
      hi[tid / 3][tid % 3] = 0u;
    }
    __syncthreads();
    // (a wave holds 256 places, so at m = 128 two segments)
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      uint32_t l = 0xFFFFFFFFu, h = 0u;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = static_cast<int>(v[r] & (kRefine - 1));
        const bool ok = e < count;
        l = min(l, ok ? static_cast<uint32_t>(co[ax][e]) : 0xFFFFFFFFu);
        h = max(h, ok ? static_cast<uint32_t>(co[ax][e]) : 0u);
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) {
        l = min(l, static_cast<uint32_t>(__shfl_xor(l, o)));
        h = max(h, static_cast<uint32_t>(__shfl_xor(h, o)));
      }
      if ((lane & 31) == 0) {
        atomicMin(&lo[g][ax], l);
        atomicMax(&hi[g][ax], h);
      }
    }
    __syncthreads();
    int ax = 0;
    float widest = -1.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float w = static_cast<float>(static_cast<int>(hi[g][a] - lo[g][a])) * len[a];
      if (w > widest) {
        widest = w;
        ax = a;
      }
    }
    __syncthreads();  // (lo and hi are cleared for the next level)
    // places past the run's end go last
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t e = v[r] & (kRefine - 1);
      v[r] = ((static_cast<int>(e) < count ? static_cast<uint32_t>(co[ax][e]) : 0xFFFFFu) << 12) |
             e;
    }
    for (int kk = 2; kk <= m; kk <<= 1)
      for (int j = kk / 2; j > 0; j >>= 1) {
        const bool asc = ((4 * tid) & (m - 1) & kk) == 0;
        if (j == 1) {
          // (stage 2 sorts the second two the other way)
          bitonic_cas(v[0], v[1], asc);
          bitonic_cas(v[2], v[3], kk == 2 ? false : asc);
        } else if (j == 2) {
          bitonic_cas(v[0], v[2], asc);
          bitonic_cas(v[1], v[3], asc);
        } else {
          uint32_t o[4];
          if (j <= 128) {
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = __shfl_xor(v[r], j / 4);
          } else {
            __syncthreads();
            key[tid] = make_uint4(v[0], v[1], v[2], v[3]);
            __syncthreads();
            const uint4 w = key[tid ^ (j / 4)];
            o[0] = w.x;
            o[1] = w.y;
            o[2] = w.z;
            o[3] = w.w;
          }
          const bool least = ((tid & (j / 4)) == 0) == asc;
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = least ? min(v[r], o[r]) : max(v[r], o[r]);
        }
      }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (4 * tid + r < count) keys[first + 4 * tid + r] = own[v[r] & (kRefine - 1)];
}

// binary64 staging of a sorted frame, one group of 64 points per wave: the
// position of the wrapped point relative to the cell centre in units of 2^22
// bins, the point's input index, and the group's boxes.
__global__ void stage_sorted64_kernel(const double *__restrict__ in,
                                      const uint64_t *__restrict__ keys, SpeciesOffsets off,
                                      int32_t k, FrameParams p, char *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t group = blockIdx.x * static_cast<int64_t>(blockDim.x / 64) + threadIdx.x / 64;
  if (64 * group >= p.n_pad) return;
  int64_t g0 = 0;
  int s = 0;
  for (; s + 1 < k; ++s) {
    const int64_t ng = (off.v[s + 1] - off.v[s] + 63) / 64;
    if (group < g0 + ng) break;
    g0 += ng;
  }
  const int64_t q = off.v[s] + 64 * (group - g0) + lane;
  const bool ok = q < off.v[s + 1];
  uint32_t u[3] = {0u, 0u, 0u};
  double c[3] = {0.0, 0.0, 0.0};
  double mag = 0.0;
  uint32_t from = 0;
  if (ok) {
    from = static_cast<uint32_t>(keys[q] & 0x7FFFFFFFull);
    const double x = in[3 * static_cast<int64_t>(from)], y = in[3 * static_cast<int64_t>(from) + 1],
                 z = in[3 * static_cast<int64_t>(from) + 2];
    const double fa = fma(z, p.h13, fma(y, p.h12, x * p.h11));
    const double fb = fma(z, p.h23, y * p.h22);
    const double fc = z * p.h33;
    const double na = wrap_cell(fa, u[0]) + 0.5, nb = wrap_cell(fb, u[1]) + 0.5,
                 nc = wrap_cell(fc, u[2]) + 0.5;
    c[0] = fma(-p.cx, nc, fma(-p.bx, nb, fma(-p.ax, na, x)));
    c[1] = fma(-p.cy, nc, fma(-p.by, nb, y));
    c[2] = fma(-p.cz, nc, z);
    mag = fabs(x) + fabs(y) + fabs(z);
    if (!(mag < 1e300)) mag = __builtin_inf();
  }
  const double scale = p.s * 0x1p-22;
  const int64_t at = 64 * group + lane, n_pad = p.n_pad;
  double *const pos = reinterpret_cast<double *>(out) + 3 * at;
  reinterpret_cast<uint32_t *>(out + 24 * n_pad)[at] = from;
  GroupBox b;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    pos[ax] = c[ax] * scale;
    const float f = static_cast<float>(c[ax]);
    b.ulo[ax] = wave_min(ok ? u[ax] : 0xFFFFFFFFu);
    b.uhi[ax] = wave_max(ok ? u[ax] : 0u);
    b.clo[ax] = wave_min(ok ? f : __builtin_inff());
    b.chi[ax] = wave_max(ok ? f : -__builtin_inff());
  }
  // (rounded up)
  b.mag = wave_max(static_cast<float>(mag)) * 1.000001f;
  for (uint32_t &v : b.unused) v = 0u;
  if (lane == 0) reinterpret_cast<GroupBox *>(out + 28 * n_pad)[group] = b;
}

// Batched staging: blockIdx.y selects the frame.
template <int PREC>
__global__ void stage_batch_kernel(const FrameParams *__restrict__ frames) {
  const FrameParams &p = frames[blockIdx.y];
  // spatially sorted frames are staged by their own sort
  if (p.box == kBoxTricSorted || p.box == kBoxSearchSorted) return;
  const int64_t n = p.n_points;
  const double *__restrict__ in = p.in;
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += step) {
    const double x = in[3 * i], y = in[3 * i + 1], z = in[3 * i + 2];
    if constexpr (PREC == 1) {
      static_cast<double4 *>(const_cast<void *>(p.coords))[i] = make_double4(x, y, z, 0.0);
    } else {
      float4 v;
      if (p.box == kBoxNone)
        v = stage_point32<kBoxNone>(x, y, z, p);
      else if (p.box == kBoxOrtho || p.box == kBoxCube)
        v = stage_point32<kBoxOrtho>(x, y, z, p);
      else
        v = stage_point32<kBoxTric>(x, y, z, p);
      static_cast<float4 *>(const_cast<void *>(p.coords))[i] = v;
    }
  }
}

// Batched zeroing of every frame's histograms, plus the work counters.
__global__ void zero_batch_kernel(const FrameParams *__restrict__ frames, int32_t *counters,
                                  int32_t n_counters) {
  const FrameParams &p = frames[blockIdx.y];
  const int64_t n = static_cast<int64_t>(p.n_hist) * p.n_bins;
  const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (blockIdx.y == 0 && i0 < n_counters) counters[i0] = 0;
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = i0; i < n; i += step) p.out[i] = 0ull;
}

// Batched out-of-range counts: blockIdx.x = histogram, blockIdx.y = frame.
__global__ void oor_batch_kernel(const FrameParams *__restrict__ frames) {
  __shared__ unsigned long long part[256];
  const FrameParams &p = frames[blockIdx.y];
  const int h = blockIdx.x;
  if (p.oor == nullptr || h >= p.n_hist) return;
  unsigned long long v = 0;
  for (int b = threadIdx.x; b < p.n_bins; b += blockDim.x)
    v += p.out[static_cast<size_t>(h) * p.n_bins + b];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) p.oor[h] = p.pairs[h] - part[0];
}

// --------------------------------------------------------------------------
// Small kernels
// --------------------------------------------------------------------------

__global__ void zero_kernel(ZeroArgs z) { zero_part(z); }

__global__ void oor_kernel(const uint64_t *__restrict__ hist, int32_t n_bins,
                           const uint64_t *__restrict__ pairs, uint64_t *__restrict__ oor) {
  __shared__ unsigned long long part[256];
  const int h = blockIdx.x;
  unsigned long long v = 0;
  for (int b = threadIdx.x; b < n_bins; b += blockDim.x)
    v += hist[static_cast<size_t>(h) * n_bins + b];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) oor[h] = pairs[h] - part[0];
}

template <typename T, int BOX>
__global__ void pair_t_kernel(const FrameParams *F, const int32_t *__restrict__ pi,
                              const int32_t *__restrict__ pj, int64_t n_pairs, int32_t n,
                              double *__restrict__ out) {
  using V = typename V4<T>::type;
  const V *X = static_cast<const V *>(F->coords);
  const typename Geo<T>::type g = Geo<T>::load(F);
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < n_pairs;
       k += step) {
    const int i = min(max(pi[k], 0), n - 1), j = min(max(pj[k], 0), n - 1);
    const V a = X[i], b = X[j];
    out[k] = static_cast<double>(pair_t<T, BOX>(a.x, a.y, a.z, b.x, b.y, b.z, g));
  }
}

PairFn pick(int precision, int r, int box, int mode) {
  switch (mode) {
    case kModeSweep:
      return precision == 1 ? pick_pairs<double, kModeSweep>(r, box)
                            : pick_pairs<float, kModeSweep>(r, box);
    case kModeGlobal:
      return precision == 1 ? pick_pairs<double, kModeGlobal>(r, box)
                            : pick_pairs<float, kModeGlobal>(r, box);
    default:
      return precision == 1 ? pick_pairs<double, kModeLds>(r, box)
                            : pick_pairs<float, kModeLds>(r, box);
  }
}

// threads a clearing launch can use
int64_t zero_span(const ZeroArgs &z) {
  return std::max<int64_t>({z.n_words, z.n_counters, z.oor ? z.n_hist : 0, 1});
}

int grid_for(int64_t n, int threads) {
  int64_t g = (n + threads - 1) / threads;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return static_cast<int>(g);
}

}  // namespace

hipError_t launch_stage_sorted(int precision, const double *in, void *out, int64_t n,
                               const int64_t *offsets, int32_t n_species, const FrameParams &fp,
                               uint64_t *keys, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n_species < 1 || n_species > kMaxSpeciesStage || n > 0x7FFFFFFFll)
    return hipErrorInvalidValue;
  const int64_t npad = sort_keys_count(n);
  SpeciesOffsets off;
  for (int s = 0; s <= kMaxSpeciesStage; ++s) off.v[s] = offsets[s < n_species ? s : n_species];
  const int threads = 256;
  const int wgs = static_cast<int>((fp.n_pad / 64 + 3) / 4);
  sort_keys_kernel<<<grid_for(npad, threads), threads, 0, st>>>(in, n, npad, off, n_species, fp,
                                                                keys);
  const int blocks = static_cast<int>(npad / kBitonicBlock);
  bitonic_local_kernel<<<blocks, 1024, 0, st>>>(keys, 0, 1);
  for (int64_t kk = 2 * kBitonicBlock; kk <= npad; kk <<= 1) {
    int64_t j = kk / 2;
    for (; j >= 2 * kBitonicBlock; j >>= 2)
      bitonic_global_kernel<true><<<grid_for(npad / 4, threads), threads, 0, st>>>(keys, npad, j,
                                                                                  kk);
    if (j >= kBitonicBlock)
      bitonic_global_kernel<false><<<grid_for(npad / 2, threads), threads, 0, st>>>(keys, npad, j,
                                                                                   kk);
    bitonic_local_kernel<<<blocks, 1024, 0, st>>>(keys, kk, 0);
  }
  if (precision == 0) {
    stage_sorted_kernel<<<wgs, threads, 0, st>>>(in, keys, off, n_species, fp,
                                                 static_cast<char *>(out));
    return hipGetLastError();
  }
  int64_t runs = 0;
  for (int s = 0; s < n_species; ++s) runs += (off.v[s + 1] - off.v[s] + kRefine - 1) / kRefine;
  refine_order_kernel<<<static_cast<int>(runs), 1024, 0, st>>>(in, keys, off, n_species, fp);
  stage_sorted64_kernel<<<wgs, threads, 0, st>>>(in, keys, off, n_species, fp,
                                                 static_cast<char *>(out));
  return hipGetLastError();
}

hipError_t launch_stage(int precision, int box_kind, const double *in, void *out, int64_t n,
                        const FrameParams &fp, const ZeroArgs &z, hipStream_t st) {
  if (padded_frame(box_kind)) return hipErrorInvalidValue;  // launch_stage_sorted
  const int threads = 256;
  const int grid = grid_for(std::max(n, zero_span(z)), threads);
  if (precision == 1) {
    stage64_kernel<<<grid, threads, 0, st>>>(in, static_cast<double4 *>(out), n, z);
  } else {
    float4 *o = static_cast<float4 *>(out);
    switch (box_kind) {
      case kBoxNone: stage32_kernel<kBoxNone><<<grid, threads, 0, st>>>(in, o, n, fp, z); break;
      case kBoxOrtho:
      case kBoxCube: stage32_kernel<kBoxOrtho><<<grid, threads, 0, st>>>(in, o, n, fp, z); break;
      default: stage32_kernel<kBoxTric><<<grid, threads, 0, st>>>(in, o, n, fp, z); break;
    }
  }
  return hipGetLastError();
}

hipError_t launch_zero(const ZeroArgs &z, hipStream_t st) {
  const int threads = 256;
  zero_kernel<<<grid_for(zero_span(z), threads), threads, 0, st>>>(z);
  return hipGetLastError();
}

// Allows a pair kernel the whole LDS of a CU. Every caller sets the same
// value, so contexts launching from several host threads cannot lower the
// limit between another thread's check and launch.
static void allow_full_lds(PairFn fn) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)hipGetLastError();
}

hipError_t launch_pairs(int precision, int box_kind, int mode, const KernelConfig &cfg,
                        const PairKernelArgs &args, int grid, size_t lds_bytes, hipStream_t st) {
  PairFn fn = pick(precision, cfg.r, box_kind, mode);
  allow_full_lds(fn);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(cfg.threads), lds_bytes, st, args);
  return hipGetLastError();
}

int pairs_occupancy(int precision, int box_kind, int mode, const KernelConfig &cfg,
                    size_t lds_bytes) {
  PairFn fn = pick(precision, cfg.r, box_kind, mode);
  allow_full_lds(fn);
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, cfg.threads, lds_bytes) !=
      hipSuccess) {
    (void)hipGetLastError();
    return 1;
  }
  return blocks > 0 ? blocks : 1;
}

hipError_t launch_oor(const uint64_t *hist, int32_t n_hist, int32_t n_bins, const uint64_t *pairs,
                      uint64_t *oor, hipStream_t st) {
  if (n_hist <= 0) return hipSuccess;
  oor_kernel<<<n_hist, 256, 0, st>>>(hist, n_bins, pairs, oor);
  return hipGetLastError();
}

hipError_t launch_stage_batch(int precision, const FrameParams *d_frames, int32_t n_frames,
                              int64_t max_points, hipStream_t st) {
  if (n_frames <= 0 || max_points <= 0) return hipSuccess;
  const int threads = 256;
  int gx = static_cast<int>(std::min<int64_t>((max_points + threads - 1) / threads, 64));
  dim3 grid(gx, n_frames);
  if (precision == 1)
    stage_batch_kernel<1><<<grid, threads, 0, st>>>(d_frames);
  else
    stage_batch_kernel<0><<<grid, threads, 0, st>>>(d_frames);
  return hipGetLastError();
}

hipError_t launch_zero_batch(const FrameParams *d_frames, int32_t n_frames, int64_t max_words,
                             int32_t *counters, int32_t n_counters, hipStream_t st) {
  if (n_frames <= 0) return hipSuccess;
  const int threads = 256;
  int64_t need = std::max<int64_t>(max_words, n_counters);
  int gx = static_cast<int>(std::min<int64_t>(std::max<int64_t>((need + threads - 1) / threads, 1), 64));
  zero_batch_kernel<<<dim3(gx, n_frames), threads, 0, st>>>(d_frames, counters, n_counters);
  return hipGetLastError();
}

hipError_t launch_oor_batch(const FrameParams *d_frames, int32_t n_frames, int32_t max_hist,
                            hipStream_t st) {
  if (n_frames <= 0 || max_hist <= 0) return hipSuccess;
  oor_batch_kernel<<<dim3(max_hist, n_frames), 256, 0, st>>>(d_frames);
  return hipGetLastError();
}

hipError_t launch_pair_t(int precision, int box_kind, const FrameParams *d_fp, const int32_t *pi,
                         const int32_t *pj, int64_t n_pairs, int32_t n, double *t,
                         hipStream_t st) {
  if (n_pairs <= 0) return hipSuccess;
  const int threads = 256;
  const int grid = grid_for(n_pairs, threads);
  if (precision == 1) {
    switch (box_kind) {
      case kBoxNone: pair_t_kernel<double, kBoxNone><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      case kBoxOrtho:
      case kBoxCube: pair_t_kernel<double, kBoxOrtho><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      case kBoxTric: pair_t_kernel<double, kBoxTric><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      default: pair_t_kernel<double, kBoxTricSearch><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
    }
  } else {
    switch (box_kind) {
      case kBoxNone: pair_t_kernel<float, kBoxNone><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      case kBoxOrtho: pair_t_kernel<float, kBoxOrtho><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      case kBoxCube: pair_t_kernel<float, kBoxCube><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      case kBoxTric: pair_t_kernel<float, kBoxTric><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
      default: pair_t_kernel<float, kBoxTricSearch><<<grid, threads, 0, st>>>(d_fp, pi, pj, n_pairs, n, t); break;
    }
  }
  return hipGetLastError();
}

}  // namespace dh
