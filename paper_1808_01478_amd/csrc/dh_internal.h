// Internal types shared by the host planner and the gfx950 kernels of
// libdisthist. Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>

namespace dh {

enum BoxKind : int32_t {
  kBoxNone = 0,
  kBoxOrtho = 1,
  kBoxTric = 2,        // Eq. 5 reduction only (r_max below half the smallest width)
  kBoxTricSearch = 3,  // Eq. 5 reduction, then the 27 neighbouring images
  kBoxCube = 4,        // binary32 only: orthorhombic cell with equal edges
  // Eq. 5 reduction only, points spatially sorted within each species at
  // staging (frames of at least kSortMinPoints; see staged_kind)
  kBoxTricSorted = 5,
  // the same with the neighbouring images (binary64; see staged_kind)
  kBoxSearchSorted = 6,
};

// Largest species count of a frame (the staging kernels take the offsets by
// value).
constexpr int kMaxSpeciesStage = 64;
// frames with at least this many points may be staged in spatial order
// (kBoxTricSorted, see staged_kind)
constexpr int64_t kSortMinPoints = int64_t{1} << 16;

// i-span of a work unit of a sorted frame (see dh_sorted.h)
constexpr int32_t kUnitPoints = 512;

// Sorted frames are staged with every species at a multiple of 64 points
// ("padded" indices, used by their work items too), so that index / 64 is a
// point's group: binary32 the Cartesian positions (float4) and the fixed-point
// words (three each), binary64 the scaled positions (three doubles) and the
// input indices (one word), then the groups' boxes. Together they fit in the
// 32 bytes per point of staged_point_bytes (29 per padded point plus one box;
// frames have at least kSortMinPoints points and at most kMaxSpeciesStage
// species).
inline bool padded_frame(int kind) {
  return kind == kBoxTricSorted || kind == kBoxSearchSorted;
}
__host__ __device__ inline int64_t padded_start(const int64_t *off, int32_t s) {
  int64_t p = 0;
  for (int32_t u = 0; u < s; ++u) p += (off[u + 1] - off[u] + 63) / 64 * 64;
  return p;
}
inline void padded_starts(const int64_t *off, int32_t k, int64_t (&start)[kMaxSpeciesStage + 1]) {
  for (int32_t s = 0; s <= k; ++s) start[s] = padded_start(off, s);
}
// Bounding boxes of a group of 64 points of one species: fixed-point
// fractional coordinates and Cartesian positions relative to the cell centre.
struct GroupBox {
  uint32_t ulo[3], uhi[3];
  float clo[3], chi[3];
  float mag;  // binary64: largest |x| + |y| + |z| of the input (inf: not all finite)
  uint32_t unused[3];
};
static_assert(sizeof(GroupBox) == 64, "one box per 64 points at one byte a point");

// First of the three fixed-point words of padded point i (binary32): beyond 32
// bits from 715,827,883 points on, and frames may have almost 2^31.
__host__ __device__ inline int64_t first_word(int32_t i) { return 3 * static_cast<int64_t>(i); }

// The cell n a fractional coordinate f lies in and its place in that cell as
// 32-bit fixed point, floor(2^32 (f - n)). Both come from one decision: for f
// just below an integer f - floor(f) rounds to 1, and the point is then at the
// lower face of the next cell in both. (With n = floor(f) and the place wrapped
// to 0 a group's box named one image of such a point and its position the
// next, a whole cell vector away.)
__host__ __device__ inline double wrap_cell(double f, uint32_t &place) {
  double n = floor(f), w = f - n;
  if (w >= 1.0) {
    n += 1.0;
    w = 0.0;
  }
  place = static_cast<uint32_t>(static_cast<uint64_t>(w * 4294967296.0));
  return n;
}

// Bytes per staged point (binary64 double4; binary32 float4, two of them
// for spatially sorted frames) and the sort workspace of a frame.
inline size_t staged_point_bytes(int precision, int kind) {
  return precision != 0 || padded_frame(kind) ? 32 : 16;
}
inline int64_t sort_keys_count(int64_t n) {
  int64_t p = 8192;  // one block of the sort
  while (p < n) p <<= 1;
  return p;
}

// Whether the species are large enough for the sorted image search: groups of 64
// points of a small one span much of the cell, so that too many images stay open
// between two groups. Sorted over unsorted time at 2,062, 2,812, 3,125, 4,062,
// 4,125 and 6,250 points a species (66,000 to 200,000 uniform points, cut-off 1.6
// half widths): 3.4, 1.3, 1.1, 0.7, 0.8 and 0.9. A sixteenth of the points may be
// in smaller species.
inline bool tight_species(const int64_t *off, int32_t k) {
  int64_t loose = 0;
  for (int32_t s = 0; s < k; ++s) loose += off[s + 1] - off[s] < 4096 ? off[s + 1] - off[s] : 0;
  return 16 * loose <= off[k];
}

// Bin windows from which one pass of global atomics replaces them by default, in
// binary64 (see kWideDefault32)
constexpr int32_t kWideDefault64 = 20;

// How a pair kernel accumulates its counts.
enum HistMode : int32_t {
  kModeLds = 0,     // the whole histogram in LDS sub-histograms
  kModeSweep = 1,   // LDS sub-histograms of one bin window per item
  kModeGlobal = 2,  // uint64 atomics straight into the output (wide histograms)
};

// WorkItem::flags
constexpr int32_t kItemDiag = 1;  // the j-range lies in the i-block: count j > i only

constexpr int kShifts = 27;
// index of the zero shift (i = j = k = 0) in the shift tables
constexpr int kZeroShift = 13;
// the image search keeps at most kOctCap images per octant of a reduced
// vector (octants that need more search all 27)
constexpr int kOctCap = 12;
// the search's LDS table: 8 octant rows of kOctCap shift vectors, then the
// 27 shift vectors (the full list)
constexpr int kSearchTable = 8 * kOctCap + kShifts;
// slack e of the octant boxes in fractional coordinates (see octant_images)
constexpr double kOctSlack = 0x1p-30;
// bytes of LDS before the histogram's guard: the workgroup's control words
constexpr int kControlBytes = 32;
constexpr int kDump = 64;  // per-lane discard slots after the bin window
// Per-wave LDS ring of reduced vectors waiting for the 27-image search: the
// wave searches 64 of them as soon as 64 are queued, after each slice of
// pairs, so a slice adds at most 64 on top of fewer than 64 (the same for
// every number of slices r).
constexpr int queue_cap(int /* slices per lane */) { return 128; }

// Constants of one frame, computed once on the host.
//
// binary64 members follow the canonical op sequence: s = n_bins / r_max,
// iL = 1 / L, and the inverse of the upper-triangular cell matrix
//   h11 = 1/ax, h22 = 1/by, h33 = 1/cz, h12 = -bx/(ax*by),
//   h23 = -cy/(by*cz), h13 = (bx*cy - by*cx)/(ax*by*cz),
// with shifts S = i*a + j*b + k*c for i, j, k in {-1, 0, 1}.
//
// binary32 members serve the reduced-precision path. Without a box the
// coordinates are staged pre-scaled by s. With a periodic cell they are
// staged as 32-bit fixed-point fractional coordinates u = 2^32 * (f mod 1),
// f = B^-1 x: the wrapped difference u_j - u_i read as a signed integer is
// 2^32 * (f_j - f_i - nint(f_j - f_i)), the reduced vector of Eq. 5 in
// fractional form, and the cell matrix scaled by s / 2^32 maps it to t units.
struct FrameParams {
  const void *coords;  // staged float4 / double4 [N] (device)
  uint64_t *out;       // [H][n_bins] (device)
  const double *in;    // caller's binary64 [N][3] (device)
  uint64_t *oor;       // caller's out-of-range counts [H] or null (device)
  const uint64_t *pairs;  // pairs per histogram [H] (device)
  int64_t n_points;
  int32_t n_pad;   // sorted frames: points with every species padded
  int32_t n_hist;
  int32_t oor_by_flush;  // 1: oor starts at pairs and every flush subtracts its counts
  int32_t n_bins;
  int32_t box;         // BoxKind
  int32_t win;         // bin window of one sweep (<= n_bins)
  int32_t n_sweeps;
  double s;
  double L[3], iL[3];
  double ax, bx, by, cx, cy, cz;
  double h11, h12, h13, h22, h23, h33;
  double shift64[kShifts][3];
  float k32[3];        // orthorhombic: L_c * s / 2^32 (cube: k32[0])
  float ryz32[2];      // orthorhombic: (L_y / L_x)^2, (L_z / L_x)^2
  float Bk[6];         // ax bx by cx cy cz, times s / 2^32
  float Bn[5];         // bx by cx cy cz divided by ax
  float shift32[kShifts][3];  // image shifts times s
  int32_t noclamp;     // 1: every t of a full block fits below `stride` slots
  float qskip32;       // binary32 q (t units) below which no image is nearer
  double qskip64;      // binary64 q below which the reduced vector is nearest
  // image search: pairs that went through the image search are added to
  // searched[0], the images evaluated for them to searched[1] (device,
  // 8-byte aligned) unless null
  unsigned long long *searched;
  // spatially sorted binary32 frames: the cell rows (ax bx by cx cy cz), the
  // entries of B^-1 (h11 h12 h13 h22 h23 h33) and s = n_bins / r_max,
  // rounded to binary32
  float cell32[6];
  float hinv32[6];
  float s32;
  // image search: for each octant of a reduced vector's fractional
  // coordinates (bit k set when component k is negative) the images that
  // can be nearer than the vector itself, as indices into the shift tables
  // padded with the zero shift (kZeroShift); oct_full bit o when octant o
  // needs more than kOctCap images (it searches all 27); oct_n the longest
  // of the other lists; oct_seven 1 when every octant's list holds only
  // images shifted against the vector's signs
  uint8_t oct_shift[8][kOctCap];
  uint8_t oct_full;
  uint8_t oct_n;
  uint8_t oct_seven;
};

// Whether binary32 squares of lengths decide about groups of pairs in a cell whose
// entries add up to `size`.
__host__ __device__ inline bool bounds_decide(double size) {
  return size > 0x1p-40 && size < 0x1p60;
}

// The minimum-image kind the kernels use for a frame: the geometric kind of
// frame_constants (fp), with large frames staged in spatial order (triclinic
// frames in both precisions; orthorhombic ones in binary64, where the sorted
// kernel with a diagonal cell matrix gives the orthorhombic sequence's
// counts bit for bit; frames with image search in binary64, see below) and the
// binary32 special case of equal orthorhombic edges.
//
// Sorted kernels decide whole groups of pairs from squares of lengths in
// binary32, widened by 2^-16 of the cell's entries (their sum); where the squares
// of the cell or of that widening come near the ends of binary32 they decide
// nothing (cube of edge 6e-22: subnormal squares rounded by up to 1/2 of
// themselves, and group pairs with a pair within the cut-off were left out).
// Such binary64 frames stay unsorted; binary32 frames, whose counts depend on the
// kernel in the last places, keep their order and compute every pair.
//
// Without image search a wrap that rounding decides otherwise than the canonical
// sequence must not matter: such a pair is half a cell apart along some axis up
// to 2^-25 of it (see rounding_bound), so it is out of range under either wrap
// when the cut-off keeps 2^-22 from half the smallest width; binary64 frames that
// come closer stay unsorted. (In an orthorhombic cell the two images are equally
// far to within the bound of the rounding.)
//
// The sorted binary64 kernel takes bins from a binary32 root of numbers scaled
// by s 2^-22: fewer than 2^20 bins, and a scale whose square is a normal
// number. With image search it takes a pair's nearest image, which is the
// canonical minimum over 27 images when no image outside them can be nearer:
// such an image differs by two or more cell vectors along some axis from the
// reduced vector, so it is at least 1.5 times the smallest cell width long,
// and the reduced vector is no longer than the longest half diagonal.
// (may_search: the caller can hold the sort workspace such a frame needs, and its
// species are large enough, see tight_species.)
inline int staged_kind(int kind, int precision, const FrameParams &fp, int64_t n_points,
                       bool may_search = true) {
  const bool fits =
      precision == 0 || (fp.n_bins < (1 << 20) - 2 && fp.s > 0x1p-400 && fp.s < 0x1p400);
  double size = 0.0;
  for (double v : {fp.ax, fp.bx, fp.by, fp.cx, fp.cy, fp.cz}) size += fabs(v);
  const bool ranged = precision == 0 || bounds_decide(size);
  // (padded indices fit in 32 bits, those of a unit past the last point too)
  const bool large =
      n_points >= kSortMinPoints && n_points <= 0x7FFFFFFF - 128 * kMaxSpeciesStage && fits &&
      ranged;
  // 1 / width^2 along each axis: the squared rows of B^-1
  const double ra = fp.h11 * fp.h11 + fp.h12 * fp.h12 + fp.h13 * fp.h13;
  const double rb = fp.h22 * fp.h22 + fp.h23 * fp.h23, rc = fp.h33 * fp.h33;
  const double r = ra > rb ? (ra > rc ? ra : rc) : (rb > rc ? rb : rc);
  const double cut = 2.0 * fp.n_bins / fp.s;  // twice the cut-off
  const bool clear = precision == 0 || kind != kBoxTric || cut * cut * r < 1.0 - 0x1p-21;
  if (large && clear && (kind == kBoxTric || (kind == kBoxOrtho && precision != 0)))
    return kBoxTricSorted;
  if (large && kind == kBoxTricSearch && precision != 0 && may_search) {
    double diagonal2 = 0.0;
    for (int q = 0; q < 8; ++q) {
      const double a = q & 1 ? 0.5 : -0.5, b = q & 2 ? 0.5 : -0.5, c = q & 4 ? 0.5 : -0.5;
      const double x = a * fp.ax + b * fp.bx + c * fp.cx, y = b * fp.by + c * fp.cy,
                   z = c * fp.cz;
      const double d2 = x * x + y * y + z * z;
      diagonal2 = d2 > diagonal2 ? d2 : diagonal2;
    }
    if (diagonal2 * r < 2.25 * (1.0 - 1e-6)) return kBoxSearchSorted;
  }
  if (precision != 0) return kind;
  if (kind == kBoxOrtho && fp.L[0] == fp.L[1] && fp.L[1] == fp.L[2]) return kBoxCube;
  return kind;
}

// One unit of work: particles [i0, i1) of the frame against [j0, j1), for
// histogram `hist`, bin window `sweep`; flags: kItemDiag.
struct WorkItem {
  int32_t frame, hist, sweep, flags;
  int32_t i0, i1, j0, j1;
};

struct PairKernelArgs {
  const FrameParams *frames;
  const WorkItem *items;
  int32_t *counter;  // dynamic work counter, zero before launch
  int32_t n_items;
  int32_t stride;    // LDS slots (>= win + kDump of every frame); 0 in kModeGlobal
  int32_t tj;        // longest j-piece of a unit (unsorted frames)
};

// Kernel configuration (chosen per launch by the tuner).
struct KernelConfig {
  int32_t threads;   // workgroup size: 256, 512 or 1024
  int32_t r;         // i-particles per lane (4 or 8)
  int32_t copies;    // histograms the LDS of a workgroup is sized for (1, 2, 4)
  int32_t tj;        // longest j-piece of a unit (unsorted frames)
  int32_t iblock;    // i-range of one work item (multiple of 64 r)
  int32_t jchunk;    // j-range of one work item
  int32_t dchunk;    // j-range of one item on the diagonal of its i-block
  int32_t wg_per_cu; // 0 = as many as fit
};

// How a work list cuts pairs into items: `work` pairs over `grid` workgroups,
// about items_per_wg items each, as i-blocks of whole 64 r-particle slices by
// j-ranges.
//
// Unsorted frames: an item's waves share it in units (see run_units), so its
// i-block may be any number of slices. It starts as one slice per wave and is
// halved while the item would be wider in i than in j: a frame of a few
// thousand points then still gives every CU an item, where whole
// threads x r blocks left most of the chip idle. An item costs a few
// microseconds to draw, start and, where the histogram changes, flush, in
// which a CU counts some 5e4 binary32 pairs: items are not cut below
// kMinItemPairs, nor, once every workgroup has one, below the size given
// here (20,000 points in a cube, 1,000 bins: binary32 123 us with 8 items of
// 32k pairs a workgroup, 86 us with two of 122k; binary64 234 and 202 us).
//
// Sorted frames are cut alike, in units of kUnitPoints, four times as
// fine: items beyond the cut-off cost next to nothing, so the others make the
// end of the launch (1M clustered points: 89.9 ms, now 86.7 ms).
constexpr int64_t kMinItemPairs = int64_t{1} << 15;
constexpr int32_t kMinChunk = 32;
// Whether the last items of a list are cut into pieces (see refine_tail): lists of
// fewer than four items per workgroup are cut fine already, and where a histogram
// has fewer than four items every piece adds a flush of its own (20,000 points of
// 64 species without a box, binary32, 4,160 items of 2,080 histograms: 199 us with
// the last 1,024 in quarters, 143 us without).
inline bool cut_tail(const WorkItem *items, size_t n, size_t grid) {
  if (grid == 0 || n < 4 * grid) return false;
  size_t runs = 0;
  for (size_t q = 0; q < n; ++q)
    runs += q == 0 || items[q].frame != items[q - 1].frame || items[q].hist != items[q - 1].hist ||
            items[q].sweep != items[q - 1].sweep;
  return n >= 4 * runs;
}
// granularity of the j-pieces the tail of a work list is cut into
inline int32_t tail_step(int32_t kind) {
  return padded_frame(kind) ? kUnitPoints : kMinChunk;
}
inline void set_items(KernelConfig &c, int32_t precision, int32_t kind, int grid, uint64_t work,
                      int items_per_wg) {
  const uint64_t g = static_cast<uint64_t>(grid > 0 ? grid : 1);
  int64_t bi = static_cast<int64_t>(c.threads) * c.r, jc;
  if (padded_frame(kind)) {
    const int64_t target = static_cast<int64_t>(work / (g * 4 * items_per_wg));
    bi = 16 * kUnitPoints;
    while (bi > kUnitPoints && target / bi < bi) bi /= 2;
    jc = (target / bi + kUnitPoints - 1) / kUnitPoints * kUnitPoints;
    jc = jc < kUnitPoints ? kUnitPoints : jc;
    jc = jc > 32 * kUnitPoints ? 32 * kUnitPoints : jc;
    c.dchunk = static_cast<int32_t>(jc);
  } else {
    const int64_t per_wg = static_cast<int64_t>(work / g), small = int64_t{1}
                                                                   << (precision ? 16 : 17);
    int64_t target = per_wg < small ? per_wg : small;
    target = target < kMinItemPairs ? kMinItemPairs : target;
    target = per_wg / items_per_wg > target ? per_wg / items_per_wg : target;
    while (bi > 64 * c.r && target / bi < bi) bi /= 2;
    jc = (target / bi + kMinChunk - 1) / kMinChunk * kMinChunk;
    jc = jc < kMinChunk ? kMinChunk : jc;
    jc = jc > 64 * c.tj ? 64 * c.tj : jc;
    c.dchunk = static_cast<int32_t>(jc);
  }
  c.iblock = static_cast<int32_t>(bi);
  c.jchunk = static_cast<int32_t>(jc);
}

// The next coarser cut (about a quarter of the items), for contexts whose memory
// budget has no room for the list; false at the coarsest, 8,192 i by 16,384 j an
// item.
inline bool coarsen_items(KernelConfig &c) {
  constexpr int32_t kTopI = 16 * kUnitPoints, kTopJ = 32 * kUnitPoints;
  if (c.iblock >= kTopI && c.jchunk >= kTopJ && c.dchunk >= kTopJ) return false;
  auto twice = [](int32_t v, int32_t top) { return v < top / 2 ? 2 * v : v < top ? top : v; };
  c.iblock = twice(c.iblock, kTopI);
  c.jchunk = twice(c.jchunk, kTopJ);
  c.dchunk = twice(c.dchunk, kTopJ);
  return true;
}

// Species pair (s, t) of histogram h among k species, in the library order:
// (0,0), (1,1), ..., (k-1,k-1), then (s,t) for s < t lexicographically.
__host__ __device__ inline void hist_pair(int32_t k, int32_t h, int32_t &s, int32_t &t) {
  s = t = h;
  if (h < k) return;
  int32_t idx = h - k;
  for (s = 0; s < k; ++s) {
    const int32_t m = k - 1 - s;
    if (idx < m) {
      t = s + 1 + idx;
      return;
    }
    idx -= m;
  }
}

// How the work list of one histogram is cut (the host planner and the
// device planner of the allocation-free entry point emit the same items):
// rows are blocks of bi particles in the lanes; an intra-species row has
// diagonal items (when its block holds at least two particles) of at most dc
// j each, followed by j-chunks of at most jc particles from the end of its
// block to the end of the species; a cross-species row puts the larger
// species in the lanes and streams the smaller one in j-chunks.
struct HistRows {
  int64_t lane0, lane1;  // particles in the lanes
  int64_t str0, str1;    // particles streamed as j (cross-species)
  bool intra;
  uint64_t pairs;        // pairs of the histogram
};

// (start: where the species begin in a sorted frame's padded indices, see
// padded_starts; else null)
__host__ __device__ inline HistRows hist_rows(const int64_t *off, int32_t k, int32_t h,
                                              const int64_t *start = nullptr) {
  int32_t s, t;
  hist_pair(k, h, s, t);
  HistRows r;
  const int64_t ns = off[s + 1] - off[s], nt = off[t + 1] - off[t];
  const int64_t ps = start ? start[s] : off[s], pt = start ? start[t] : off[t];
  r.intra = s == t;
  if (r.intra) {
    r.lane0 = r.str0 = ps;
    r.lane1 = r.str1 = ps + ns;
    r.pairs = static_cast<uint64_t>(ns) * static_cast<uint64_t>(ns > 0 ? ns - 1 : 0) / 2;
  } else {
    // the larger species in the lanes
    r.lane0 = ns >= nt ? ps : pt;
    r.lane1 = r.lane0 + (ns >= nt ? ns : nt);
    r.str0 = ns >= nt ? pt : ps;
    r.str1 = r.str0 + (ns >= nt ? nt : ns);
    r.pairs = static_cast<uint64_t>(ns) * static_cast<uint64_t>(nt);
  }
  return r;
}

// (in 32 bits, where the sums of two particle indices and a chunk fit unsigned:
// the device planner divides per histogram)
__host__ __device__ inline int64_t chunks(int64_t n, int64_t size) {
  return (static_cast<uint32_t>(n) + static_cast<uint32_t>(size) - 1u) / static_cast<uint32_t>(size);
}
__host__ __device__ inline int64_t hist_row_count(const HistRows &r, int64_t bi) {
  return chunks(r.lane1 - r.lane0, bi);
}

__host__ __device__ inline int64_t row_item_count(const HistRows &r, int64_t row, int64_t bi,
                                                  int64_t jc, int64_t dc) {
  const int64_t b0 = r.lane0 + row * bi;
  const int64_t b1 = b0 + bi < r.lane1 ? b0 + bi : r.lane1;
  if (r.intra)
    return (b1 - b0 >= 2 ? chunks(b1 - b0, dc) : 0) + chunks(r.lane1 - b1, jc);
  return chunks(r.str1 - r.str0, jc);
}

// Writes the items of one row (for bin window `sweep`) from dst on; returns
// how many. Flags as in WorkItem.
__host__ __device__ inline int64_t emit_row(const HistRows &r, int32_t h, int32_t sweep,
                                            int64_t row, int64_t bi, int64_t jc, int64_t dc,
                                            WorkItem *dst) {
  const int64_t b0 = r.lane0 + row * bi;
  const int64_t b1 = b0 + bi < r.lane1 ? b0 + bi : r.lane1;
  int64_t n = 0;
  auto put = [&](int64_t j0, int64_t j1, int32_t diag) {
    WorkItem w;
    w.frame = 0; w.hist = h; w.sweep = sweep; w.flags = diag;
    w.i0 = static_cast<int32_t>(b0); w.i1 = static_cast<int32_t>(b1);
    w.j0 = static_cast<int32_t>(j0); w.j1 = static_cast<int32_t>(j1);
    dst[n++] = w;
  };
  if (r.intra) {
    if (b1 - b0 >= 2)
      for (int64_t j = b0; j < b1; j += dc) put(j, j + dc < b1 ? j + dc : b1, kItemDiag);
    for (int64_t j = b1; j < r.lane1; j += jc) put(j, j + jc < r.lane1 ? j + jc : r.lane1, 0);
  } else {
    for (int64_t j = r.str0; j < r.str1; j += jc) put(j, j + jc < r.str1 ? j + jc : r.str1, 0);
  }
  return n;
}

// The pair kernel of a precision (T = float or double) and accumulation mode
// for r i-particles per lane and a box kind (dh_pairs.hip).
using PairFn = void (*)(PairKernelArgs);
template <typename T, int MODE>
PairFn pick_pairs(int r, int box);
template <> PairFn pick_pairs<float, kModeLds>(int r, int box);
template <> PairFn pick_pairs<float, kModeSweep>(int r, int box);
template <> PairFn pick_pairs<float, kModeGlobal>(int r, int box);
template <> PairFn pick_pairs<double, kModeLds>(int r, int box);
template <> PairFn pick_pairs<double, kModeSweep>(int r, int box);
template <> PairFn pick_pairs<double, kModeGlobal>(int r, int box);

// host-side launchers (dh_kernels.hip)
// Staging of a sorted frame: the points of every species in Morton
// order of their wrapped fractional coordinates (keys: a workspace of
// sort_keys_count(n) words); staged arrays and group boxes at
// padded indices (see padded_frame).
hipError_t launch_stage_sorted(int precision, const double *in, void *out, int64_t n,
                               const int64_t *offsets, int32_t n_species, const FrameParams &fp,
                               uint64_t *keys, hipStream_t st);
// Clearing of a call's output: out[n_words] and counters[n_counters] become 0
// and, with oor, oor[h] = pairs[h] for h < n_hist (the flushes then subtract
// the in-range counts).
struct ZeroArgs {
  uint64_t *out = nullptr;
  int64_t n_words = 0;
  int32_t *counters = nullptr;
  int32_t n_counters = 0;
  int32_t n_hist = 0;
  uint64_t *oor = nullptr;
  const uint64_t *pairs = nullptr;
};
// staging of an unsorted frame and the clearing in one launch
hipError_t launch_stage(int precision, int box_kind, const double *in, void *out, int64_t n,
                        const FrameParams &fp, const ZeroArgs &z, hipStream_t st);
hipError_t launch_zero(const ZeroArgs &z, hipStream_t st);
hipError_t launch_pairs(int precision, int box_kind, int mode, const KernelConfig &cfg,
                        const PairKernelArgs &args, int grid, size_t lds_bytes, hipStream_t st);
hipError_t launch_oor(const uint64_t *hist, int32_t n_hist, int32_t n_bins, const uint64_t *pairs,
                      uint64_t *oor, hipStream_t st);
// batched staging / zeroing / out-of-range over a device table of frames
hipError_t launch_stage_batch(int precision, const FrameParams *d_frames, int32_t n_frames,
                              int64_t max_points, hipStream_t st);
hipError_t launch_zero_batch(const FrameParams *d_frames, int32_t n_frames, int64_t max_words,
                             int32_t *counters, int32_t n_counters, hipStream_t st);
hipError_t launch_oor_batch(const FrameParams *d_frames, int32_t n_frames, int32_t max_hist,
                            hipStream_t st);
hipError_t launch_pair_t(int precision, int box_kind, const FrameParams *d_fp, const int32_t *pi,
                         const int32_t *pj, int64_t n_pairs, int32_t n, double *t,
                         hipStream_t st);
// Occupancy of the pair kernel (workgroups per CU) for a config and LDS size.
int pairs_occupancy(int precision, int box_kind, int mode, const KernelConfig &cfg,
                    size_t lds_bytes);

}  // namespace dh

struct dh_ctx;
namespace dh {
// device bytes held by a context's scratch (staged coordinates, work blob)
size_t ctx_device_bytes(const dh_ctx *ctx);
// binary64 constants of a frame (s, inverse cell, shifts, box kind; returns
// the kind: none, ortho, triclinic, triclinic with image search)
int frame_constants(int32_t box_type, const double *box, double r_max, int32_t n_bins,
                    FrameParams &fp);
// device ordinal of a context
int ctx_device(const dh_ctx *ctx);
// The launch shape a frame gets with the built-in default knobs (no tuning
// cache) on a device with n_cu compute units and lds_per_block bytes of LDS
// per workgroup; fp comes from frame_constants (box kind, n_bins).
struct LaunchPlan {
  KernelConfig cfg;
  int32_t mode, win, n_sweeps, stride, grid;
  bool noclamp;
  size_t lds;
};
LaunchPlan default_launch(int n_cu, size_t lds_per_block, int precision, const FrameParams &fp,
                          uint64_t total_pairs);
// The same with a given workgroup size (0 = automatic): launches that mix
// frames need one shape for all of them.
LaunchPlan serve_launch(int n_cu, size_t lds_per_block, int precision, const FrameParams &fp,
                        uint64_t total_pairs, int threads);
// Records the message of a failure that has no context (read back by
// dh_ctx_last_error(NULL); a fixed thread-local buffer, so it allocates
// nothing) and returns code.
int thread_fail(int code, const char *fmt, ...);
// zeroes n words with a kernel on stream st (never a memset node in graphs)
int zero_u64(uint64_t *p, int64_t n, hipStream_t st);
// dh_histo_async with an accumulate option: when set, the frame's counts are
// added into d_out (not zeroed first) and no out-of-range counts are written;
// total_pairs (optional) receives the frame's pair count.
int histo_job(dh_ctx *ctx, hipStream_t stream, const double *d_coords, const int64_t *offsets,
              int32_t n_species, int32_t box_type, const double *box, double r_max,
              int32_t n_bins, int32_t precision, uint64_t *d_out, uint64_t *d_out_of_range,
              bool accumulate, uint64_t *total_pairs, bool stepped = false);
// A stepped job (histo_job with stepped set) enqueues staging and zeroing
// only and holds its pair-kernel launches back in the context; step_job
// enqueues the next one on st, or, when none is left, the closing
// out-of-range pass if the job needs one (*done then becomes true). *pairs_left receives the
// pairs of the launches still held back. The context runs nothing else
// until the job is done.
int step_job(dh_ctx *ctx, hipStream_t st, uint64_t *pairs_left, bool *done);
// pairs of a stepped job's next held-back launch (0: the closing pass is next)
uint64_t stepped_next_pairs(const dh_ctx *ctx);
}  // namespace dh
