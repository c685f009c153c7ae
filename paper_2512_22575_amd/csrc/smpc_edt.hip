// Signed Euclidean distance field from an occupancy grid (Sec. III-B) for gfx950.
//
// The field is built from two exact squared Euclidean distance transforms on the
// voxel lattice: D_out, the squared index distance from every voxel to the nearest
// occupied voxel, and D_in, to the nearest free voxel.  Each is separable: a 1-D
// transform along every axis in turn, D(p) = min_q ((p - q)^2 + f(q)), starting
// from 0 on the sources and "none" elsewhere.  The paper runs the 1-D
// Felzenszwalb-Huttenlocher (FH) lower-envelope transform along y, x, z on a layout
// whose contiguous axis is y, gathering each strided line into a per-thread buffer.
// The exact result does not depend on the order of the axes; on the planner's
// x-fastest layout the same plan (contiguous axis first) is x, y, z:
//
//   pass x  (binary input): 16 lanes per row; the ends of the run of equal voxels that a
//           voxel lies in give the nearest voxel of the other kind on either side;
//   pass y  32 (x, z) lines per block, staged in an LDS tile;
//   pass z  the same over 32 (x, y) lines per block, writing the outputs: phi =
//           voxel * (sqrt(D_out) - sqrt(D_in)) and/or the two squared fields.
//
// Compact intermediates: after every pass a voxel's value in its own field is 0 (a
// free voxel is a source of D_in, an occupied one of D_out), so one value per voxel
// plus its occupancy bit carries both fields: 16 bits after the x pass, 32 after the
// y pass.
//
// Passes y and z do not build FH's envelope.  Its lists are serial chains with a branch
// per sample: split over 16 lanes per line they took 75 us (y) and 107 us (z) of a 200^3
// field of 40 obstacles, at 150 VALU and as many SALU instructions per output.  They use
// the other property of the same minimisation, that the minimiser over q moves right with
// p (transform_lines): 48 and 53 us on the same grid.  Four blocks of seven waves fit a CU, so
// 1024 of such a grid's 1250 run at once and the others as those end; blocks inside obstacles
// take up to twice the mean time.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "smpc_internal.h"

namespace smpc {
namespace {

// Compact per-voxel records: a voxel's occupancy and its distance to the nearest voxel of
// the other kind.
//   after x: bit 15 occupied, bits 0..14 the distance along the row
//   after y: bit 31 occupied, bits 0..30 the squared distance in the plane
// No such voxel: the distance is kNoDist, whose square is above any squared distance in a
// grid (3 * 511^2 < 2^20) and, like any distance, carries through the passes that follow:
// a result of 2^20 or more means none.
constexpr uint16_t kXOcc = 0x8000u;
constexpr uint32_t kYOcc = 0x80000000u;
constexpr int kNoDist = 1254;
constexpr uint32_t kNoneD = 1u << 20;
static_assert((long long)kNoDist * kNoDist >= kNoneD &&
                  3ll * (kEdtMaxSide - 1) * (kEdtMaxSide - 1) < kNoneD,
              "kNoDist tells an absent source");

// ---------------------------------------------------------------------------
// Pass x: per voxel, the distance along its row to the nearest voxel of the other kind
// (occupied for a free voxel, free for an occupied one).
//
// A row is cut into runs of one kind; the distance is to the near end of the run on
// either side.  A row lies on 16 lanes, kVox consecutive voxels on each: one or two
// loads, a bit per voxel that begins a run, a scan over the 16 lanes for the last
// begin to the left and the first one to the right, and from there along the lane's own
// voxels two operations per voxel and side.  Rows begin at any byte, so loads and stores
// are unaligned ones.  A voxel per lane (byte loads, four bit scans of 64-bit ballots per
// voxel) took 29 us of 333x257x141, four voxels per lane by the same scans 14.2 us of
// 200^3 and 3.4 us of 64^3; this one 17.2, 7.9 and 2.8.  Moving 3 bytes per voxel
// takes about 5 us of 200^3.
// ---------------------------------------------------------------------------
constexpr int kRowWaves = 4;      // waves per block
constexpr int kRowLanes = 16;     // lanes per row (a row of the DPP shifts)
constexpr int kRowsPerBlock = kRowWaves * 64 / kRowLanes;

// x of the lane kN to the left / right among the row's 16; `none` where there is none.
template <int kN>
__device__ __forceinline__ int from_left(int none, int x) {
  return __builtin_amdgcn_update_dpp(none, x, 0x110 + kN, 0xF, 0xF, false);
}
template <int kN>
__device__ __forceinline__ int from_right(int none, int x) {
  return __builtin_amdgcn_update_dpp(none, x, 0x100 + kN, 0xF, 0xF, false);
}

template <int kVox>
__global__ __launch_bounds__(64 * kRowWaves) void edt_pass_x_kernel(
    const uint8_t* __restrict__ occ, int nx, uint32_t rows, uint32_t nvox,
    uint16_t* __restrict__ xrec) {
  static_assert(kVox % 8 == 0 && kVox <= 32);
  const uint32_t row = blockIdx.x * kRowsPerBlock + threadIdx.x / kRowLanes;
  const int p0 = (threadIdx.x % kRowLanes) * kVox;  // the lane's first voxel
  const int own = row < rows ? nx - p0 : 0;         // voxels from there on
  const uint32_t at = row * (uint32_t)nx + p0;
  uint32_t word[kVox / 4] = {};
  if (own > 0) {
    if (at + kVox <= nvox) {
      __builtin_memcpy(word, occ + at, kVox);
    } else {  // the grid's last bytes
#pragma unroll
      for (int k = 0; k < kVox; ++k)
        if (at + k < nvox) word[k / 4] |= (uint32_t)occ[at + k] << (8 * (k % 4));
    }
  }
  uint32_t m = 0u;  // bit k: voxel p0 + k is occupied
#pragma unroll
  for (int i = 0; i < kVox / 4; ++i) {
    const uint32_t high = 0x80808080u;
    const uint32_t set = ((((word[i] & ~high) + ~high) | word[i]) & high) >> 7;
    m |= __builtin_amdgcn_udot4(set, 0x08040201u, 0u, false) << (4 * i);
  }
  // Bit k: voxel p0 + k is of another kind than the one before it.
  const uint32_t before = (uint32_t)from_left<1>((int)(m << (kVox - 1)), (int)m) >> (kVox - 1);
  uint32_t begin = m ^ ((m << 1) | (before & 1u));
  if (own < kVox) begin &= (1u << max(own, 0)) - 1u;
  if (kVox < 32) begin &= (1u << (kVox % 32)) - 1u;

  // The last begin in the lanes to the left, the first one in those to the right; kNoDist
  // and more away from any voxel of the row if there is none.
  constexpr int kNone = 2048;
  int l = begin ? p0 + 31 - __clz((int)begin) : -kNone;
  int r = begin ? p0 + __ffs((int)begin) - 1 : kNone;
  l = max(l, from_left<1>(-kNone, l));
  r = min(r, from_right<1>(kNone, r));
  l = max(l, from_left<2>(-kNone, l));
  r = min(r, from_right<2>(kNone, r));
  l = max(l, from_left<4>(-kNone, l));
  r = min(r, from_right<4>(kNone, r));
  l = max(l, from_left<8>(-kNone, l));
  r = min(r, from_right<8>(kNone, r));
  l = from_left<1>(-kNone, l);
  r = from_right<1>(kNone, r);
  if (own <= 0) return;

  // Distances to the voxel before the run and to the one after it.
  int left[kVox];
  int d = p0 - l;
#pragma unroll
  for (int k = 0; k < kVox; ++k) {
    d = (begin >> k) & 1u ? 1 : d + 1;
    left[k] = d;
  }
  uint32_t out[kVox / 2] = {};
  d = r - (p0 + kVox);
#pragma unroll
  for (int k = kVox - 1; k >= 0; --k) {
    d = (k < kVox - 1 && (begin >> (k + 1)) & 1u) ? 1 : d + 1;
    const uint32_t rec = (uint32_t)min(min(left[k], d), kNoDist) | ((m >> k) & 1u) << 15;
    out[k / 2] |= rec << (16 * (k % 2));
  }
  uint16_t* dst = xrec + at;
  if (own >= kVox) {
    __builtin_memcpy(dst, out, 2 * kVox);
    return;
  }
  // The row's last lane: the powers of two in its count, in turn.
#pragma unroll
  for (int h = 16; h >= 2; h /= 2) {
    if (h < kVox && (own & h)) {
      __builtin_memcpy(dst, out, 2 * h);
      dst += h;
#pragma unroll
      for (int i = 0; i < h / 2 && i + h / 2 < kVox / 2; ++i) out[i] = out[i + h / 2];
    }
  }
  if (own & 1) *dst = (uint16_t)out[0];
}

// The flags of all threads of the block (at most kWaves waves) or'ed; a block barrier.  Call
// sites that can follow one another without a barrier have their own kSite.
// (__syncthreads_or costs this kernel about 40 registers and two more barriers.)
template <int kWaves, int kSite>
__device__ __forceinline__ uint32_t block_or(bool bit0, bool bit1) {
  __shared__ uint32_t waves_or[kWaves];
  const int lane = threadIdx.x & 63;
  const uint32_t mine = (__any(bit0) ? 1u : 0u) | (__any(bit1) ? 2u : 0u);
  if (lane == 0) waves_or[threadIdx.x / 64] = mine;
  __syncthreads();
  const uint32_t w = lane < (int)(blockDim.x / 64) ? waves_or[min(lane, kWaves - 1)] : 0u;
  return (__any(w & 1u) ? 1u : 0u) | (__any(w & 2u) ? 2u : 0u);
}

// ---------------------------------------------------------------------------
// Passes y and z: the 1-D transform D(p) = min_q (f(q) + (p - q)^2) of 32 lines per
// block, the line's samples in a column of an LDS tile, one half-wave ("team") of lanes
// per group of outputs, lane l of a team on line l (each half of a wave reads one row of
// 32 banks at a time, whatever row its lanes are at, so no read has bank conflicts).
//
// The minimiser of output p over q moves right as p does (the cost is a Monge array), so
// the minimisers of outputs kLeaf apart ("cuts") are found first, those of a unit's first
// output over the whole line, the ones between by halving, each between its neighbours'
// minimisers; then the kLeaf outputs from one cut to the next scan the rows between the
// two minimisers, with all their minima in registers.  A line of n outputs costs about
// n^2 / (8 kPer) + 20 n pair evaluations (kPer = 1, 2 or 4, below) instead of the n^2 of the
// definition, in loops without data-dependent lists; all of it is integer arithmetic on 32-bit
// words, so the result is exact.
//
// Tile words.  A D_out sample f(q) is stored as (f(q) + q^2) << kShift, from which
// f(q) + (p - q)^2 follows by adding (p^2 - 2 p q) << kShift: one addition per pair.
// f + q^2 < 2^21 - 2^18 (also where f is the square of kNoDist), so no sum leaves 31 bits.
// The low kShift bits are free: bit 0 tells an occupied voxel and the search for a
// minimiser adds q << 1, so that one signed minimum finds value and minimiser together
// (the leftmost one on ties).  While D_in is computed, an occupied voxel's word is
// the complement of its D_in sample instead (negative, a free voxel's is not).
// ---------------------------------------------------------------------------
constexpr int kLines = 32;              // lines per block, one per lane of a team
constexpr int kLeaf = 8;                // outputs between two cuts
constexpr int kPad = 3;                 // rows of "no sample" after a line
constexpr int kTry = 8, kReach = 64;    // rows the D_in search goes out from a leaf (below)
constexpr int kShift = 10;
constexpr int kFar = kNoDist * kNoDist;  // sample of a padding row
static_assert((2ll * (kEdtMaxSide - 1) + 1) < (1 << kShift), "q and the flag fit the low bits");
static_assert(((long long)kFar + (kEdtMaxSide + kPad) * (kEdtMaxSide + kPad)) << kShift < (1ll << 31),
              "words and sums fit 31 bits");

// A team stages one unit of kPer leaves of its block's lines and searches the minimiser at
// the unit's first output over the whole line; the cuts in between and the leaves are
// dealt to the teams in turn (obstacles and far regions cover neighbouring outputs).
// kPer = 1, 2, 4 for lines of up to 64, 384 and 512 samples, at most twelve waves per
// block: small grids still fill the chip, and a block inside an obstacle, which the pass
// ends with, has twice the waves that kPer = 4 gives it.  Fields with kPer = 4 and with 2:
// 200^3 104.8 and 103.1 us, 300x300x100 146 and 139, 64x128x400 61.6 and 59.3; 200x512x64, where
// every block scans its lines 32 times, 95.8 and 101.7.
__host__ __device__ constexpr int line_leaves(int n) { return (n + kLeaf - 1) / kLeaf; }
__host__ __device__ constexpr int unit_leaves(int n) { return n <= 64 ? 1 : n <= 384 ? 2 : 4; }
__host__ __device__ constexpr int line_waves(int n) {
  return ((line_leaves(n) + unit_leaves(n) - 1) / unit_leaves(n) + 1) / 2;
}
constexpr int kMaxWaves = line_waves(384);  // 12
static_assert(line_waves(256) <= kMaxWaves && line_waves(kEdtMaxSide) <= kMaxWaves, "most waves");

// LDS of a block: the padded tile, then the minimisers at the cuts (Index: uint8_t for
// lines of at most 256 samples, else uint16_t).
template <class Index>
constexpr size_t line_lds_bytes(int n) {
  return (size_t)(n + kPad) * kLines * sizeof(int) +
         (size_t)(line_leaves(n) + 1) * kLines * sizeof(Index);
}

__device__ __forceinline__ int min3(int a, int b, int c) { return min(min(a, b), c); }
__device__ __forceinline__ int key_row(int key) { return (key >> 1) & ((1 << (kShift - 1)) - 1); }

// x, opaque to the optimiser.  Where it is used, this toolchain otherwise folds
// d * d + q * q behind a select into one v_dot4_u32_u8, which adds the select's condition
// and drops the bits above the eighth (wrong fields; seen in the assembly), or turns the
// loop's 32 differences into as many induction variables (95 registers, half again as
// many instructions).
__device__ __forceinline__ int opaque(int x) {
  asm("" : "+v"(x));
  return x;
}

// Minima over rows lo .. hi (rows past hi are candidates like any other, at worst padding)
// of the tile word plus (p^2 - 2 p q) << kShift for the kLeaf outputs p from p0 on, less
// p^2: four rows per round, every row serving all outputs.
__device__ __forceinline__ void leaf_minima(const int* col, int p0, int lo, int hi,
                                            int (&acc)[kLeaf]) {
#pragma unroll
  for (int j = 0; j < kLeaf; ++j) acc[j] = 0x7FFFFFFF;
  const int s0 = p0 << (kShift + 1), s1 = -s0, s2 = -2 * s0, s3 = -3 * s0;
  for (int q = lo; q <= hi; q += 4) {
    const int* r = col + q * kLines;
    const int g0 = r[0], g1 = r[kLines], g2 = r[2 * kLines], g3 = r[3 * kLines];
    const int v0 = opaque(q << (kShift + 1)), v1 = opaque(v0 + (1 << (kShift + 1))),
              v2 = opaque(v0 + (2 << (kShift + 1))), v3 = opaque(v0 + (3 << (kShift + 1)));
    const int m = opaque(__mul24(q, s1));
    int b0 = g0 + m, b1 = g1 + m + s1, b2 = g2 + m + s2, b3 = g3 + m + s3;
#pragma unroll
    for (int j = 0; j < kLeaf; ++j) {
      acc[j] = min3(min3(acc[j], b0, b1), b2, b3);
      b0 -= v0;
      b1 -= v1;
      b2 -= v2;
      b3 -= v3;
    }
  }
}

// Transforms the block's lines of n samples: load(q) is the record of row q of the calling
// lane's line (lanes past the grid repeat its last line: the same values to the same
// places).  A voxel's record after the previous pass holds its occupancy and one value:
// the sample of the field it is not a source of.  decode(rec, occ) returns it, at most
// kFar; emit(p, D, occ) receives D_out of each free voxel and D_in of each occupied one.
// Every thread of the block calls this.
template <int kPer, class Index, class Load, class Decode, class Emit>
__device__ __forceinline__ void transform_lines(int* lds, int n, Load&& load, Decode&& decode,
                                                Emit&& emit) {
  const int team = threadIdx.x / kLines, teams = blockDim.x / kLines;
  const int nleaf = line_leaves(n);
  constexpr int kRows = kPer * kLeaf;  // rows of a unit
  const int row0 = team * kRows;
  int* col = lds + threadIdx.x % kLines;  // row q of this lane's line: col[q * kLines]
  Index* cut =
      reinterpret_cast<Index*>(lds + (n + kPad) * kLines) + threadIdx.x % kLines;  // cut[i * kLines]

  uint32_t occ_rows = 0u;  // bit kRows - 1 - k: row row0 + k of this lane's line is occupied
  {
    // Rows past the line repeat its last row.
    decltype(load(0)) v[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) v[k] = load(min(row0 + k, n - 1));
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int q = min(row0 + k, n - 1);
      bool occ = false;
      const int x = opaque((int)decode(v[k], occ));
      col[q * kLines] = occ ? ~x : (x + __mul24(q, q)) << kShift;
      occ_rows = (occ_rows << 1) | (occ ? 1u : 0u);
    }
  }
  if (team == 0) {
#pragma unroll
    for (int k = 0; k < kPad; ++k)  // rows after the line: no source
      col[(n + k) * kLines] = (kFar + (n + k) * (n + k)) << kShift;
    cut[0] = 0;                            // minimisers before the first cut and after the
    cut[nleaf * kLines] = (Index)(n - 1);  // last one: the ends of the line bound them
  }
  constexpr uint32_t kAllRows = 0xFFFFFFFFu >> (32 - kRows);
  const uint32_t kinds = block_or<kMaxWaves, 0>(occ_rows != 0u, occ_rows != kAllRows);
  const bool any_occ = kinds & 1u, any_free = kinds & 2u;
  // D_in at the occupied voxels, f_in being 0 on free ones: the rows of a leaf first, then
  // outward from it (most obstacles are thin against a line) until no farther row can matter to
  // any lane.  A row index clamped into the line is a candidate at more than its true
  // cost, which changes nothing.  Blocks inside obstacles are the last to end, and this is
  // what they spend their time on: with the test of the reach before each pair of rows, and
  // no loop before it, the 200^3 passes went from 53 and 57 us to 49 and 54.
  //
  // After kTry rows the minima found bound the rest of the search: a leaf that could go on
  // beyond kReach rows (the middle of a solid of some 130 voxels and more; a floor's or wall's
  // own plane, where a line has no free voxel and no sample) ends here, and its block, now
  // "deep", gets these leaves' D_in from the scan that gives D_out, in time that does not
  // grow with the thickness.  Without that, 200^3 took 446 us with every voxel occupied and
  // 414 with one free, 200x512x64 with one occupied xy plane 323; now 95, 114 and 80.
  // kReach: 200^3 seen through a camera cone 164, 178, 188 us at 32, 48, 64 rows, with a
  // solid cube of 100 voxels 109, 110, 91 (the search alone: 271 and 89).
  bool deep = false;   // block: some leaf is left to the scan
  uint32_t todo = 0u;  // bit k: the team's k-th leaf is, in this lane
  if (any_occ) {
    for (int turn = 0; team + turn * teams < nleaf; ++turn) {
      const int i = team + turn * teams, p0 = i * kLeaf;
      int own[kLeaf], acc[kLeaf], most = -1;  // own: f_in at occupied voxels, negative at free ones
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) own[j] = ~col[min(p0 + j, n - 1) * kLines];
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) most = max(most, own[j]);
      if (most < 0) continue;
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) {
        acc[j] = max(own[j], 0);
#pragma unroll
        for (int k = 0; k < kLeaf; k += 2)
          acc[j] = min3(acc[j], max(own[k], 0) + (j - k) * (j - k),
                        max(own[k + 1], 0) + (j - k - 1) * (j - k - 1));
      }
      const int dmax = max(p0, n - p0 - kLeaf);  // rows on the longer side
      bool far = false;
      for (int d = 1; d <= dmax; d += 2) {
        // Every output's rows nearer than d are in.
        int worst = acc[0];
#pragma unroll
        for (int j = 1; j < kLeaf; ++j) worst = max(worst, acc[j]);
        if (worst <= d * d) break;
        if (d == kTry + 1 && worst > kReach * kReach) {
          far = true;
          break;
        }
        int f[4];
        f[0] = col[max(p0 - d, 0) * kLines];
        f[1] = col[max(p0 - d - 1, 0) * kLines];
        f[2] = col[min(p0 + kLeaf - 1 + d, n - 1) * kLines];
        f[3] = col[min(p0 + kLeaf + d, n - 1) * kLines];
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = max(~f[c], 0);
#pragma unroll
        for (int j = 0; j < kLeaf; ++j) {
          const int lo = d + j, hi = d + kLeaf - 1 - j;
          acc[j] = min3(acc[j], f[0] + lo * lo, f[1] + (lo + 1) * (lo + 1));
          acc[j] = min3(acc[j], f[2] + hi * hi, f[3] + (hi + 1) * (hi + 1));
        }
      }
      if (far) {
        todo |= 1u << turn;
        continue;
      }
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) {
        const int p = p0 + j;
        if (p < n && own[j] >= 0) emit(p, (uint32_t)acc[j], true);
      }
    }
    deep = block_or<kMaxWaves, 1>(todo != 0u, false) != 0u;
  }

  // The tile of a field's samples, which are 0 on its sources, marked by bit 0; the records
  // are read a second time.
  auto fill = [&](bool in) {
    int first = row0;  // opaque: the loads are not those of the staging, kept in registers
    asm volatile("" : "+v"(first));
    constexpr int kAtOnce = kRows < 16 ? kRows : 16;
#pragma unroll 1
    for (int k0 = 0; k0 < kRows; k0 += kAtOnce) {
      decltype(load(0)) v[kAtOnce];
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) v[k] = load(min(first + k0 + k, n - 1));
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const int q = min(first + k0 + k, n - 1);
        bool occ = false;
        const int x = opaque((int)decode(v[k], occ));
        const int q2 = __mul24(q, q);
        col[q * kLines] = occ == in ? (x + q2) << kShift : (q2 << kShift) | 1;
      }
    }
  };
  // The leaves between cuts: those left to it (D_in) or all (D_out).
  auto scan = [&](auto field) {
    constexpr bool in = decltype(field)::value;
    // The minimiser at the unit's first output, over the whole line (the first unit's is
    // bounded by row 0 instead), the next eight rows in flight.
    if (row0 > 0 && row0 < n) {
      int best = 0x7FFFFFFF;
      // Row q adds q dt: (p^2 - 2 p q) << kShift | 2 q, less p^2.
      const int dt = 2 - (row0 << (kShift + 1));
      int ct[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) ct[c] = opaque(c * dt);
      const int* r = col;
      int t = 0;
      int g[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) g[c] = r[c * kLines];
      for (int left = n / 8; left > 1; --left) {
        r += 8 * kLines;
        int next[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) next[c] = r[c * kLines];
#pragma unroll
        for (int c = 0; c < 8; c += 2) best = min3(best, g[c] + ct[c] + t, g[c + 1] + ct[c + 1] + t);
        t = opaque(t + 8 * dt);
#pragma unroll
        for (int c = 0; c < 8; ++c) g[c] = next[c];
      }
#pragma unroll
      for (int c = 0; c < 8; c += 2) best = min3(best, g[c] + ct[c] + t, g[c + 1] + ct[c + 1] + t);
      t += 8 * dt;
      r += 8 * kLines;
      for (int q = n & ~7; q < n; ++q, t += dt, r += kLines) best = min(best, r[0] + t);
      cut[team * kPer * kLines] = (Index)key_row(best);
    }
    __syncthreads();

    // The other cuts, by halving, each between its neighbours' minimisers.
#pragma unroll
    for (int s = kPer / 2; s >= 1; s >>= 1) {
      for (int i = (2 * team + 1) * s; i < nleaf; i += 2 * teams * s) {
        const int lo = cut[(i - s) * kLines], hi = cut[min(i + s, nleaf) * kLines];
        int key = 0x7FFFFFFF;
        const int s1 = 2 - ((i * kLeaf) << (kShift + 1)), s2 = 2 * s1, s3 = 3 * s1;
        for (int q = lo; q <= hi; q += 4) {
          const int* r = col + q * kLines;
          const int m = __mul24(q, s1);
          key = min3(key, r[0] + m, r[kLines] + m + s1);
          key = min3(key, r[2 * kLines] + m + s2, r[3 * kLines] + m + s3);
        }
        cut[i * kLines] = (Index)min(key_row(key), hi);
      }
      __syncthreads();
    }

    for (int turn = 0; team + turn * teams < nleaf; ++turn) {
      if (in && !(todo & (1u << turn))) continue;
      const int i = team + turn * teams, p0 = i * kLeaf;
      int acc[kLeaf];
      leaf_minima(col, p0, cut[i * kLines], cut[(i + 1) * kLines], acc);
      int own[kLeaf];
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) own[j] = col[min(p0 + j, n - 1) * kLines];
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) {
        const int p = p0 + j;
        if (p < n && !(own[j] & 1))
          emit(p, (uint32_t)(acc[j] + (__mul24(p, p) << kShift)) >> kShift, in);
      }
    }
  };
  if (deep) {
    fill(true);
    __syncthreads();
    scan(std::true_type{});
    if (any_free) {
      __syncthreads();
      fill(false);
      __syncthreads();
    }
  } else if (any_occ) {
    // The occupied voxels become D_out's sources (sample 0), marked by bit 0.
    for (uint32_t rows = occ_rows; rows != 0u; rows &= rows - 1u) {
      const int q = min(row0 + kRows - 1 - __builtin_ctz(rows), n - 1);
      col[q * kLines] = (__mul24(q, q) << kShift) | 1;
    }
    __syncthreads();
  }
  if (any_free) scan(std::false_type{});  // else no voxel takes D_out
}

// Block b's tile.  Blocks are dispatched to XCD b mod 8; the G neighbouring tiles that
// share 128-byte lines of the records form a group that runs on one XCD, so each line is
// fetched into one L2 once, and consecutive groups go to consecutive XCDs, so that every
// XCD gets a share of every region of the grid.  Tiles past the last are padding.
template <int G>
__host__ __device__ __forceinline__ long long xcd_blocks(long long tiles) {
  return 8 * (((tiles + G - 1) / G + 7) / 8) * G;
}
template <int G>
__device__ __forceinline__ uint32_t xcd_tile() {
  const uint32_t b = blockIdx.x, k = b / 8;  // k-th tile of this XCD
  return ((b % 8) + 8 * (k / G)) * G + k % G;
}
// In a grid whose rows do not start on 128-byte lines, each tile shares the first and the last
// line of every row with its neighbours, and two halves of a line written through different
// L2s go to memory twice (z pass of 333x257x141: 3.5 M write requests for 2.3 M lines' worth).
// Field of 333x257x141 by tiles per group: 182.1 us (2 and 1, what aligned rows need), 164.4
// (4), 161.4 (8), 161.3 (16); 200^3, whose rows are aligned in the z pass: 103.2, 102.7, 103.3,
// 104.3.
constexpr int kGroup = 8;

// The element `off` bytes after a uniform base (off < 2^32).
template <class T>
__device__ __forceinline__ T& at_byte(T* base, uint32_t off) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + off);
}
template <class T>
__device__ __forceinline__ const T& at_byte(const T* base, uint32_t off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}

// Pass y: block = 32 consecutive lines (z, x).
template <int kPer, class Index>
__global__ __launch_bounds__(64 * kMaxWaves) void edt_pass_y_kernel(
    const uint16_t* __restrict__ xrec, uint32_t* __restrict__ yrec, int nx, int ny, int nz) {
  extern __shared__ int lds[];
  const uint32_t lines = (uint32_t)nx * nz, tile = xcd_tile<kGroup>();
  if (tile * kLines >= lines) return;  // whole block
  const uint32_t l = min(tile * kLines + threadIdx.x % kLines, lines - 1u);
  const uint32_t z = l / (uint32_t)nx, x = l - z * nx;
  const uint32_t at = z * (uint32_t)(nx * ny) + x;  // the line's first voxel, < 2^27
  transform_lines<kPer, Index>(
      lds, ny, [&](int q) { return at_byte(xrec, 2u * at + __umul24(q, 2 * nx)); },
      [](uint16_t r, bool& occ) -> uint32_t {
        occ = r & kXOcc;
        const uint32_t d = r & 0x7FFFu;
        return __umul24(d, d);
      },
      [&](int p, uint32_t d, bool occ) {
        at_byte(yrec, 4u * at + __umul24(p, 4 * nx)) = d | (occ ? kYOcc : 0u);
      });
}

// The outputs of voxel i, which is occupied or not and has squared distance D to the
// nearest voxel of the other kind (none_value: none in the grid): phi = voxel *
// (sqrt(D_out) - sqrt(D_in)), in float64 and rounded to float32 once, and/or the two
// squared fields.  One of D_out, D_in is 0 (a voxel is a source of one field), so phi
// is exactly +-voxel * sqrt(D) (subtracting sqrt(0) = 0 and negating are exact).
struct FieldOut {
  float* phi;     // [nvox] or null
  uint32_t* d2;   // [2][nvox] or null
  uint32_t nvox;
  double voxel;
  uint32_t none_value;
  // off: four times the voxel's index.
  __device__ __forceinline__ void put(uint32_t off, bool occ, uint32_t d) const {
    const uint32_t D = d >= kNoneD ? none_value : d;
    if (d2) {
      at_byte(d2, off) = occ ? 0u : D;
      at_byte(d2 + nvox, off) = occ ? D : 0u;
    }
    if (phi) {
      const double v = voxel * __builtin_sqrt((double)D);
      at_byte(phi, off) = (float)(occ ? -v : v);
    }
  }
};

// Pass z: block = 32 consecutive lines (y, x); writes the outputs.  At 81 scalar registers
// (what it takes without the limit) fewer waves fit a SIMD: 200^3 with no obstacle 67 us
// instead of 66.
template <int kPer, class Index>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_num_sgpr(80)))
void edt_pass_z_kernel(const uint32_t* __restrict__ yrec, int nx, int ny, int nz, FieldOut fo) {
  extern __shared__ int lds[];
  const uint32_t plane = (uint32_t)nx * ny, tile = xcd_tile<kGroup>();
  if (tile * kLines >= plane) return;  // whole block
  const uint32_t at = min(tile * kLines + threadIdx.x % kLines, plane - 1u);
  transform_lines<kPer, Index>(
      lds, nz, [&](int q) { return at_byte(yrec, 4u * (at + __umul24(q, plane))); },
      [](uint32_t r, bool& occ) -> uint32_t {
        occ = r & kYOcc;
        return r & ~kYOcc;
      },
      [&](int p, uint32_t d, bool occ) { fo.put(4u * (at + __umul24(p, plane)), occ, d); });
}

template <int kPer, class Index>
void launch_pass_y(const uint16_t* xrec, uint32_t* yrec, int nx, int ny, int nz,
                   hipStream_t stream) {
  const long long tiles = ((long long)nx * nz + kLines - 1) / kLines;
  hipLaunchKernelGGL((edt_pass_y_kernel<kPer, Index>), dim3((unsigned)xcd_blocks<kGroup>(tiles)),
                     dim3(64 * line_waves(ny)), line_lds_bytes<Index>(ny), stream, xrec, yrec, nx,
                     ny, nz);
}
template <int kPer, class Index>
void launch_pass_z(const uint32_t* yrec, int nx, int ny, int nz, const FieldOut& fo,
                   hipStream_t stream) {
  const long long tiles = ((long long)nx * ny + kLines - 1) / kLines;
  hipLaunchKernelGGL((edt_pass_z_kernel<kPer, Index>), dim3((unsigned)xcd_blocks<kGroup>(tiles)),
                     dim3(64 * line_waves(nz)), line_lds_bytes<Index>(nz), stream, yrec, nx, ny,
                     nz, fo);
}

void launch_line_passes(const uint16_t* xrec, uint32_t* yrec, int nx, int ny, int nz,
                        const FieldOut& fo, hipStream_t stream) {
  const auto y = ny <= 64    ? launch_pass_y<1, uint8_t>
                 : ny <= 256 ? launch_pass_y<2, uint8_t>
                 : ny <= 384 ? launch_pass_y<2, uint16_t>
                             : launch_pass_y<4, uint16_t>;
  const auto z = nz <= 64    ? launch_pass_z<1, uint8_t>
                 : nz <= 256 ? launch_pass_z<2, uint8_t>
                 : nz <= 384 ? launch_pass_z<2, uint16_t>
                             : launch_pass_z<4, uint16_t>;
  y(xrec, yrec, nx, ny, nz, stream);
  z(yrec, nx, ny, nz, fo, stream);
}

}  // namespace

size_t edt_workspace_bytes(long long nvox) {
  // y-pass records (u32), then the x-pass records (u16).
  return (size_t)nvox * (2 * sizeof(uint32_t));
}

size_t edt_lds_bytes(int n_line) {
  return n_line <= 256 ? line_lds_bytes<uint8_t>(n_line) : line_lds_bytes<uint16_t>(n_line);
}

int launch_edt(const uint8_t* occ, int nx, int ny, int nz, float voxel, float* phi,
               uint32_t* d2, void* work, hipStream_t stream) {
  const long long plane = (long long)nx * ny;
  const long long nvox = plane * nz;
  uint32_t* yrec = static_cast<uint32_t*>(work);
  uint16_t* xrec = reinterpret_cast<uint16_t*>(yrec + nvox);
  const long long rows = (long long)ny * nz;
  const uint32_t none_value = (uint32_t)nx * nx + (uint32_t)ny * ny + (uint32_t)nz * nz;
  // 16 lanes of 16 voxels hold a row of up to 256, of 24 one of up to 384, of 32 one of up
  // to 512 (a 333-voxel row takes 14 lanes of 24 or 11 of 32: the field of 333x257x141 160.0
  // and 161.4 us).
  const auto x_kernel = nx <= 256   ? edt_pass_x_kernel<16>
                        : nx <= 384 ? edt_pass_x_kernel<24>
                                    : edt_pass_x_kernel<kEdtMaxSide / kRowLanes>;
  hipLaunchKernelGGL(x_kernel, dim3((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock)),
                     dim3(64 * kRowWaves), 0, stream, occ, nx, (uint32_t)rows, (uint32_t)nvox,
                     xrec);
  const FieldOut fo{phi, d2, (uint32_t)nvox, (double)voxel, none_value};
  launch_line_passes(xrec, yrec, nx, ny, nz, fo, stream);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace smpc
