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
//   pass x  (binary input): one wave per row; ballots of the sources of each
//           64-voxel chunk give the nearest source on either side by bit scans;
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
// p (transform_lines): 49 and 54 us on the same grid, VALU issue (half of the time) and
// the waves' LDS latency being the bound.
#include <hip/hip_runtime.h>

#include <cstdint>

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
// Pass x: per voxel, the distance along its row to the nearest voxel of the other
// kind (occupied for a free voxel, free for an occupied one).
// ---------------------------------------------------------------------------
constexpr int kRowWaves = 4;
constexpr int kRowsPerWave = 4;

// kChunks: 64-voxel chunks a row may hold (nx <= 64 kChunks).
template <int kChunks>
__global__ __launch_bounds__(64 * kRowWaves) void edt_pass_x_kernel(
    const uint8_t* __restrict__ occ, int nx, long long rows, uint16_t* __restrict__ xrec) {
  const int lane = threadIdx.x & 63;
  const long long row0 =
      ((long long)blockIdx.x * kRowWaves + (threadIdx.x >> 6)) * kRowsPerWave;
  if (row0 >= rows) return;  // whole wave leaves together
  const int nch = (nx + 63) >> 6;
  // All loads of the wave's rows first, so their latencies overlap.
  uint8_t v[kRowsPerWave][kChunks];
#pragma unroll
  for (int w = 0; w < kRowsPerWave; ++w) {
    const long long row = row0 + w;
    const uint8_t* src = occ + row * nx;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int p = c * 64 + lane;
      v[w][c] = (row < rows && c < nch && p < nx) ? src[p] : 0;
    }
  }
#pragma unroll
  for (int w = 0; w < kRowsPerWave; ++w) {
    const long long row = row0 + w;
    if (row >= rows) break;
    uint64_t m_occ[kChunks], m_free[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int p = c * 64 + lane;
      m_occ[c] = __ballot(p < nx && v[w][c] != 0);
      m_free[c] = __ballot(p < nx && v[w][c] == 0);
    }
    // Nearest source strictly left of chunk c / strictly right of it (-1 / 2^30: none).
    int left_o[kChunks], left_f[kChunks], right_o[kChunks], right_f[kChunks];
    int lo = -1, lf = -1;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      left_o[c] = lo;
      left_f[c] = lf;
      if (m_occ[c]) lo = c * 64 + 63 - __clzll(m_occ[c]);
      if (m_free[c]) lf = c * 64 + 63 - __clzll(m_free[c]);
    }
    int ro = 1 << 30, rf = 1 << 30;
#pragma unroll
    for (int c = kChunks - 1; c >= 0; --c) {
      right_o[c] = ro;
      right_f[c] = rf;
      if (m_occ[c]) ro = c * 64 + __ffsll((unsigned long long)m_occ[c]) - 1;
      if (m_free[c]) rf = c * 64 + __ffsll((unsigned long long)m_free[c]) - 1;
    }
    const uint64_t at_or_below = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const uint64_t at_or_above = ~0ull << lane;
    uint16_t* out = xrec + row * nx;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int p = c * 64 + lane;
      if (c < nch && p < nx) {
        const bool o = v[w][c] != 0;
        const uint64_t m = o ? m_free[c] : m_occ[c];  // sources of the voxel's other field
        const uint64_t ml = m & at_or_below, mr = m & at_or_above;
        const int l = ml ? c * 64 + 63 - __clzll(ml) : (o ? left_f[c] : left_o[c]);
        const int r = mr ? c * 64 + __ffsll((unsigned long long)mr) - 1
                         : (o ? right_f[c] : right_o[c]);
        int dist = 1 << 30;
        if (l >= 0) dist = p - l;
        if (r < (1 << 30)) dist = min(dist, r - p);
        out[p] = (uint16_t)((o ? kXOcc : 0u) | (uint32_t)min(dist, kNoDist));
      }
    }
  }
}

// Rows whose length is a multiple of 4, at most 256 voxels, in a 4-byte-aligned grid
// (records 8-byte aligned): lane l holds voxels 4l .. 4l + 3 of a row, read as one
// 32-bit word and written as one 8-byte record group.  The nearest voxel of the other
// kind is found in the lane's own four voxels, else in the nearest lane on that side
// holding one (a ballot of the lanes holding each kind, then a lane shuffle of that
// lane's first or last such voxel).
__device__ __forceinline__ int last_bit4(uint32_t m) { return 31 - __clz(m); }  // m != 0
__device__ __forceinline__ int first_bit4(uint32_t m) { return __ffs(m) - 1; }  // m != 0

constexpr int kWordRows = 2;  // rows per wave of the word-per-lane kernel

__global__ __launch_bounds__(64 * kRowWaves) void edt_pass_x_words_kernel(
    const uint8_t* __restrict__ occ, int nx, long long rows, uint16_t* __restrict__ xrec) {
  const int lane = threadIdx.x & 63;
  const long long row0 =
      ((long long)blockIdx.x * kRowWaves + (threadIdx.x >> 6)) * kWordRows;
  if (row0 >= rows) return;  // whole wave leaves together
  const int nw = nx >> 2;    // 32-bit words per row
  const bool has = lane < nw;
  uint32_t word[kWordRows];
#pragma unroll
  for (int w = 0; w < kWordRows; ++w) {
    const long long row = row0 + w;
    word[w] = (row < rows && has)
                  ? *reinterpret_cast<const uint32_t*>(occ + row * nx + 4 * lane)
                  : 0u;
  }
  const uint64_t below = (1ull << lane) - 1ull;               // lanes left of this one
  const uint64_t above = lane == 63 ? 0ull : ~0ull << (lane + 1);
  // "None" on the left / right: p - kNoLeft and kNoRight - p are >= 2^20 for every p.
  constexpr int kNoLeft = -(1 << 20), kNoRight = 1 << 21;
#pragma unroll
  for (int w = 0; w < kWordRows; ++w) {
    const long long row = row0 + w;
    if (row >= rows) break;
    uint32_t mo = 0u;  // bit k: voxel 4 lane + k occupied
#pragma unroll
    for (int k = 0; k < 4; ++k) mo |= (((word[w] >> (8 * k)) & 0xFFu) != 0u ? 1u : 0u) << k;
    const uint32_t mf = has ? (~mo & 0xFu) : 0u;              // free voxels
    const uint64_t lanes_o = __ballot(mo != 0u), lanes_f = __ballot(mf != 0u);
    // This lane's first and last voxel of each kind (absolute indices).
    const int fo = mo ? 4 * lane + first_bit4(mo) : 0, lo = mo ? 4 * lane + last_bit4(mo) : 0;
    const int ff = mf ? 4 * lane + first_bit4(mf) : 0, lf = mf ? 4 * lane + last_bit4(mf) : 0;
    // Nearest lane on each side holding each kind, and its nearest voxel of that kind.
    const uint64_t lo_m = lanes_o & below, ro_m = lanes_o & above;
    const uint64_t lf_m = lanes_f & below, rf_m = lanes_f & above;
    const int lo_src = lo_m ? 63 - __clzll(lo_m) : lane;
    const int ro_src = ro_m ? __ffsll((unsigned long long)ro_m) - 1 : lane;
    const int lf_src = lf_m ? 63 - __clzll(lf_m) : lane;
    const int rf_src = rf_m ? __ffsll((unsigned long long)rf_m) - 1 : lane;
    const int sh_lo = __shfl(lo, lo_src), sh_fo = __shfl(fo, ro_src);
    const int sh_lf = __shfl(lf, lf_src), sh_ff = __shfl(ff, rf_src);
    const int left_o = lo_m ? sh_lo : kNoLeft, right_o = ro_m ? sh_fo : kNoRight;
    const int left_f = lf_m ? sh_lf : kNoLeft, right_f = rf_m ? sh_ff : kNoRight;
    if (!has) continue;
    uint16_t rec[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int p = 4 * lane + k;
      const bool o = (mo >> k) & 1u;
      const uint32_t m = o ? mf : mo;                          // sources of the other kind
      const uint32_t ml = m & ((1u << k) - 1u), mr = m & (0xEu << k) & 0xFu;
      const int l = ml ? 4 * lane + last_bit4(ml) : (o ? left_f : left_o);
      const int r = mr ? 4 * lane + first_bit4(mr) : (o ? right_f : right_o);
      const int dist = min(p - l, r - p);
      rec[k] = (uint16_t)((o ? kXOcc : 0u) | (uint32_t)min(dist, kNoDist));
    }
    uint2 out;
    out.x = (uint32_t)rec[0] | ((uint32_t)rec[1] << 16);
    out.y = (uint32_t)rec[2] | ((uint32_t)rec[3] << 16);
    *reinterpret_cast<uint2*>(xrec + row * nx + 4 * lane) = out;
  }
}

// Whether x holds in any thread of the block (at most kWaves waves); a block barrier.
// (__syncthreads_or costs this kernel about 40 registers and two more barriers.)
template <int kWaves>
__device__ __forceinline__ bool block_any(bool x) {
  __shared__ uint32_t waves_any[kWaves];
  const int lane = threadIdx.x & 63;
  const bool any = __any(x);
  if (lane == 0) waves_any[threadIdx.x / 64] = any;
  __syncthreads();
  return __any(lane < (int)(blockDim.x / 64) && waves_any[min(lane, kWaves - 1)] != 0u);
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
// n^2 / 32 + 20 n pair evaluations instead of the n^2 of the definition, in loops without
// data-dependent lists; all of it is integer arithmetic on 32-bit words, so the result is
// exact.
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
constexpr int kShift = 10;
constexpr int kFar = kNoDist * kNoDist;  // sample of a padding row
static_assert((2ll * (kEdtMaxSide - 1) + 1) < (1 << kShift), "q and the flag fit the low bits");
static_assert(((long long)kFar + (kEdtMaxSide + kPad) * (kEdtMaxSide + kPad)) << kShift < (1ll << 31),
              "words and sums fit 31 bits");

// A team stages one unit of kPer leaves of its block's lines and searches the minimiser at
// the unit's first output over the whole line; the cuts in between and the leaves are
// dealt to the teams in turn (obstacles and far regions cover neighbouring outputs).
// kPer = 1, 2, 4 for lines of up to 64, 128 and 512 samples: about eight teams (four
// waves) per block, so that small grids still fill the chip.
__host__ __device__ constexpr int line_leaves(int n) { return (n + kLeaf - 1) / kLeaf; }
__host__ __device__ constexpr int unit_leaves(int n) { return n <= 64 ? 1 : n <= 128 ? 2 : 4; }
__host__ __device__ constexpr int line_waves(int n) {
  return ((line_leaves(n) + unit_leaves(n) - 1) / unit_leaves(n) + 1) / 2;
}
constexpr int kMaxWaves = line_waves(kEdtMaxSide);  // 8

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
  // D_in at the occupied voxels, f_in being 0 on free ones: the rows of a leaf first, then
  // outward from it (obstacles are thin against a line) until no farther row can matter to
  // any lane.  A row index clamped into the line is a candidate at more than its true
  // cost, which changes nothing.  Blocks inside obstacles are the last to end, and this is
  // what they spend their time on: with the test of the reach before each pair of rows, and
  // no loop before it, the 200^3 passes went from 53 and 57 us to 49 and 54.
  if (block_any<kMaxWaves>(occ_rows != 0u)) {
    for (int i = team; i < nleaf; i += teams) {
      const int p0 = i * kLeaf;
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
      for (int d = 1; d <= dmax; d += 2) {
        // Every output's rows nearer than d are in.
        int worst = acc[0];
#pragma unroll
        for (int j = 1; j < kLeaf; ++j) worst = max(worst, acc[j]);
        if (worst <= d * d) break;
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
#pragma unroll
      for (int j = 0; j < kLeaf; ++j) {
        const int p = p0 + j;
        if (p < n && own[j] >= 0) emit(p, (uint32_t)acc[j], true);
      }
    }
    __syncthreads();
    // The occupied voxels become D_out's sources (sample 0), marked by bit 0.
    for (uint32_t rows = occ_rows; rows != 0u; rows &= rows - 1u) {
      const int q = min(row0 + kRows - 1 - __builtin_ctz(rows), n - 1);
      col[q * kLines] = (__mul24(q, q) << kShift) | 1;
    }
    __syncthreads();
  }
  // The minimiser at the unit's first output, over the whole line (the first unit's is
  // bounded by row 0 instead), eight reads in flight.
  if (row0 > 0 && row0 < n) {
    int best = 0x7FFFFFFF, t = 0;  // t = (p^2 - 2 p q) << kShift | 2 q, less the p^2 term
    const int dt = 2 - (row0 << (kShift + 1));
    int q = 0;
    for (; q + 8 <= n; q += 8) {
      const int* r = col + q * kLines;
      int g[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) g[c] = r[c * kLines];
#pragma unroll
      for (int c = 0; c < 8; c += 2)
        best = min3(best, g[c] + (t + c * dt), g[c + 1] + (t + (c + 1) * dt));
      t += 8 * dt;
    }
    for (; q < n; ++q, t += dt) best = min(best, col[q * kLines] + t);
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

  for (int i = team; i < nleaf; i += teams) {
    const int p0 = i * kLeaf;
    int acc[kLeaf];
    leaf_minima(col, p0, cut[i * kLines], cut[(i + 1) * kLines], acc);
    int own[kLeaf];
#pragma unroll
    for (int j = 0; j < kLeaf; ++j) own[j] = col[min(p0 + j, n - 1) * kLines];
#pragma unroll
    for (int j = 0; j < kLeaf; ++j) {
      const int p = p0 + j;
      if (p < n && !(own[j] & 1))
        emit(p, (uint32_t)(acc[j] + (__mul24(p, p) << kShift)) >> kShift, false);
    }
  }
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
// Tiles per 128-byte line: 32 lines x 2-byte x-records, 32 lines x 4-byte y-records.
constexpr int kGroupY = 2, kGroupZ = 1;

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
  const uint32_t lines = (uint32_t)nx * nz, tile = xcd_tile<kGroupY>();
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

// Pass z: block = 32 consecutive lines (y, x); writes the outputs.
template <int kPer, class Index>
__global__ __launch_bounds__(64 * kMaxWaves) void edt_pass_z_kernel(
    const uint32_t* __restrict__ yrec, int nx, int ny, int nz, FieldOut fo) {
  extern __shared__ int lds[];
  const uint32_t plane = (uint32_t)nx * ny, tile = xcd_tile<kGroupZ>();
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
  hipLaunchKernelGGL((edt_pass_y_kernel<kPer, Index>), dim3((unsigned)xcd_blocks<kGroupY>(tiles)),
                     dim3(64 * line_waves(ny)), line_lds_bytes<Index>(ny), stream, xrec, yrec, nx,
                     ny, nz);
}
template <int kPer, class Index>
void launch_pass_z(const uint32_t* yrec, int nx, int ny, int nz, const FieldOut& fo,
                   hipStream_t stream) {
  const long long tiles = ((long long)nx * ny + kLines - 1) / kLines;
  hipLaunchKernelGGL((edt_pass_z_kernel<kPer, Index>), dim3((unsigned)xcd_blocks<kGroupZ>(tiles)),
                     dim3(64 * line_waves(nz)), line_lds_bytes<Index>(nz), stream, yrec, nx, ny,
                     nz, fo);
}

void launch_line_passes(const uint16_t* xrec, uint32_t* yrec, int nx, int ny, int nz,
                        const FieldOut& fo, hipStream_t stream) {
  const auto y = ny <= 64    ? launch_pass_y<1, uint8_t>
                 : ny <= 128 ? launch_pass_y<2, uint8_t>
                 : ny <= 256 ? launch_pass_y<4, uint8_t>
                             : launch_pass_y<4, uint16_t>;
  const auto z = nz <= 64    ? launch_pass_z<1, uint8_t>
                 : nz <= 128 ? launch_pass_z<2, uint8_t>
                 : nz <= 256 ? launch_pass_z<4, uint8_t>
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
  const long long rows_per_block = (long long)kRowWaves * kRowsPerWave;
  const dim3 xgrid((unsigned)((rows + rows_per_block - 1) / rows_per_block));
  const long long word_rows_per_block = (long long)kRowWaves * kWordRows;
  if (nx <= 256 && nx % 4 == 0 && reinterpret_cast<uintptr_t>(occ) % 4 == 0 &&
      reinterpret_cast<uintptr_t>(xrec) % 8 == 0)
    hipLaunchKernelGGL(edt_pass_x_words_kernel,
                       dim3((unsigned)((rows + word_rows_per_block - 1) / word_rows_per_block)),
                       dim3(64 * kRowWaves), 0, stream, occ, nx, rows, xrec);
  else if (nx <= 256)
    hipLaunchKernelGGL(edt_pass_x_kernel<4>, xgrid, dim3(64 * kRowWaves), 0, stream, occ, nx,
                       rows, xrec);
  else
    hipLaunchKernelGGL(edt_pass_x_kernel<kEdtMaxSide / 64>, xgrid, dim3(64 * kRowWaves), 0,
                       stream, occ, nx, rows, xrec);
  const FieldOut fo{phi, d2, (uint32_t)nvox, (double)voxel, none_value};
  launch_line_passes(xrec, yrec, nx, ny, nz, fo, stream);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace smpc
