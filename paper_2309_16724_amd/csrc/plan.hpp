// Device plan: stripe products (Sec. III A) as grouped GEMM tiles.
#pragma once
#include <algorithm>
#include <vector>
#include "common.hpp"

namespace dmrg {

// Operand bases: 0 = psi (input), 1 = hpsi (output), 2 = stripe workspace,
// 3 = partial-tile buffer, 4 + k = operator data array k.
enum { BASE_PSI = 0, BASE_Y = 1, BASE_WORK = 2, BASE_PART = 3, BASE_OPS = 4 };

// One stripe product contributing to a tile: tile += s * op(A)[rows, 0:K] * B[0:K, cols].
// Operands are stacks of blocks along K (positions) and, for B, along N:
//   A(i, k) = A[(k / a_kb) * a_p + i * a_i + (k % a_kb) * a_k]      (a_base < 0: identity)
//   B(k, n) = B[(k / b_kb) * b_pk + (k % b_kb) * b_k + (n / b_nb) * b_pn + (n % b_nb) * b_n]
struct Seg {
  int64_t a_off, b_off;
  int64_t a_p, a_i, a_k;
  int64_t b_pk, b_k, b_pn, b_n;
  double s;
  int32_t a_base, b_base;
  int32_t K, a_kb, b_kb, b_nb;
  // FP64 device copies (resolve_bases; a_off and b_off are in bytes there): the
  // operands' strides over four K rows, and the extra one when that crosses a
  // position boundary (a_kb == b_kb)
  int64_t da, ea, db, eb;
};

// Element offset of a line of row `row` of position `pos` of an operand, as the
// FP64 wavefront tiles compute it.  Rows and lines have strides below 2^32 (the
// width of a block or a stripe): one multiply-add each.  Positions are whole
// blocks, 2^32 elements and more from sectors of 65536 states on: 64 bits.
__host__ __device__ inline int64_t operand_offset(uint32_t pos, int64_t pos_stride, uint32_t row, int64_t row_stride,
                                                  uint32_t line, int64_t line_stride) {
  return (int64_t)pos * pos_stride + (int64_t)((uint64_t)row * (uint32_t)row_stride) +
         (int64_t)((uint64_t)line * (uint32_t)line_stride);
}

// Work-group tiles: a tile with mb == MACRO_MB is a 64 x 64 tile computed by
// the four wavefronts of a work group together from operand tiles they stage
// in LDS once; the other tiles belong to one wavefront each.
constexpr int MACRO_MB = 8;
constexpr int MACRO_EDGE = 64;
constexpr int MACRO_MIN = 48;   // default: outputs with both dims >= 48 get work-group tiles
// Wide work-group tiles (split plans, s <= 5): WIDE_MB tiles are 128 x 128,
// computed by the eight wavefronts of a work group (two per SIMD, in 32 x 32
// blocks of v_mfma_f32_32x32x16_bf16) from two 80 KiB LDS stages.  An
// output with both sides >= wide_min is cut into 128-wide bands (a last band
// of >= wide_min lines is a wide band too); the rest of it gets 64 x 64 or
// wavefront tiles.
constexpr int WIDE_MB = 16;
constexpr int WIDE_EDGE = 128;
constexpr int WIDE_MIN = 48;
constexpr int WIDE_WAVES = 8;
constexpr int WIDE_MAX_SLICES = 5;
constexpr int F64_WIDE_MB = 32;   // 128 x 128 FP64 tiles of whole work groups (a kernel of their own)
constexpr int tile_rows(int mb) { return mb == WIDE_MB || mb == F64_WIDE_MB ? WIDE_EDGE : mb == MACRO_MB ? MACRO_EDGE : 16 * mb; }
constexpr int tile_cols(int mb) { return mb == WIDE_MB || mb == F64_WIDE_MB ? WIDE_EDGE : mb == MACRO_MB ? MACRO_EDGE : 64 / mb; }

// Per-XCD queues of a tile list: the list (cost-sorted, operand bands in
// patches) is cut into NXCD contiguous ranges of equal cost; the workers of XCD
// x take the tiles of range x in order (the first ones by their index, then
// through an atomic counter) and then help the other ranges, so the tiles
// that run side by side on one XCD are neighbours in the list and share
// operand bands in its L2.
constexpr int NXCD = 8;
constexpr int MACRO_GRID = 512;          // work groups of a work-group tile launch (two per CU)
constexpr int WIDE_GRID = 256;           // work groups of a wide tile launch (one per CU)
constexpr int QUEUE_STRIDE = 32;         // ints between counters: a 128-byte line each
constexpr int QUEUE_SET = NXCD * QUEUE_STRIDE;
constexpr int QUEUE_INTS = 2 * QUEUE_SET;   // two counter sets
struct XcdQueues {
  int32_t start[NXCD + 1];
  int32_t dyn[NXCD];   // first tile of range r that its counter hands out (set per launch)
};
// Light tiles: eleven twelfths of every range go round the workers in turn (at
// least one tile each), the rest to whoever is free first.  Heavy ones: all but
// the first round to whoever is free first.
inline XcdQueues deal(XcdQueues q, int workers, bool heavy) {
  for (int r = 0; r < NXCD; r++) {
    const int len = q.start[r + 1] - q.start[r], rounds = heavy ? 1 : (len - len / 12) / workers;
    q.dyn[r] = q.start[r] + (int)std::min<int64_t>(len, (int64_t)workers * std::max(1, rounds));
  }
  return q;
}
// Work-group tiles of four million flops and more on average are heavy (FP64,
// L=54, D=1024: 87.3 -> 83.8 ms), those of a few K steps are not: their atomics
// and the hand-over of the index to the other waves show (the first stage of
// split plans at L=54, D=768, 3.2 million each: 17.6 -> 19.2 ms).
inline bool heavy_tiles(int ntiles, double flops) { return flops >= 4194304.0 * ntiles; }

// Counters of consecutive tile launches on one stream: a launch uses the
// current set, which is zero when it starts, and clears the other one.  The
// first set is cleared by the launch_zero that opens the sequence.
struct QueueSets {
  int32_t *base;
  int launch = 0;
  int32_t *cur() const { return base + (launch & 1) * QUEUE_SET; }
  int32_t *other() const { return base + (1 - (launch & 1)) * QUEUE_SET; }
};

// Work groups of a wavefront-tile launch (a multiple of NXCD, no more than fit
// on the chip at once: `resident`) and tiles per dynamic chunk: at most about
// 2^18 flops of the list's average (eight 16 x 16 tiles of K = 64), at most 8.
inline int wave_grid(int ntiles, int resident, int waves) {
  const int blocks = (ntiles + waves - 1) / waves;
  return blocks < resident ? (blocks + NXCD - 1) / NXCD * NXCD : resident;
}
inline int wave_chunk(int ntiles, double flops) {
  const double c = 262144.0 * ntiles / (flops > 1.0 ? flops : 1.0);
  return c < 1.0 ? 1 : c > 8.0 ? 8 : (int)c;
}

// FP64 outputs with both sides >= F64_WIDE_MIN, the longer >= F64_WIDE_LONG,
// take 128 x 128 work-group tiles; other outputs (and the strips beyond the
// bands) with both sides >= F64_MACRO_MIN 64 x 64 ones (see TileLevel for
// stages of few outputs).  A 32 x 32 wavefront tile fetches 0.125 B per flop,
// 4.5 TB/s at the 36 TF/s it reached on large outputs; a 128 x 128 one a
// quarter of that.  L=54, D=1024: 138.8 ms with wavefront tiles alone, 87.6 ms
// with 64/48, 89.7 ms with 48/33, 92 ms with 96/48 or 64 x 64 tiles alone (84
// now, see heavy_tiles).  L=24, D=512 (sectors up to 83): 128-wide tiles of
// which both sides are half empty cost 0.87 ms where 64 x 64 ones take 0.63,
// hence F64_WIDE_LONG.  Sectors of WG_MAX_DIM states and more stay with
// wavefront tiles (the work-group tiles address an operand's lines by 32-bit
// byte offsets).
constexpr int F64_WIDE_MIN = 64, F64_WIDE_LONG = 96, F64_MACRO_MIN = 48, WG_MAX_DIM = 1 << 14;

// A cell of an output's tiling: top-left corner and tile kind.
struct Cell { int i0, j0, mb; };

// Time of a tile, in units of a K row of a whole tile: MFMA blocks inside the
// output (half a tile's time is not the products), and a constant for the
// descriptors, the first loads and the store -- without it the range of a list
// that holds its thousands of small tiles ran three times as long as the
// others (L=54, D=512 renormalization).
inline double tile_cost(int mb, int rows, int cols, int nseg, double ksum) {
  const double blocks = (double)((rows + 15) / 16) * ((cols + 15) / 16) /
                        ((double)tile_rows(mb) * tile_cols(mb) / 256.0);
  return 32.0 + 4.0 * nseg + ksum * (0.5 + 0.5 * blocks);
}

// MFMA row blocks of the wavefront tiles of an m x n output: skinny outputs get
// 16x64 or 64x16 tiles, the rest 32x32 (policy 1: narrow ones too)
inline int wave_mb(int m, int n, int policy) { return m <= 16 ? 1 : policy == 0 && n <= 16 ? 4 : 2; }

// Grid cells (row tile, column tile) of an nr x nc tile grid in patches of
// PATCH x PATCH, patch-major, row-major inside a patch.  The workers of an XCD
// take consecutive list entries, so the tiles that run side by side share
// PATCH operand row bands and PATCH column bands in that XCD's L2 instead of
// each fetching its own.
constexpr int PATCH = 8;
inline std::vector<std::pair<int, int>> patch_order(int nr, int nc) {
  std::vector<std::pair<int, int>> v;
  for (int pr = 0; pr < nr; pr += PATCH)
    for (int pc = 0; pc < nc; pc += PATCH)
      for (int r = pr; r < std::min(nr, pr + PATCH); r++)
        for (int c = pc; c < std::min(nc, pc + PATCH); c++) v.push_back({r, c});
  return v;
}

// Lines of the 128-wide bands of `len` lines, a last band of at least `tail`
// lines included.
inline int wide_bands(int len, int tail) { return len / WIDE_EDGE + (len % WIDE_EDGE >= tail ? 1 : 0); }
inline int wide_lines(int len, int tail) { return std::min(len, wide_bands(len, tail) * WIDE_EDGE); }

// Tiles of an m x n output.  With `wide` it is cut into 128-wide row and
// column bands (a last band of at least `tail` lines is wide too): the wide x
// wide cells in patch order, then the columns beyond the bands, then the rows
// below them, in tiles that small(rows, columns) chooses for those strips;
// without, the whole output gets one kind of tile.
// (wide: the kind of the 128 x 128 tiles, 0 for none.)
template <typename F>
std::vector<Cell> cut_output(int m, int n, int wide, int tail, F &&small) {
  std::vector<Cell> v;
  auto grid = [&](int r0, int c0, int rows, int cols) {
    if (rows <= 0 || cols <= 0) return;
    const int mb = small(rows, cols), tr = tile_rows(mb), tc = tile_cols(mb);
    for (const auto &c : patch_order((rows + tr - 1) / tr, (cols + tc - 1) / tc))
      v.push_back({r0 + c.first * tr, c0 + c.second * tc, mb});
  };
  if (!wide) {
    grid(0, 0, m, n);
    return v;
  }
  const int mw = wide_lines(m, tail), nw = wide_lines(n, tail);
  for (const auto &c : patch_order(wide_bands(m, tail), wide_bands(n, tail))) v.push_back({c.first * WIDE_EDGE, c.second * WIDE_EDGE, wide});
  grid(0, nw, mw, n - nw);
  grid(mw, 0, m - mw, n);
  return v;
}

// ... of an FP64 output; level: the largest kind allowed (0 wavefront tiles,
// 1 64 x 64, 2 128 x 128)
inline bool f64_wide(int m, int n) { return std::min(m, n) >= F64_WIDE_MIN && std::max(m, n) >= F64_WIDE_LONG; }
inline int f64_small(int rows, int cols, int policy, int level) {
  return level > 0 && std::min(rows, cols) >= F64_MACRO_MIN ? MACRO_MB : wave_mb(rows, cols, policy);
}
inline std::vector<Cell> f64_cells(int m, int n, int policy, int level) {
  return cut_output(m, n, level > 1 && f64_wide(m, n) ? F64_WIDE_MB : 0, F64_WIDE_MIN,
                    [&](int rows, int cols) { return f64_small(rows, cols, policy, level); });
}

// The level for a stage of an FP64 plan.  The three kinds of a stage run one
// after the other, each at least as long as its longest tile, so a stage of few
// outputs (a plan cut into many small chunks, or long parts along K) is sooner
// done with smaller tiles that run side by side.  Estimated from the tiles'
// costs (tile_cost) at the times measured for a K row of a whole tile, alone and
// with all work groups that fit on the chip at once.  Second stage of L=36,
// D=512 (sectors up to 137): in 64 MiB chunks 36.3 ms with all kinds, 13.8 with
// wavefront tiles (estimated 38.0 and 14.2); in one chunk 5.1 and 7.0 (5.0, 7.8).
// Sums are in the same order either way.
class TileLevel {
 public:
  // `copies` outputs of m x n, each summing nseg segments of k rows in all
  // (plans have some 10^5 first-stage outputs: shifts only, and outputs too
  // narrow for work-group tiles are counted once for all levels)
  void add(int m, int n, int nseg, double k, double copies, int policy) {
    const double each = 32.0 + 4.0 * nseg;
    auto part = [&](Kind &x, int rows, int cols, int r, int c) {   // tiles of 2^r x 2^c
      if (rows <= 0 || cols <= 0) return;
      auto blocks = [](int rows_, int cols_) { return (double)((rows_ + 15) >> 4) * ((cols_ + 15) >> 4); };
      const double share = 0.5 * k / (1 << (r + c - 8));
      const double tiles = (double)((rows + (1 << r) - 1) >> r) * ((cols + (1 << c) - 1) >> c);
      x.sum += copies * (tiles * (each + 0.5 * k) + share * blocks(rows, cols));
      x.top = std::max(x.top, each + 0.5 * k + share * blocks(std::min(rows, 1 << r), std::min(cols, 1 << c)));
    };
    auto wave = [&](Kind &x, int rows, int cols) {
      const int mb = wave_mb(rows, cols, policy);
      part(x, rows, cols, mb == 1 ? 4 : mb == 2 ? 5 : 6, mb == 1 ? 6 : mb == 2 ? 5 : 4);
    };
    if (std::min(m, n) < F64_MACRO_MIN) return wave(narrow, m, n);
    auto small = [&](int level, int rows, int cols) {
      if (std::min(rows, cols) >= F64_MACRO_MIN) part(kinds[level][1], rows, cols, 6, 6);
      else if (rows > 0 && cols > 0) wave(kinds[level][2], rows, cols);
    };
    wave(kinds[0][2], m, n);
    small(1, m, n);
    if (!f64_wide(m, n)) return small(2, m, n);
    const int mw = wide_lines(m, F64_WIDE_MIN), nw = wide_lines(n, F64_WIDE_MIN);
    part(kinds[2][0], mw, nw, 7, 7);
    small(2, mw, n - nw);
    small(2, m - mw, n);
  }
  // the usual level 2 unless another one is expected to take less than three
  // quarters of its time
  int level() const {
    // us per K row: a tile alone, and all together: 512 wide tiles at once take
    // 0.30, 1024 64 x 64 ones 0.17, 4096 wavefront ones 0.34; 8 us a launch
    constexpr double ALONE[3] = {0.16, 0.07, 0.076}, BUSY[3] = {0.30 / 512, 0.17 / 1024, 0.34 / 4096};
    double t[3] = {0.0, 0.0, 0.0};
    for (int l = 0; l < 3; l++)
      for (int k = 0; k < 3; k++) {
        const double sum = kinds[l][k].sum + (k == 2 ? narrow.sum : 0.0);
        const double top = k == 2 ? std::max(kinds[l][2].top, narrow.top) : kinds[l][k].top;
        if (sum > 0.0) t[l] += 8.0 + std::max(top * ALONE[k], sum * BUSY[k]);
      }
    const int best = t[0] < t[1] ? 0 : 1;
    return t[best] < 0.75 * t[2] ? best : 2;
  }

 private:
  struct Kind { double sum = 0.0, top = 0.0; } kinds[3][3], narrow;   // by level; wide, 64 x 64, wavefront
};

// Device copy of FP64 segments: offsets in bytes, absolute addresses where the
// operand lies in an operator array (base BASE_OPS + k at bases[k], whatever
// its alignment), so that the kernels need no look-up between a descriptor and
// its loads; the strides of the walk along K are filled in.
inline std::vector<Seg> resolve_bases(std::vector<Seg> segs, const double *const *bases) {
  auto bytes = [&](int base, int64_t off) {
    return (int64_t)sizeof(double) * off + (base >= BASE_OPS ? (int64_t)(uintptr_t)bases[base - BASE_OPS] : 0);
  };
  for (Seg &S : segs) {
    S.a_off = bytes(S.a_base, S.a_off);
    S.b_off = bytes(S.b_base, S.b_off);
    const int64_t dp = 4 / S.a_kb, dk = 4 % S.a_kb;
    S.da = dp * S.a_p + dk * S.a_k;
    S.ea = S.a_p - S.a_kb * S.a_k;
    S.db = dp * S.b_pk + dk * S.b_k;
    S.eb = S.b_pk - S.b_kb * S.b_k;
  }
  return segs;
}

// One work item: a (16*mb) x (64/mb) tile of an m x n output block (rows
// i0.., columns j0..) accumulated over segments seg0..seg0+nseg-1 and stored
// at C + (ci0 + i) + (cj0 + j) * ldc (column-major) or at
// C + (ci0 + i) * ldc + (cj0 + j) (rowmajor) (C += or C =).
struct Tile {
  int64_t c_off;
  int64_t ldc;
  int32_t c_base;
  int32_t m, n, i0, j0;
  int32_t ci0, cj0;
  int32_t mb;           // MFMA row blocks: 1, 2 or 4 (column blocks 4 / mb)
  int32_t seg0, nseg;
  int32_t nid;          // identity segments, the first ones of the tile
  int16_t accumulate;   // 1: C += acc, 0: C = acc
  int16_t rowmajor;     // output layout, see above
};

// Transposed copy of one operator record: npos column-major rows x cols
// blocks at off become cols x rows blocks at the same offset.
struct TransJob {
  int64_t off;
  int32_t rows, cols, npos, pad;
};

// Deterministic sum of the partial tiles of one output tile into Y.
struct Reduce {
  int64_t y_off, ldc;
  int64_t part_off;     // first partial; partial p at part_off + p * tm * tn (column-major, ld tm)
  int32_t m, n, i0, j0, tm, tn, nparts, pad;
};

// Diagonal of H_eff: diag[off + i + j*m] += s * dA_i * dD_j over a block's list
struct DiagTerm {
  int64_t a_off, d_off;       // diagonal element base offsets
  int64_t a_step, d_step;     // stride between consecutive diagonal elements
  double s;
  int32_t a_base, d_base;     // -1: identity
};
struct DiagBlock {
  int64_t off;
  int32_t m, n;
  int32_t t0, nt;
};

// One dressed position: dst[0:n] = sum_t alpha[t] * src[src_off[t] + 0:n]
struct DressItem {
  int64_t dst_off, n;
  int32_t t0, t1;
  int32_t src_base, dst_base;
};

// ---------------------------------------------------------------- split BF16
// Fixed-point slicing (Ozaki-style): a line x (row of an A operand or column
// of a B operand, over its K range) is scaled by 2^-e with e the smallest
// integer such that max|x| <= 2^e, then cut into s integer digits of SLICE_BITS
// bits, x = 2^e sum_t a_t 2^(-8(t+1)) + O(2^(e-8s)), |a_0| <= 256, |a_t| <= 128.
// Slice t stores a_t 2^(-8t), exact in BF16 (at most 8 significant bits), so
// that a product of slices t and u already carries the relative weight
// 2^(-8(t+u)) of its group d = t + u and every group folds with 2^-16.  A line's
// K range is cut into position blocks padded to a multiple of 8 with zeros.
// Lines are stored in panels of SLICE_PANEL: inside a panel of h lines (the last
// one may have fewer), chunk c of eight K values, slice t and line l lie at
// ((c s + t) h + l) 8 -- the operand order of the MFMAs, so that the 32 lines a
// wavefront loads for one chunk and slice are one run of 512 bytes.  Stored line
// by line, such a load took 64 pieces of 16 bytes from as many cache lines, and
// these requests bound the tiles: H.psi at L = 54, D = 768, s = 5 took 96.7 ms,
// of which 37.2 in the first stage's wide tiles (18.1 now; in all 69.2 ms), and
// slicing its operators at plan creation took 137 ms (11 now).
constexpr int SLICE_BITS = 8;
// Slice products accumulate in slice_groups(s) FP32 sums: groups d = t + u
// below s - 3 each in its own sum, exact, and all groups d >= s - 3 in one
// more sum (for s <= 3 that is the only one).  Per k an exact group d is at
// most 2^16 (d <= 1) or (d + 3) 2^14 (d >= 2) in units of its resolution
// 2^(-8d), so over split_fold_k(s) terms its sum stays an integer (in those
// units) below 2^24: exact in FP32.  The merged sum is rounded, but its terms
// weigh at most about 2^(-8(s-3)+1) of group 0, so FP32 rounding (2^-24) puts
// its error at the level of the truncation after s digits (2^-8s).  Every
// split_fold_k(s) terms of K the sums are folded into FP64.
constexpr int slice_groups(int ns) { return ns <= 3 ? 1 : ns - 2; }
constexpr int split_fold_k(int ns) { return ns <= 5 ? 256 : 128; }

// One slicing job: lines L < nl, position blocks p < npos of kb valid entries
// (padded to kbp); with rho = L % nrho and q = L / nrho the source x(L, p, kk)
// is at src[src_off + q*s_q + rho*s_rho + p*s_pos + kk*s_k]; the slices start
// at element dst_off s (panel layout, slice_index), the exponent of line L is
// at exps[exp_off + L].
struct SliceJob {
  int64_t src_off, s_q, s_rho, s_pos, s_k;
  int64_t dst_off, exp_off;
  int32_t src_base, dst_buf;
  int32_t nl, nrho, npos, kb, kbp, pad;
};
constexpr int SLICE_PANEL = 32;
// Slicing work item: panel `panel` of job `job`; of a stripe, its chunks
// [c0, c0 + TSLICE_CHUNKS).
struct SliceItem {
  int32_t job, panel, c0;
};
constexpr int TSLICE_CHUNKS = 64;

// Split segment (same role as Seg): A lines are operand rows, B lines operand
// columns.  The output's row i is line a_line0 + i of a_nl, its K index k is a_k0 + k
// of lines of a_ld; exponents at a_exp + i.
struct SegS {
  int64_t a_off, a_ld, a_exp;
  int64_t b_off, b_ld, b_exp;
  int32_t a_buf, b_buf;
  int32_t a_line0, a_nl, a_k0;
  int32_t b_line0, b_nl, b_k0;
  int32_t K;          // padded K (multiple of 8); 0 for an identity segment
  int32_t t_nb;       // first-stage segments: stripe columns per slot (line = column mod t_nb)
  int64_t t_exp;      // first-stage segments: exponent offset of the stripe's lines, else -1
};

// slice buffers: 0 operator records (plan), 1 psi rows, 2 psi columns, 3 stripes
enum { SBUF_OPS = 0, SBUF_PSIR = 1, SBUF_PSIC = 2, SBUF_T = 3, N_SBUF = 4 };

struct SliceBufs {
  uint16_t *data[N_SBUF];     // bf16 bit patterns, slices interleaved (slice_index)
  int32_t *exps[N_SBUF];
};
// position of slice t of K index k of line L, for lines of length ld (a multiple
// of 8), nl of them, stored from element off s on
__host__ __device__ inline int64_t slice_index(int64_t off, int64_t ld, int nl, int64_t L, int64_t k, int t, int s) {
  const int64_t p0 = L - L % SLICE_PANEL;
  const int64_t h = nl - p0 < SLICE_PANEL ? nl - p0 : SLICE_PANEL;
  return (off + p0 * ld) * s + ((k / 8 * s + t) * h + (L - p0)) * 8 + k % 8;
}


// bookkeeping that lets the split-precision plan mirror the FP64 segments
struct StripeInfo {
  int prob, E, rec, adj, dress;
  int64_t off;
  int dL, dRin, dRout, nslots;
  int first_slot_pos;          // unused
};
struct Seg1Info { int stripe, s0, pD0; };
struct Seg2Info { int prob, E, stripe, slot0, recA, adjA, pA0, run; };

struct Chunk {
  std::vector<StripeInfo> stripes;
  std::vector<Seg1Info> s1info;
  std::vector<Seg2Info> s2info;
  std::vector<Seg> seg1, seg2;
  std::vector<Tile> tile1, tile2;       // one wavefront per tile
  std::vector<Tile> tile1m, tile2m;     // work-group (macro) tiles
  std::vector<Tile> tile1x, tile2x;     // wide work-group tiles
  XcdQueues q1{}, q2{}, q1m{}, q2m{}, q1x{}, q2x{};   // per-XCD ranges of the six lists
  std::vector<Reduce> red2;
  Seg *d_seg1 = nullptr, *d_seg2 = nullptr;
  Tile *d_tile1 = nullptr, *d_tile2 = nullptr;
  Tile *d_tile1m = nullptr, *d_tile2m = nullptr;
  Tile *d_tile1x = nullptr, *d_tile2x = nullptr;
  Reduce *d_red2 = nullptr;
  double flops1 = 0.0, flops2 = 0.0;    // algorithmic flops of each stage
  double flops1m = 0.0, flops2m = 0.0;  // ... of its work-group tiles
  double flops1x = 0.0, flops2x = 0.0;  // ... of its wide tiles
  double flops1w = 0.0, flops2w = 0.0;  // ... of its wavefront tiles
  int64_t part_elems = 0;               // partial-tile buffer needed
  // split precision (filled only for split plans)
  std::vector<SegS> sseg1, sseg2;
  std::vector<SliceJob> tjobs;          // stripe slicing after the first stage
  std::vector<SliceItem> titems;        // its work items
  SegS *d_sseg1 = nullptr, *d_sseg2 = nullptr;
  SliceJob *d_tjobs = nullptr;
  SliceItem *d_titems = nullptr;
  int64_t t_elems = 0, t_exps = 0;
};

constexpr int TILE = 32;      // nominal tile edge (tiles are 16*mb x 64/mb)
constexpr int WAVES = 4;      // wavefronts per workgroup (one work item each)
constexpr int KPART = 2048;   // target summed K of one second-stage work item
// default cap of the stripe workspace (288 GB of HBM hold the largest plans in one chunk)
constexpr int64_t DEFAULT_WORKSPACE = (int64_t)64 << 30;

// y := 0, and the counters of the first tile launch that follows (may be NULL)
void launch_zero(double *y, int64_t n, int32_t *counters, void *stream);
void launch_dress(const DressItem *items, int nitems, const int64_t *src_off, const double *alpha,
                  const double *const *bases, double *dst, void *stream);
// tiles from per-XCD queues; flops: of the list; qs: QUEUE_INTS ints of device
// memory (QueueSets)
void launch_tiles_f64(int stage, const Tile *tiles, const Seg *segs, int ntiles, double flops, const XcdQueues &q,
                      QueueSets &qs, const double *psi, double *y, double *work, double *part, void *stream);
// 128 x 128 (mb == F64_WIDE_MB) or 64 x 64 (MACRO_MB) FP64 tiles of whole work groups
void launch_wg_tiles_f64(int stage, int mb, const Tile *tiles, const Seg *segs, int ntiles, double flops, const XcdQueues &q,
                         QueueSets &qs, const double *psi, double *y, double *work, double *part, void *stream);

// NXCD contiguous ranges of a tile list with about equal summed cost
inline XcdQueues xcd_queues(const double *cost, int n) {
  XcdQueues q{};
  double tot = 0.0, acc = 0.0;
  for (int i = 0; i < n; i++) tot += cost[i];
  int i = 0;
  for (int x = 1; x < NXCD; x++) {
    while (i < n && acc + 0.5 * cost[i] < tot * x / NXCD) acc += cost[i++];
    q.start[x] = i;
  }
  q.start[NXCD] = n;
  return q;
}

// An FP64 tile list sorted by kind (wide, 64 x 64, wavefront tiles), each kind
// by falling cost, with its queues; flops: 2 (rows) (columns) K of its tiles.
struct KindLists {
  int first[4] = {0, 0, 0, 0};   // of each kind; first[3]: length
  double flops[3] = {0.0, 0.0, 0.0};
  XcdQueues q[3];
};
inline KindLists sort_by_kind(std::vector<Tile> &tiles, const std::vector<double> &cost, const std::vector<Seg> &segs) {
  auto kind = [&](int i) { return tiles[i].mb == F64_WIDE_MB ? 0 : tiles[i].mb == MACRO_MB ? 1 : 2; };
  std::vector<int> ord(tiles.size());
  for (size_t i = 0; i < ord.size(); i++) ord[i] = (int)i;
  std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) {
    return kind(a) != kind(b) ? kind(a) < kind(b) : cost[a] > cost[b];
  });
  KindLists L;
  std::vector<Tile> t(tiles.size());
  std::vector<double> c(tiles.size());
  for (size_t i = 0; i < ord.size(); i++) {
    const int k = kind(ord[i]);
    t[i] = tiles[ord[i]];
    c[i] = cost[ord[i]];
    L.first[k + 1] = (int)i + 1;
    const double area = (double)std::min(tile_rows(t[i].mb), t[i].m - t[i].i0) * std::min(tile_cols(t[i].mb), t[i].n - t[i].j0);
    for (int e = 0; e < t[i].nseg; e++) L.flops[k] += 2.0 * area * segs[t[i].seg0 + e].K;
  }
  for (int k = 0; k < 3; k++) {
    L.first[k + 1] = std::max(L.first[k], L.first[k + 1]);
    L.q[k] = xcd_queues(c.data() + L.first[k], L.first[k + 1] - L.first[k]);
  }
  tiles.swap(t);
  return L;
}
// the launches of such a list
inline void launch_lists_f64(int stage, const Tile *tiles, const Seg *segs, const KindLists &L, QueueSets &qs,
                             const double *psi, double *y, double *work, double *part, void *stream) {
  for (int k = 0; k < 2; k++)
    launch_wg_tiles_f64(stage, k == 0 ? F64_WIDE_MB : MACRO_MB, tiles + L.first[k], segs, L.first[k + 1] - L.first[k],
                        L.flops[k], L.q[k], qs, psi, y, work, part, stream);
  launch_tiles_f64(stage, tiles + L.first[2], segs, L.first[3] - L.first[2], L.flops[2], L.q[2], qs, psi, y, work, part,
                   stream);
}
void launch_reduce(const Reduce *red, int nred, const double *part, double *y, void *stream);
void launch_transpose(const TransJob *jobs, int njobs, const double *src, double *dst, void *stream);
void launch_diag(const DiagBlock *blocks, const DiagTerm *terms, int nblocks,
                 const double *const *bases, double *diag, void *stream);

}  // namespace dmrg

namespace dmrg {
void launch_slices(const SliceJob *jobs, const SliceItem *items, int nitems, int nslices, const double *const *bases,
                   const double *psi, const double *work, SliceBufs bufs, void *stream);
// stripe slicing with line exponents already in place (the first stage's
// epilogue takes their maxima with atomicMax; sentinel INT_MIN = all zero)
void launch_tslices(const SliceJob *jobs, const SliceItem *items, int nitems, int nslices, const double *work,
                    SliceBufs bufs, void *stream);
void launch_fill_int(int32_t *p, int64_t n, int32_t v, void *stream);
// scratch memory of one H.psi: byte offsets of the stripe workspace, partial
// tiles, stripe slices, stripe exponents and work-queue counters; returns the
// total bytes
constexpr int SCRATCH_REGIONS = 5;
int64_t plan_scratch_layout(const dmrg_plan_t *p, int64_t off[SCRATCH_REGIONS]);
// one H.psi with that scratch memory at base (device address)
int enqueue_scratch(dmrg_plan_t *p, const double *psi, double *hpsi, void *stream, char *base);
// wavefront tiles (one tile per wavefront) from per-XCD queues
void launch_tiles_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles,
                        double flops, const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                        const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream);
// work-group (MACRO_MB) tiles from per-XCD queues
void launch_macro_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles, double flops,
                        const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                        const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream);
// wide (WIDE_MB) tiles, s <= WIDE_MAX_SLICES, same queue protocol
void launch_wide_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles, double flops,
                       const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                       const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream);

}  // namespace dmrg
