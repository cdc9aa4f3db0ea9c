// FP64 MFMA kernels for the grouped stripe products of H.psi.
//
// Every H.psi is two stages.  The first computes, for each wavefunction block X
// and run of right-block operator positions, T = X [op(D_1) ... op(D_c)]
// (positions concatenated along N).  The second accumulates
// Y_F += sum v [A_1 ... A_c] [T_1; ...; T_c] for every output block F.  Output
// tiles are owned by work items; a tile whose segment list is long is split
// into parts (split K) that write partial tiles, summed afterwards in a fixed
// order, so the result is bitwise reproducible.  Large outputs are cut into
// tiles of whole work groups, staged through LDS (wg_f64_kernel); the rest into
// tiles of one wavefront (stage_f64_kernel), (16 mb) x (64/mb) as mb x (4/mb)
// v_mfma_f64_16x16x4 products with operands in registers several K steps ahead.
// Lane layout of v_mfma_f64_16x16x4f64 (lane l, accumulator element r):
// A[l%16][l/16], B[l/16][l%16], D[l/16 + 4r][l%16].
#include <hip/hip_runtime.h>
#include <algorithm>
#include "plan.hpp"
#include "queue.hpp"

namespace dmrg {

typedef double v4d __attribute__((ext_vector_type(4)));


// Operand pointers come from a table of generic pointers; every one of them
// addresses device global memory, and saying so lets the compiler emit global
// (not flat) loads, whose counters allow waiting for the oldest loads only --
// otherwise each wait drains every load in flight and the prefetch is lost.
typedef const double __attribute__((address_space(1))) *gcptr;
typedef double __attribute__((address_space(1))) *gptr;
typedef const char __attribute__((address_space(1))) *gbptr;
__device__ __forceinline__ double gld(const double *p) { return *(gcptr)p; }


// Operands lie in psi, in the stripe workspace or in operator arrays, which are
// addressed absolutely (resolve_bases; off in bytes).  First-stage tiles are
// stored in the workspace, second-stage ones in the output or among the partial
// tiles.
__device__ __forceinline__ const double *seg_ptr(int id, int64_t off, const double *psi, const double *work) {
  return (const double *)((const char *)(id == BASE_PSI ? psi : id == BASE_WORK ? work : nullptr) + off);
}
template <int STAGE>
__device__ __forceinline__ double *out_ptr(int id, double *y, double *work, double *part) {
  return STAGE == 1 ? work : id == BASE_Y ? y : part;
}

// descriptors do not change during a launch: scalar loads
typedef const Seg __attribute__((address_space(4))) CSegF;

// Wavefront tiles.  The stages have kernels of their own, each holding only
// what its segments need: a first-stage tile has one segment, one position
// along K and column positions of B, and is stored row-major; a second-stage
// (or density-matrix) tile sums many segments with positions along K and is
// stored column-major.  With both in one kernel and the walk over segments
// inlined for every buffer the code took 61 KB, as much as the instruction
// cache, and wavefronts of short tiles spent half their time waiting for
// instructions.  MB x NB are the MFMA blocks inside the output (a 16 x 64
// tile of a 3 x 7 output is one block, not four).
//
// Each operand's K steps (four rows) are DEPTH deep in flight in registers:
// while the matrix core works on one, the loads of the step DEPTH later fill
// its buffer.  A lane whose next row lies past the end of K stays on its last
// row; such rows are scaled by zero instead of s (the operands are finite).
// Lanes outside the output read its last line (never stored), so no load
// depends on a condition.  Scheduling barriers keep each buffer's refill in
// program order: the oldest buffer's loads are always the ones waited for.
template <int MB, int NB>
struct StepF64 {
  double a[MB], b[NB];
};

template <int MB, int NB>
__device__ __forceinline__ void mma_f64(v4d (&acc)[MB][NB], const StepF64<MB, NB> &x, double sk) {
  double a[MB], b[NB];
#pragma unroll
  for (int bi = 0; bi < MB; bi++) a[bi] = sk * x.a[bi];
#pragma unroll
  for (int bj = 0; bj < NB; bj++) b[bj] = x.b[bj];
#pragma unroll
  for (int bi = 0; bi < MB; bi++)
#pragma unroll
    for (int bj = 0; bj < NB; bj++)
      acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[bi], b[bj], acc[bi][bj], 0, 0, 0);
}

// first stage: T = X op(D), one segment
template <int MB, int NB>
__device__ __forceinline__ void item1_f64(const Tile &T, const Seg *__restrict__ segs, const double *psi, double *y,
                                          double *work, double *part, int r16, int q4) {
  constexpr int DEPTH = 4;
  v4d acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; a++)
#pragma unroll
    for (int b = 0; b < NB; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
  const int mrem = T.m - T.i0, nrem = T.n - T.j0;
  CSegF &S = ((const CSegF *)segs)[T.seg0];
  const int K = S.K;
  const double s = S.s;
  int k = min(q4, K - 1);
  const double *pa[MB], *pb[NB];
  const double *A = seg_ptr(S.a_base, S.a_off, psi, work), *B = seg_ptr(S.b_base, S.b_off, psi, work);
#pragma unroll
  for (int bi = 0; bi < MB; bi++)
    pa[bi] = A + operand_offset(0, 0, k, S.a_k, T.i0 + min(16 * bi + r16, mrem - 1), S.a_i);
#pragma unroll
  for (int bj = 0; bj < NB; bj++) {
    const unsigned n = T.j0 + min(16 * bj + r16, nrem - 1);
    unsigned pn = 0;
    if (S.b_nb < T.n) pn = n / (unsigned)S.b_nb;
    pb[bj] = B + operand_offset(pn, S.b_pn, k, S.b_k, n - pn * S.b_nb, S.b_n);
  }
  k = q4;
  const int64_t da = 4 * S.a_k, db = 4 * S.b_k;
  StepF64<MB, NB> st[DEPTH];
  auto refill = [&](StepF64<MB, NB> &x) {
#pragma unroll
    for (int bi = 0; bi < MB; bi++) x.a[bi] = gld(pa[bi]);
#pragma unroll
    for (int bj = 0; bj < NB; bj++) x.b[bj] = gld(pb[bj]);
    k += 4;
    if (k < K) {
#pragma unroll
      for (int bi = 0; bi < MB; bi++) pa[bi] += da;
#pragma unroll
      for (int bj = 0; bj < NB; bj++) pb[bj] += db;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < DEPTH; u++) refill(st[u]);
  for (int k0 = 0; k0 < K; k0 += 4 * DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; u++) {
      if (k0 + 4 * u < K) mma_f64<MB, NB>(acc, st[u], k0 + 4 * u + q4 < K ? s : 0.0);
      refill(st[u]);
    }
  }
  double *C = out_ptr<1>(T.c_base, y, work, part) + T.c_off;
#pragma unroll
  for (int bi = 0; bi < MB; bi++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = 16 * bi + q4 + 4 * r;
      gptr c = (gptr)(C + (int64_t)(T.ci0 + i) * T.ldc + (T.cj0 + r16));
#pragma unroll
      for (int bj = 0; bj < NB; bj++)
        if (i < mrem && 16 * bj + r16 < nrem) c[16 * bj] = acc[bi][bj][r];
    }
}

// second stage: the K steps of all segments form one sequence, loaded ahead
// across segment boundaries.  Tiles of small sectors sum hundreds of segments
// of a few rows (L=8: 138 of 8 rows); with the loads started anew at every
// segment each one cost its descriptor's and its operands' latency, 3.3 us.
// The next segment's descriptor is read while the current one is walked.
// Every lane walks its own row: `k`, its row `kk` in the position and its two
// operand pointers move by the same uniform strides, with one more at a
// position boundary (both operands have the same positions).
template <int MB, int NB, int DEPTH>
__device__ __forceinline__ void item2_f64(const Tile &T, const Seg *__restrict__ segs, const double *psi, double *y,
                                          double *work, double *part, int r16, int q4) {
  v4d acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; a++)
#pragma unroll
    for (int b = 0; b < NB; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
  const int mrem = T.m - T.i0, nrem = T.n - T.j0;
  const CSegF *cs = (const CSegF *)segs + T.seg0;
  // identity left operators (the first segments): tile += s * B restricted to
  // the tile (one position, K == rows).  (The lane's coordinates pass through
  // an empty asm so that offsets derived from them are not kept in registers
  // during the loop below.)
  asm volatile("" : "+v"(r16), "+v"(q4));
  for (int si = 0; si < T.nid; si++) {
    CSegF &S = cs[si];
    const double *B = seg_ptr(S.b_base, S.b_off, psi, work) + T.i0 * S.b_k + T.j0 * S.b_n;
    const double s = S.s;
    double v[MB][NB][4];
#pragma unroll
    for (int bi = 0; bi < MB; bi++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const uint32_t row = min(16 * bi + q4 + 4 * r, mrem - 1);
#pragma unroll
        for (int bj = 0; bj < NB; bj++)
          v[bi][bj][r] = gld(B + operand_offset(0, 0, row, S.b_k, min(16 * bj + r16, nrem - 1), S.b_n));
      }
#pragma unroll
    for (int bi = 0; bi < MB; bi++)
#pragma unroll
      for (int bj = 0; bj < NB; bj++)
#pragma unroll
        for (int r = 0; r < 4; r++) acc[bi][bj][r] += s * v[bi][bj][r];
  }
  asm volatile("" : "+v"(r16), "+v"(q4));
  if (T.nid < T.nseg) {
    // uniform state of the walk ...
    int si = T.nid, K = 0, kb = 1, dk = 0, k0 = 0;
    double s = 0.0;
    int64_t da = 0, ea = 0, db = 0, eb = 0;   // per step, extra at a position boundary
    // ... and this lane's
    int k = 0, kk = 0;
    const double *pa = nullptr, *pb = nullptr;
    uint32_t ao[MB], bo[NB];   // lines of the further blocks, elements past the first one's
    const unsigned i0 = min(r16, mrem - 1), j0 = min(r16, nrem - 1);
    struct {
      int64_t a_off, b_off, a_p, da, ea, db, eb;
      double s;
      uint32_t a_i, a_k, b_pk, b_k, b_n;   // strides below 2^32 (see operand_offset)
      int a_base, b_base, K, kb;
    } nx;   // descriptor of segment si
    auto fetch_desc = [&]() {
      CSegF &S = cs[si];
      nx.a_off = S.a_off; nx.b_off = S.b_off;
      nx.a_p = S.a_p; nx.a_i = (uint32_t)S.a_i; nx.a_k = (uint32_t)S.a_k;
      nx.b_pk = (uint32_t)S.b_pk; nx.b_k = (uint32_t)S.b_k; nx.b_n = (uint32_t)S.b_n;
      nx.da = S.da; nx.ea = S.ea; nx.db = S.db; nx.eb = S.eb;
      nx.s = S.s;
      nx.a_base = S.a_base; nx.b_base = S.b_base;
      nx.K = S.K; nx.kb = S.a_kb;
    };
    auto open = [&]() {
      K = nx.K;
      kb = nx.kb;
      s = nx.s;
      k0 = 0;
      dk = kb > 4 ? 4 : kb == 3 ? 1 : 0;   // 4 mod kb
      da = nx.da;
      ea = nx.ea;
      db = nx.db;
      eb = nx.eb;
      k = min(q4, K - 1);
      const unsigned p = kb >= 4 ? 0 : kb == 3 ? (k == 3) : kb == 2 ? k >> 1 : k;
      kk = k - p * kb;
      pa = seg_ptr(nx.a_base, nx.a_off, psi, work) + operand_offset(p, nx.a_p, kk, nx.a_k, T.i0 + i0, nx.a_i);
      pb = seg_ptr(nx.b_base, nx.b_off, psi, work) + operand_offset(p, nx.b_pk, kk, nx.b_k, T.j0 + j0, nx.b_n);
      k = q4;
#pragma unroll
      for (int bi = 1; bi < MB; bi++) ao[bi] = (uint32_t)(min(16 * bi + r16, mrem - 1) - i0) * nx.a_i;
#pragma unroll
      for (int bj = 1; bj < NB; bj++) bo[bj] = (uint32_t)(min(16 * bj + r16, nrem - 1) - j0) * nx.b_n;
      si++;
      if (si < T.nseg) fetch_desc();
    };
    StepF64<MB, NB> st[DEPTH];
    double ss[DEPTH];   // scale and rows left of each buffered step (rows <= 0: none)
    int rem[DEPTH];
    fetch_desc();
    open();
#pragma unroll
    for (int u = 0; u < DEPTH; u++) rem[u] = 0;
    // rounds of DEPTH steps: the first one only fills the buffers, the last one
    // is the one whose first refill found no step
    do {
#pragma unroll
      for (int u = 0; u < DEPTH; u++) {
        if (rem[u] > 0) mma_f64<MB, NB>(acc, st[u], q4 < rem[u] ? ss[u] : 0.0);
        if (k0 >= K && si < T.nseg) open();
        ss[u] = s;
        rem[u] = K - k0;
        st[u].a[0] = gld(pa);
#pragma unroll
        for (int bi = 1; bi < MB; bi++) st[u].a[bi] = gld(pa + ao[bi]);
        st[u].b[0] = gld(pb);
#pragma unroll
        for (int bj = 1; bj < NB; bj++) st[u].b[bj] = gld(pb + bo[bj]);
        k0 += 4;
        k += 4;
        if (k < K) {
          pa += da;
          pb += db;
          kk += dk;
          if (kk >= kb) {
            kk -= kb;
            pa += ea;
            pb += eb;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } while (rem[0] > 0);
  }
  double *C = out_ptr<2>(T.c_base, y, work, part) + T.c_off;
#pragma unroll
  for (int bj = 0; bj < NB; bj++) {
    const int j = 16 * bj + r16;
    gptr c = (gptr)(C + (int64_t)(T.cj0 + j) * T.ldc + (T.ci0 + q4));
#pragma unroll
    for (int bi = 0; bi < MB; bi++)
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (16 * bi + 4 * r + q4 < mrem && j < nrem)
          c[16 * bi + 4 * r] = T.accumulate ? c[16 * bi + 4 * r] + acc[bi][bj][r] : acc[bi][bj][r];
  }
}

// One launch per stage: every wavefront takes tiles from the per-XCD queues
// of the stage's cost-sorted list and runs the work item of the tile's shape.
// Four wavefronts per SIMD (at most 128 registers, no spills).
constexpr int F64_GRID = 256 * 4;   // resident work groups
template <int STAGE>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(4, 4))) stage_f64_kernel(
    const Tile *__restrict__ tiles, const Seg *__restrict__ segs, XcdQueues q, int32_t *__restrict__ counters,
    int32_t *__restrict__ next_counters, int chunk, const double *__restrict__ psi, double *__restrict__ y,
    double *__restrict__ work, double *__restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, q4 = lane >> 4;
  clear_counters(next_counters);
  // the tile index is the same for the whole wavefront: saying so makes the
  // descriptors scalar loads and the K loops uniform (no exec masking)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  WorkQueue wq(q, counters, (int)(blockIdx.x / NXCD) * WAVES + wave, (int)(gridDim.x / NXCD) * WAVES, chunk);
  do {
    const int tend = __builtin_amdgcn_readfirstlane(wq.tend), step = __builtin_amdgcn_readfirstlane(wq.step);
    for (int t = __builtin_amdgcn_readfirstlane(wq.t); t < tend; t += step) {
      if (t + step >= tend) wq.request(lane == 0);
      const Tile T = tiles[t];
      const int nbi = min((T.m - T.i0 + 15) / 16, T.mb), nbj = min((T.n - T.j0 + 15) / 16, 4 / T.mb);
#define ITEM(M, N, D)                                                          \
  if (STAGE == 1) item1_f64<M, N>(T, segs, psi, y, work, part, r16, q4);       \
  else item2_f64<M, N, D>(T, segs, psi, y, work, part, r16, q4);
      if (nbi == 1 && nbj == 1) {
        ITEM(1, 1, 6)
      } else if (nbi == 1 && nbj == 2) {
        ITEM(1, 2, 4)
      } else if (nbi == 1) {
        ITEM(1, 4, 4)
      } else if (T.mb == 2) {
        ITEM(2, 2, 4)
      } else {
        ITEM(4, 1, 4)
      }
#undef ITEM
    }
  } while (wq.next(lane));
}

// ------------------------------------------------------------ work-group tiles
// Output tiles of whole work groups: WM x WN wavefronts, each with MBW x NBW
// MFMA blocks.  The 16 x 16 blocks of the tile go to the wavefronts in turn
// (block row b to wavefront row b % WM, likewise the columns), so that a
// ragged tile leaves every wavefront about the same share; blocks outside the
// output are skipped.  Each 16-wide K step of both operands goes from global
// memory through registers into one of two LDS stages (64 consecutive lines
// of one K per wavefront and load: whole 128-byte lines, K wave-uniform)
// while the step before is computed from the other; the row strides in LDS
// are 16 modulo 32 doubles, which spreads the four K rows of an operand read
// over all banks.
template <int WM_, int WN_, int MBW_, int NBW_, int WAVES_PER_SIMD>
struct WgTile {
  static constexpr int WM = WM_, WN = WN_, MBW = MBW_, NBW = NBW_, EU = WAVES_PER_SIMD;
  static constexpr int BM = 16 * WM * MBW, BN = 16 * WN * NBW, NT = 64 * WM * WN;
  static constexpr int KS = 16, LDA = BM + 16, LDB = BN + 16;
  static constexpr int RA = NT / BM, RB = NT / BN;       // K rows one load of all threads covers
  static constexpr int NA = KS / RA, NB = KS / RB;       // loads per thread and step
  static constexpr int STAGE = KS * (LDA + LDB);         // doubles
  static_assert(BM % 64 == 0 && BN % 64 == 0, "a wavefront's loads have one K");
};
typedef WgTile<2, 4, 4, 2, 4> WideF64;    // 128 x 128
typedef WgTile<2, 2, 2, 2, 4> MacroF64;   // 64 x 64
static_assert(WideF64::BM == WIDE_EDGE && WideF64::BN == WIDE_EDGE, "F64_WIDE_MB tiles");
static_assert(MacroF64::BM == MACRO_EDGE && MacroF64::BN == MACRO_EDGE, "MACRO_MB tiles");

template <typename G, int STAGE>
__device__ __forceinline__ void wg_tile_f64(const Tile &T, const Seg *__restrict__ segs, const double *psi, double *y,
                                            double *work, double *part, double *lds, int wave, int lane) {
  const CSegF *cs = (const CSegF *)segs + T.seg0;
  const int r16 = lane & 15, q4 = lane >> 4;
  const int wr = wave / G::WN, wc = wave % G::WN;
  const int mt = min(G::BM, T.m - T.i0), nt = min(G::BN, T.n - T.j0);
  // blocks of this wavefront inside the output
  const int nbi = max(0, ((mt + 15) / 16 - wr + G::WM - 1) / G::WM);
  const int nbj = max(0, ((nt + 15) / 16 - wc + G::WN - 1) / G::WN);
  v4d acc[G::MBW][G::NBW];
#pragma unroll
  for (int a = 0; a < G::MBW; a++)
#pragma unroll
    for (int b = 0; b < G::NBW; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
  // identity left operators: tile += s * B restricted to the tile (one
  // position, K == rows).  Lanes outside the output read its last row or
  // column, so that no load waits for another.
  // (the lane index passes through an empty asm, here and below, so that the
  // offsets derived from it are not kept in registers during the K loop)
  asm volatile("" : "+v"(lane));
  for (int e = 0; STAGE == 2 && e < T.nid; e++) {
    CSegF &S = cs[e];
    const double *B = seg_ptr(S.b_base, S.b_off, psi, work);
    const double s = S.s;
#pragma unroll
    for (int bi = 0; bi < G::MBW; bi++) {
      double v[G::NBW][4];
#pragma unroll
      for (int bj = 0; bj < G::NBW; bj++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int i = T.i0 + min(16 * (wr + G::WM * bi) + (lane >> 4) + 4 * r, mt - 1);
          const int j = T.j0 + min(16 * (wc + G::WN * bj) + (lane & 15), nt - 1);
          v[bj][r] = gld(B + i * S.b_k + j * S.b_n);
        }
#pragma unroll
      for (int bj = 0; bj < G::NBW; bj++)
#pragma unroll
        for (int r = 0; r < 4; r++) acc[bi][bj][r] += s * v[bj][r];
    }
  }
  asm volatile("" : "+v"(lane));
  int si = T.nid;   // identity segments come first
  if (si < T.nseg) {
    // this thread's line of each operand (lines past the output read the last
    // one, never stored) and its wave-uniform first K row of a step; element e
    // of a thread is row `kr + R e`.  Addresses are a uniform pointer plus the
    // line's 32-bit byte offset (a tile's lines span at most BM a_i or a few
    // positions' blocks of B).  The pointer walks along K by additions, over
    // the position boundaries that both operands share: computing (position,
    // offset) by division cost some 900 scalar instructions per step, as long
    // as its products.
    static_assert(G::BM == G::BN && G::RA * G::NA == G::KS, "both operands have the same rows per thread");
    constexpr int R = G::RA, N = G::NA;
    const int line = (wave * 64 + lane) % G::BM, kr = wave * 64 / G::BM;
    const int il = min(line, mt - 1), jl = T.j0 + min(line, nt - 1);
    double pa[N], pb[N];
    // walk of the segment being loaded: row pointers, row within the position
    const double *wa, *wb;
    int64_t da, ea, db, eb;    // per R rows, extra at a position boundary
    int wk, wkb, wK;
    uint32_t ao, bo;
    auto open = [&](int qi) {
      CSegF &S = cs[qi];
      wK = S.K;
      wkb = S.a_kb;
      int64_t ak = S.a_k, bk = S.b_k;
      if (wkb == 1) {   // one row per position: the rows are the positions
        wkb = wK;
        ak = S.a_p;
        bk = S.b_pk;
      }
      da = R * ak;
      db = R * bk;
      ea = S.a_p - wkb * ak;
      eb = S.b_pk - wkb * bk;
      const int p0 = STAGE == 2 || T.j0 < S.b_nb ? 0 : T.j0 / S.b_nb;
      const int row = min(kr, wK - 1);
      wk = row;
      wa = seg_ptr(S.a_base, S.a_off, psi, work) + (int64_t)T.i0 * S.a_i + row * ak;
      wb = seg_ptr(S.b_base, S.b_off, psi, work) + (int64_t)p0 * S.b_pn + row * bk;
      if (wk >= wkb) {   // kr < R <= 4, positions of at least two rows
        wk -= wkb;
        wa += ea;
        wb += eb;
        if (wk >= wkb) {
          wk -= wkb;
          wa += ea;
          wb += eb;
        }
      }
      ao = 8u * (uint32_t)il * (uint32_t)S.a_i;
      int pn = 0, jn = jl - p0 * S.b_nb;
      if (STAGE == 1 && S.b_nb < T.n && jn >= S.b_nb) {
        pn = jn / S.b_nb;
        jn -= pn * S.b_nb;
      }
      bo = 8u * ((uint32_t)pn * (uint32_t)S.b_pn + (uint32_t)jn * (uint32_t)S.b_n);
    };
    // the step at k0; the walk ends at the first row of the next step, or
    // stays on the segment's last rows (read again for the rows past K)
    auto load = [&](int k0) {
#pragma unroll
      for (int e = 0; e < N; e++) {
        pa[e] = *(gcptr)((gbptr)wa + ao);
        pb[e] = *(gcptr)((gbptr)wb + bo);
        if (k0 + kr + R * (e + 1) < wK) {
          wa += da;
          wb += db;
          wk += R;
          if (STAGE == 2 && wk >= wkb) {
            wk -= wkb;
            wa += ea;
            wb += eb;
            if (R > 2 && wk >= wkb) {
              wk -= wkb;
              wa += ea;
              wb += eb;
            }
          }
        }
      }
    };
    // ... into an LDS stage: A scaled by the segment's factor, K rows past the
    // segment's end as zeros
    auto store = [&](int qi, int k0, double *st) {
      const int K = cs[qi].K;
      const double s = cs[qi].s;
      double *as = st + line, *bs = st + G::KS * G::LDA + line;
#pragma unroll
      for (int e = 0; e < N; e++) {
        const int k = kr + R * e;
        as[k * G::LDA] = k0 + k < K ? s * pa[e] : 0.0;
        bs[k * G::LDB] = k0 + k < K ? pb[e] : 0.0;
      }
    };
    // ksteps K steps of four from stage st, the operands of the next one read
    // while this one's products run.  One path with a uniform branch per
    // block: a separate path for whole tiles made the accumulators live twice.
    auto compute = [&](const double *st, int ksteps) {
      const double *as = st + q4 * G::LDA + 16 * wr + r16, *bs = st + G::KS * G::LDA + q4 * G::LDB + 16 * wc + r16;
#pragma unroll
      for (int kk = 0; kk < G::KS / 4; kk++) {
        if (kk < ksteps) {
          double a[G::MBW], b[G::NBW];
#pragma unroll
          for (int bi = 0; bi < G::MBW; bi++) a[bi] = as[4 * kk * G::LDA + 16 * G::WM * bi];
#pragma unroll
          for (int bj = 0; bj < G::NBW; bj++) b[bj] = bs[4 * kk * G::LDB + 16 * G::WN * bj];
#pragma unroll
          for (int bi = 0; bi < G::MBW; bi++)
#pragma unroll
            for (int bj = 0; bj < G::NBW; bj++)
              if (bi < nbi && bj < nbj)
                acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[bi], b[bj], acc[bi][bj], 0, 0, 0);
        }
      }
    };
    int k0 = 0, cur = 0;
    open(si);
    load(0);
    store(si, 0, lds);
    for (;;) {
      __syncthreads();   // this step is in stage cur, the other stage is free
      const int K = cs[si].K;
      int nsi = si, nk0 = k0 + G::KS;
      if (nk0 >= K) {
        nk0 = 0;
        nsi++;
      }
      const bool more = nsi < T.nseg;
      if (more) {
        if (nsi != si) open(nsi);
        load(nk0);
      }
      __builtin_amdgcn_sched_barrier(0);
      compute(lds + cur * G::STAGE, (min(G::KS, K - k0) + 3) / 4);
      __builtin_amdgcn_sched_barrier(0);
      if (!more) break;
      cur ^= 1;
      store(nsi, nk0, lds + cur * G::STAGE);
      si = nsi;
      k0 = nk0;
    }
  }
  asm volatile("" : "+v"(lane));
  double *C = out_ptr<STAGE>(T.c_base, y, work, part) + T.c_off;
#pragma unroll
  for (int bi = 0; bi < G::MBW; bi++)
#pragma unroll
    for (int bj = 0; bj < G::NBW; bj++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int i = 16 * (wr + G::WM * bi) + (lane >> 4) + 4 * r, j = 16 * (wc + G::WN * bj) + (lane & 15);
        if (i < mt && j < nt) {
          gptr c = (gptr)(STAGE == 1 ? C + (int64_t)(T.ci0 + i) * T.ldc + (T.cj0 + j)
                                     : C + (int64_t)(T.ci0 + i) + (int64_t)(T.cj0 + j) * T.ldc);
          *c = STAGE == 2 && T.accumulate ? *c + acc[bi][bj][r] : acc[bi][bj][r];
        }
      }
}

template <typename G, int STAGE>
__global__ void __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(G::EU, G::EU))) wg_f64_kernel(
    const Tile *__restrict__ tiles, const Seg *__restrict__ segs, XcdQueues q, int32_t *__restrict__ counters,
    int32_t *__restrict__ next_counters, const double *__restrict__ psi,
    double *__restrict__ y, double *__restrict__ work, double *__restrict__ part) {
  __shared__ double lds[2 * G::STAGE];
  // the next tiles, in the padding of the first LDS row (with ints of their own
  // the 64 x 64 tiles would exceed a quarter of the LDS)
  int *taken = (int *)(lds + G::BM);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  clear_counters(next_counters);
  WorkQueue wq(q, counters, (int)(blockIdx.x / NXCD), (int)(gridDim.x / NXCD), 1);
  for (bool more = true; more;) {
    for (; wq.t < wq.tend; wq.t += wq.step) {
      if (wave == 0 && wq.last()) wq.request(lane == 0);
      const Tile T = tiles[__builtin_amdgcn_readfirstlane(wq.t)];
      wg_tile_f64<G, STAGE>(T, segs, psi, y, work, part, lds, wave, lane);
      __syncthreads();   // everyone has read the last LDS stage
    }
    if (wave == 0) {
      more = wq.next(lane);
      if (lane == 0) {
        taken[0] = more ? wq.t : 0;
        taken[1] = more ? wq.tend : -1;
      }
    }
    __syncthreads();
    wq.t = __builtin_amdgcn_readfirstlane(taken[0]);
    wq.tend = __builtin_amdgcn_readfirstlane(taken[1]);
    wq.step = 1;
    more = wq.t < wq.tend;
    __syncthreads();   // everyone has read `taken`
  }
}

// Y tile += sum of its partial tiles, in part order
// one output tile per blockIdx.x (grid-stride), its elements shared by the
// REDUCE_SPLIT blocks along y: the 128 x 128 tiles of wide plans have 16384
// elements, which one block of 256 threads would take alone
constexpr int REDUCE_SPLIT = 16;
__global__ void reduce_kernel(const Reduce *__restrict__ red, int nred, const double *__restrict__ part,
                              double *__restrict__ y) {
  for (int r = blockIdx.x; r < nred; r += gridDim.x) {
    const Reduce R = red[r];
    int mt = min(R.tm, R.m - R.i0);
    int nt = min(R.tn, R.n - R.j0);
    const int64_t ps = (int64_t)R.tm * R.tn;
    for (int e = blockIdx.y * blockDim.x + threadIdx.x; e < mt * nt; e += gridDim.y * blockDim.x) {
      int i = e % mt, j = e / mt;
      double v = 0.0;
      for (int p = 0; p < R.nparts; p++) v += part[R.part_off + (int64_t)p * ps + i + (int64_t)j * R.tm];
      y[R.y_off + (int64_t)(R.i0 + i) + (int64_t)(R.j0 + j) * R.ldc] += v;
    }
  }
}

__global__ void zero_kernel(double *y, int64_t n, int32_t *counters) {
  if (counters) clear_counters(counters);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = 0.0;
}

__global__ void diag_kernel(const DiagBlock *__restrict__ blocks, const DiagTerm *__restrict__ terms,
                            int nblocks, const double *const *__restrict__ bases, double *__restrict__ diag) {
  for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const DiagBlock B = blocks[b];
    int64_t n = (int64_t)B.m * B.n;
    for (int64_t e = threadIdx.x; e < n; e += blockDim.x) {
      int i = (int)(e % B.m), j = (int)(e / B.m);
      double acc = 0.0;
      for (int t = 0; t < B.nt; t++) {
        const DiagTerm T = terms[B.t0 + t];
        double a = T.a_base < 0 ? 1.0 : bases[T.a_base - BASE_OPS][T.a_off + (int64_t)i * T.a_step];
        double d = T.d_base < 0 ? 1.0 : bases[T.d_base - BASE_OPS][T.d_off + (int64_t)j * T.d_step];
        acc += T.s * a * d;
      }
      diag[B.off + e] = acc;
    }
  }
}

// dressed right-block operators (once per plan)
__global__ void dress_kernel(const DressItem *__restrict__ items, int nitems,
                             const int64_t *__restrict__ src_off, const double *__restrict__ alpha,
                             const double *const *__restrict__ bases, double *__restrict__ dst) {
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const DressItem D = items[it];
    const double *src = bases[D.src_base - BASE_OPS];
    for (int64_t e = threadIdx.x; e < D.n; e += blockDim.x) {
      double acc = 0.0;
      for (int t = D.t0; t < D.t1; t++) acc += alpha[t] * src[src_off[t] + e];
      dst[D.dst_off + e] = acc;
    }
  }
}

void launch_dress(const DressItem *items, int nitems, const int64_t *src_off, const double *alpha,
                  const double *const *bases, double *dst, void *stream) {
  if (nitems <= 0) return;
  hipLaunchKernelGGL(dress_kernel, dim3(std::min(nitems, 8192)), dim3(256), 0, (hipStream_t)stream, items,
                     nitems, src_off, alpha, bases, dst);
}

void launch_zero(double *y, int64_t n, int32_t *counters, void *stream) {
  if (n <= 0 && !counters) return;
  int grid = (int)std::min<int64_t>((std::max<int64_t>(n, 1) + 255) / 256, 4096);
  hipLaunchKernelGGL(zero_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, y, n, counters);
}

void launch_tiles_f64(int stage, const Tile *tiles, const Seg *segs, int ntiles, double flops, const XcdQueues &q,
                      QueueSets &qs, const double *psi, double *y, double *work,
                      double *part, void *stream) {
  if (ntiles <= 0) return;
  hipStream_t s = (hipStream_t)stream;
  const int grid = wave_grid(ntiles, F64_GRID, WAVES), chunk = wave_chunk(ntiles, flops);
  const XcdQueues dq = deal(q, grid / NXCD * WAVES, false);
  if (stage == 1)
    hipLaunchKernelGGL(stage_f64_kernel<1>, dim3(grid), dim3(64 * WAVES), 0, s, tiles, segs, dq, qs.cur(), qs.other(),
                       chunk, psi, y, work, part);
  else
    hipLaunchKernelGGL(stage_f64_kernel<2>, dim3(grid), dim3(64 * WAVES), 0, s, tiles, segs, dq, qs.cur(), qs.other(),
                       chunk, psi, y, work, part);
  qs.launch++;
}

template <typename G>
static void launch_wg_f64(int stage, const Tile *tiles, const Seg *segs, int ntiles, double flops, const XcdQueues &q, QueueSets &qs,
                          const double *psi, double *y, double *work, double *part,
                          hipStream_t s) {
  // as many work groups as are resident at once: G::EU wavefronts per SIMD
  const int resident = 256 * (G::EU * 4 * 64 / G::NT);
  const int grid = std::min((ntiles + NXCD - 1) / NXCD * NXCD, resident);
  const XcdQueues dq = deal(q, grid / NXCD, heavy_tiles(ntiles, flops));
  if (stage == 1)
    hipLaunchKernelGGL((wg_f64_kernel<G, 1>), dim3(grid), dim3(G::NT), 0, s, tiles, segs, dq, qs.cur(), qs.other(),
                       psi, y, work, part);
  else
    hipLaunchKernelGGL((wg_f64_kernel<G, 2>), dim3(grid), dim3(G::NT), 0, s, tiles, segs, dq, qs.cur(), qs.other(),
                       psi, y, work, part);
  qs.launch++;
}

void launch_wg_tiles_f64(int stage, int mb, const Tile *tiles, const Seg *segs, int ntiles, double flops, const XcdQueues &q,
                         QueueSets &qs, const double *psi, double *y, double *work,
                         double *part, void *stream) {
  if (ntiles <= 0) return;
  if (mb == F64_WIDE_MB)
    launch_wg_f64<WideF64>(stage, tiles, segs, ntiles, flops, q, qs, psi, y, work, part, (hipStream_t)stream);
  else
    launch_wg_f64<MacroF64>(stage, tiles, segs, ntiles, flops, q, qs, psi, y, work, part, (hipStream_t)stream);
}

void launch_reduce(const Reduce *red, int nred, const double *part, double *y, void *stream) {
  if (nred <= 0) return;
  hipLaunchKernelGGL(reduce_kernel, dim3(std::min(nred, 8192), REDUCE_SPLIT), dim3(256), 0, (hipStream_t)stream, red,
                     nred, part, y);
}

void launch_diag(const DiagBlock *blocks, const DiagTerm *terms, int nblocks, const double *const *bases,
                 double *diag, void *stream) {
  if (nblocks <= 0) return;
  int grid = std::min(nblocks, 4096);
  hipLaunchKernelGGL(diag_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, blocks, terms, nblocks,
                     bases, diag);
}

// dst block (c, r) = src block (r, c) for every position of every job.  The
// blocks along y share a job's 32 x 32 pieces, which pass through LDS so that
// both sides are runs of 256 bytes; blocks of fewer than 16 rows or columns go
// element by element.  One work group per job, writing 8 bytes at a time, took
// 190 ms for the operators of L=54, D=768 (4.9 now) and 87 us for the
// transpose of U before a renormalization at L=24, D=512 (5 now).
constexpr int TRANS_EDGE = 32;
__global__ void __launch_bounds__(256) transpose_kernel(const TransJob *__restrict__ jobs, int njobs,
                                                        const double *__restrict__ src, double *__restrict__ dst) {
  __shared__ double piece[TRANS_EDGE][TRANS_EDGE + 1];
  const int tx = threadIdx.x % TRANS_EDGE, ty = threadIdx.x / TRANS_EDGE;
  for (int j = blockIdx.x; j < njobs; j += gridDim.x) {
    const TransJob J = jobs[j];
    const int64_t bs = (int64_t)J.rows * J.cols;
    if (J.rows < 16 || J.cols < 16) {
      const int64_t tot = bs * J.npos;
      for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < tot; e += (int64_t)gridDim.y * 256) {
        const int64_t p = e / bs, rem = e - p * bs;
        const int64_t c = rem / J.rows, r = rem - c * J.rows;
        dst[J.off + p * bs + c + r * J.cols] = src[J.off + e];
      }
      continue;
    }
    const int nr = (J.rows + TRANS_EDGE - 1) / TRANS_EDGE, nc = (J.cols + TRANS_EDGE - 1) / TRANS_EDGE;
    for (int u = blockIdx.y; u < nr * nc * J.npos; u += gridDim.y) {
      const int p = u / (nr * nc), t = u - p * (nr * nc);
      const int c0 = t / nr * TRANS_EDGE, r0 = (t - t / nr * nr) * TRANS_EDGE;
      const double *s = src + J.off + p * bs;
      double *d = dst + J.off + p * bs;
      for (int i = ty; i < TRANS_EDGE; i += 256 / TRANS_EDGE)
        if (c0 + i < J.cols && r0 + tx < J.rows) piece[i][tx] = s[(int64_t)(c0 + i) * J.rows + r0 + tx];
      __syncthreads();
      for (int i = ty; i < TRANS_EDGE; i += 256 / TRANS_EDGE)
        if (r0 + i < J.rows && c0 + tx < J.cols) d[(int64_t)(r0 + i) * J.cols + c0 + tx] = piece[tx][i];
      __syncthreads();   // the piece is reused
    }
  }
}

void launch_transpose(const TransJob *jobs, int njobs, const double *src, double *dst, void *stream) {
  if (njobs <= 0) return;
  const int share = std::min(64, std::max(1, 16384 / njobs));
  hipLaunchKernelGGL(transpose_kernel, dim3(std::min(njobs, 65535), share), dim3(256), 0, (hipStream_t)stream, jobs,
                     njobs, src, dst);
}

}  // namespace dmrg
