// Split-precision (BF16 slices) kernels for the stripe products of H.psi.
//
// A product C = A B of FP64 operands is computed from fixed-point BF16 slices
// (see SliceJob): C_ij = 2^(e_i + f_j - 16) sum_{t+u <= s-1} sum_k a^t_ik b^u_kj
// with slice t holding digit t at its weight 2^(-8t).  The inner sums run on
// MFMA into FP32 sums per product group d = t + u (exact for the leading
// groups, one rounded sum for the trailing ones, see slice_groups), and every
// split_fold_k terms the sums are folded into FP64 with the line scales.
// FP64 remains for the fold, the scales and the identity segments.
// Lane layouts (lane l, element e/r):
//   v_mfma_f32_16x16x32_bf16: A[l%16][8(l/16)+e], B[8(l/16)+e][l%16], D[4(l/16)+r][l%16];
//   v_mfma_f32_32x32x16_bf16: A[l%32][8(l/32)+e], B[8(l/32)+e][l%32],
//                             D[8(r/4)+4(l/32)+r%4][l%32].
#include <hip/hip_runtime.h>
#include <climits>
#include "plan.hpp"
#include "queue.hpp"

namespace dmrg {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ __forceinline__ const double *sbase_ptr(int id, const double *const *bases, const double *psi,
                                                   const double *y, const double *work, const double *part) {
  return id == BASE_PSI ? psi : id == BASE_Y ? y : id == BASE_WORK ? work : id == BASE_PART ? part
                                                                                             : bases[id - BASE_OPS];
}

// ------------------------------------------------------------------ slicing
// 2^(-8t), the weight at which slice t stores its digit
static_assert(SLICE_BITS == 8, "digit weights assume 8-bit slices");
__device__ constexpr float digit_weight(int t) {
  return t == 0 ? 1.0f : t == 1 ? 0x1p-8f : t == 2 ? 0x1p-16f : t == 3 ? 0x1p-24f : t == 4 ? 0x1p-32f
                                                                                        : t == 5 ? 0x1p-40f : 0x1p-48f;
}

// the eight values at K index kk of one line (position block already in `line`;
// padding reads a valid entry) ...
__device__ __forceinline__ void load_chunk(const double *__restrict__ line, int kk, int kb, int64_t s_k, double *x) {
#pragma unroll
  for (int i = 0; i < 8; i++) x[i] = line[(int64_t)min(kk + i, kb - 1) * s_k];
}
// ... and their slices, scaled by 2^-e, to out + t hs (padding slices zero)
__device__ __forceinline__ void slice_chunk(const double *x, int kk, int kb, int e, int ns, uint16_t *__restrict__ out,
                                            int hs) {
  typedef unsigned int v4u __attribute__((ext_vector_type(4)));
  double yv[8];
#pragma unroll
  for (int i = 0; i < 8; i++) yv[i] = ldexp(kk + i < kb ? x[i] : 0.0, -e);
  for (int t = 0; t < ns; t++) {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const double a = rint(yv[i] * 256.0);
      yv[i] = yv[i] * 256.0 - a;
      w[i] = __float_as_uint((float)a * digit_weight(t)) >> 16;   // |a| <= 256 at weight 2^(-8t): exact in BF16
    }
    *(v4u *)(out + t * hs) = (v4u){w[0] | w[1] << 16, w[2] | w[3] << 16, w[4] | w[5] << 16, w[6] | w[7] << 16};
  }
}

// slice_kernel: one work group per panel, the line maxima first, then the
// slices; tslice_kernel (exponents in place): one work group per K range of a
// panel.  Thread (l, g) takes the chunks g, g + 8, ... of line l.  The lines of
// a panel are neighbours in memory for all sources but the transposed ones, and
// their slices of one chunk are one run, so neither the loads nor the stores
// pass through LDS.  The stripes' slicing moves 3.8 TB/s of a copy's 4.7 (L=54,
// D=768: 45 GB in 12.1 ms; L=24, D=512: 3.9 GB in 1.0 ms); whole rows at a time
// were 13 % slower (scattered stores), 64 columns or the next values requested
// ahead made no difference.
struct PanelLine {
  int h, l;              // lines of the panel, this thread's line in it
  int64_t L;             // its line of the job
  const double *line;    // its values
  int64_t out;           // element of its first slice chunk
};
__device__ __forceinline__ PanelLine panel_line(const SliceJob &J, int panel, const double *src, int ns) {
  PanelLine p;
  p.h = min(SLICE_PANEL, J.nl - SLICE_PANEL * panel);
  p.l = min((int)threadIdx.x % SLICE_PANEL, p.h - 1);
  p.L = SLICE_PANEL * panel + p.l;
  const unsigned q = (unsigned)p.L / (unsigned)J.nrho, rho = (unsigned)p.L - q * (unsigned)J.nrho;
  p.line = src + J.src_off + (int64_t)q * J.s_q + (int64_t)rho * J.s_rho;
  p.out = (J.dst_off + (int64_t)SLICE_PANEL * panel * J.npos * J.kbp) * ns + 8 * p.l;
  return p;
}

// slices of the chunks c, c + 8, ... < c1 of a line
__device__ __forceinline__ void slice_range(const SliceJob &J, const PanelLine &P, int c, int c1, int e, int ns,
                                            uint16_t *__restrict__ out) {
  const int pch = J.kbp / 8, hs = 8 * P.h;
  for (; c < c1; c += 256 / SLICE_PANEL) {
    const int p = c / pch, kk = 8 * (c - p * pch);
    double x[8];
    load_chunk(P.line + (int64_t)p * J.s_pos, kk, J.kb, J.s_k, x);
    slice_chunk(x, kk, J.kb, e, ns, out + (int64_t)c * (ns * hs), hs);
  }
}

__global__ void __launch_bounds__(256) slice_kernel(const SliceJob *__restrict__ jobs,
                                                     const SliceItem *__restrict__ items, int nitems, int ns,
                                                     const double *const *__restrict__ bases,
                                                     const double *__restrict__ psi,
                                                     const double *__restrict__ work, SliceBufs bufs) {
  __shared__ double mx[256 / SLICE_PANEL][SLICE_PANEL];
  const int g = threadIdx.x / SLICE_PANEL, l0 = threadIdx.x % SLICE_PANEL;
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const SliceItem I = items[it];
    const SliceJob J = jobs[I.job];
    const double *src = sbase_ptr(J.src_base, bases, psi, nullptr, work, nullptr);
    const PanelLine P = panel_line(J, I.panel, src, ns);
    // line lengths fit in 31 bits (checked when the plan is built)
    const int nch = J.npos * (J.kbp / 8), pch = J.kbp / 8;
    double m = 0.0;
    for (int c = g; c < nch; c += 256 / SLICE_PANEL) {
      const int p = c / pch, kk = 8 * (c - p * pch);
      const double *line = P.line + (int64_t)p * J.s_pos;
      double v[8];
      load_chunk(line, kk, J.kb, J.s_k, v);
#pragma unroll
      for (int i = 0; i < 8; i++) m = fmax(m, fabs(v[i]));
    }
    mx[g][l0] = m;
    __syncthreads();
    for (int i = 0; i < 256 / SLICE_PANEL; i++) m = fmax(m, mx[i][l0]);
    int e = 0;
    if (m > 0.0) {
      int ex;
      const double mant = frexp(m, &ex);    // m = mant 2^ex, mant in [0.5, 1)
      e = (mant == 0.5) ? ex - 1 : ex;      // smallest e with m <= 2^e
    }
    if (l0 < P.h) {
      if (g == 0) bufs.exps[J.dst_buf][J.exp_off + P.L] = e;
      uint16_t *out = bufs.data[J.dst_buf] + P.out;
      slice_range(J, P, g, nch, e, ns, out);
    }
    __syncthreads();   // mx is reused by the next panel
  }
}

__global__ void __launch_bounds__(256) tslice_kernel(const SliceJob *__restrict__ jobs,
                                                      const SliceItem *__restrict__ items, int nitems, int ns,
                                                      const double *__restrict__ work, SliceBufs bufs) {
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const SliceItem I = items[it];
    const SliceJob J = jobs[I.job];
    if ((int)threadIdx.x % SLICE_PANEL >= J.nl - SLICE_PANEL * I.panel) continue;
    const PanelLine P = panel_line(J, I.panel, work, ns);
    const int e = bufs.exps[SBUF_T][J.exp_off + P.L];
    slice_range(J, P, I.c0 + threadIdx.x / SLICE_PANEL, min(J.npos * (J.kbp / 8), I.c0 + TSLICE_CHUNKS),
                e == INT_MIN ? 0 : e, ns, bufs.data[SBUF_T] + P.out);
  }
}

__global__ void fill_int_kernel(int32_t *__restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_tslices(const SliceJob *jobs, const SliceItem *items, int nitems, int nslices, const double *work,
                    SliceBufs bufs, void *stream) {
  if (nitems <= 0) return;
  hipLaunchKernelGGL(tslice_kernel, dim3(std::min(nitems, 65535)), dim3(256), 0, (hipStream_t)stream, jobs, items,
                     nitems, nslices, work, bufs);
}

void launch_fill_int(int32_t *p, int64_t n, int32_t v, void *stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_int_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65535)), dim3(256), 0,
                     (hipStream_t)stream, p, n, v);
}

void launch_slices(const SliceJob *jobs, const SliceItem *items, int nitems, int nslices, const double *const *bases,
                   const double *psi, const double *work, SliceBufs bufs, void *stream) {
  if (nitems <= 0) return;
  hipLaunchKernelGGL(slice_kernel, dim3(std::min(nitems, 8192)), dim3(256), 0, (hipStream_t)stream, jobs, items,
                     nitems, nslices, bases, psi, work, bufs);
}

// ------------------------------------------------------------------ split products
// descriptor arrays read through the constant address space (scalar loads)
typedef const SegS __attribute__((address_space(4))) CSegS;
typedef const Seg __attribute__((address_space(4))) CSeg;
// slice buffers live in device global memory: global (not flat) loads
typedef const void __attribute__((address_space(1))) *gvptr;
typedef void __attribute__((address_space(3))) *lvptr;
typedef const v8bf __attribute__((address_space(3))) *lv8ptr;
// s_waitcnt immediates (gfx9 encoding): vmcnt(0) alone, lgkmcnt(0) alone
constexpr int WAIT_VM0 = 0x0F70, WAIT_LGKM0 = 0xC07F;

// LDS stage of one wavefront: (MB + NB) * NS chunks of 64 lanes x 16 bytes
constexpr int stage_bytes(int ns) { return 5 * ns * 1024; }
constexpr int LDS_BYTES = 160 * 1024;   // per CU

// FP32 sum of slice-product group d for s = NS (see slice_groups)
template <int NS>
__device__ constexpr int sgroup(int d) { return d < slice_groups(NS) - 1 ? d : slice_groups(NS) - 1; }
static_assert(SLICE_BITS == 8, "fold weights assume 8-bit slices");

// fold of the group sums of one element: their FP64 sum (group 0 first)
template <int G, typename V>
__device__ __forceinline__ double fold_groups(const V *q, int r) {
  double x = (double)q[0][r];
  for (int g = 1; g < G; g++) x += (double)q[g][r];
  return x;
}

// Byte offset of chunk 0, slice 0 of line L of nl lines of length ld, from the
// first slice of its operand, and the stride hs between the slices of a chunk
// (chunks follow at NS hs).  64-bit: the lines of a segment's operand begin
// anywhere in the record's panels.
template <int NS>
__device__ __forceinline__ uint64_t line_offset(uint32_t L, uint32_t nl, uint32_t ld, uint32_t &hs) {
  const uint32_t p = L / SLICE_PANEL;
  hs = 16u * min((uint32_t)SLICE_PANEL, nl - SLICE_PANEL * p);
  return (uint64_t)(SLICE_PANEL * 2u * NS * p) * ld + 16u * (L % SLICE_PANEL);
}

// One wavefront tile.  The K steps of all segments are one sequence: the
// operands of a step go straight from global memory into this wave's LDS stage
// (one 1 KiB chunk per operand row block and slice, 16 bytes per lane), and the
// loads of the next step, also across a segment boundary, fly while the MFMAs
// of this one run without holding a second set of registers.  What bounds it is
// the latency of that round trip, so as many waves run per CU as their stages
// fit (SPLIT_WAVES).
template <int MB, int NS>
__device__ __forceinline__ void item_split(const Tile &T, const Seg *__restrict__ segs,
                                           const SegS *__restrict__ ssegs, const double *const *bases,
                                           const double *psi, double *y, double *work, double *part,
                                           const SliceBufs &bufs, char *stage, int r16, int q4) {
  constexpr int NB = 4 / MB;
  constexpr int FOLD = split_fold_k(NS);
  static_assert(FOLD % 32 == 0, "the K loop folds after whole 32-wide steps");
  // descriptors: scalar loads
  const CSegS *cs = (const CSegS *)ssegs + T.seg0;
  const CSeg *cg = (const CSeg *)segs + T.seg0;
  asm volatile("" : "+v"(r16), "+v"(q4));   // nothing derived from the lane is kept across tiles
  v4d acc[MB][NB];
  for (int a = 0; a < MB; a++)
    for (int b = 0; b < NB; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
  const int mrem = T.m - T.i0, nrem = T.n - T.j0;
  // identity left operators (first in the list): exact FP64 additions of the FP64 operand
  for (int si = 0; si < T.nid; si++) {
    CSeg &S = cg[si];
    const double *B = sbase_ptr(S.b_base, bases, psi, y, work, part) + S.b_off;
    for (int bi = 0; bi < MB; bi++)
      for (int bj = 0; bj < NB; bj++) {
        int jj = 16 * bj + r16;
        if (jj >= nrem) continue;
        int n = T.j0 + jj;
        int pn = n / S.b_nb;
        int64_t bo = (int64_t)pn * S.b_pn + (int64_t)(n - pn * S.b_nb) * S.b_n;
        for (int r = 0; r < 4; r++) {
          int i = 16 * bi + 4 * q4 + r;
          if (i < mrem) {
            int k = T.i0 + i;
            int pk = k / S.b_kb;
            acc[bi][bj][r] += S.s * B[(int64_t)pk * S.b_pk + (int64_t)(k - pk * S.b_kb) * S.b_k + bo];
          }
        }
      }
  }
  if (T.nid < T.nseg) {
    // chunk 0 of this lane's operand lines in segment si, and the strides
    // between slices.  Lanes past the last row / column read the last one: their
    // outputs are never stored, so every operand load is unconditional.
    const char *arow[MB], *bcol[NB];
    uint32_t ahs[MB], bhs[NB];
    auto lines = [&](int si) {
      CSegS &Q = cs[si];
      const char *A = (const char *)(bufs.data[Q.a_buf] + Q.a_off * NS);   // the slices start at NS times the offset
      const char *B = (const char *)(bufs.data[Q.b_buf] + Q.b_off * NS);
      for (int bi = 0; bi < MB; bi++) {
        arow[bi] = A + line_offset<NS>(Q.a_line0 + T.i0 + min(16 * bi + r16, mrem - 1), Q.a_nl, (uint32_t)Q.a_ld, ahs[bi]);
        arow[bi] += (uint64_t)(NS * (Q.a_k0 / 8)) * ahs[bi];
      }
      for (int bj = 0; bj < NB; bj++) {
        bcol[bj] = B + line_offset<NS>(Q.b_line0 + T.j0 + min(16 * bj + r16, nrem - 1), Q.b_nl, (uint32_t)Q.b_ld, bhs[bj]);
        bcol[bj] += (uint64_t)(NS * (Q.b_k0 / 8)) * bhs[bj];
      }
    };
    // scale exponents of this lane's output elements
    auto exps = [&](int si, int (*er)[4], int *fc) {
      CSegS &Q = cs[si];
      const int32_t *ea = bufs.exps[Q.a_buf] + Q.a_exp;
      const int32_t *eb = bufs.exps[Q.b_buf] + Q.b_exp;
      for (int bi = 0; bi < MB; bi++)
        for (int r = 0; r < 4; r++) er[bi][r] = ea[T.i0 + min(16 * bi + 4 * q4 + r, mrem - 1)];
      for (int bj = 0; bj < NB; bj++) fc[bj] = eb[T.j0 + min(16 * bj + r16, nrem - 1)];
    };
    // one K step into the stage.  K is a multiple of 8 and the lines are
    // zero-padded to it, so the chunk of 8 at min(k, K - 8) is always inside the
    // operand; a lane whose chunk starts at or past K multiplies a zeroed A operand.
    auto dma = [&](int k0, int K) {
      const uint32_t kc = NS * ((uint32_t)min(k0 + 8 * q4, K - 8) / 8);
      for (int bi = 0; bi < MB; bi++) {
        const char *at = arow[bi] + (uint64_t)kc * ahs[bi];
        for (int t = 0; t < NS; t++)
          __builtin_amdgcn_global_load_lds((gvptr)(at + t * ahs[bi]), (lvptr)(stage + (bi * NS + t) * 1024), 16, 0, 0);
      }
      for (int bj = 0; bj < NB; bj++) {
        const char *bt = bcol[bj] + (uint64_t)kc * bhs[bj];
        for (int t = 0; t < NS; t++)
          __builtin_amdgcn_global_load_lds((gvptr)(bt + t * bhs[bj]), (lvptr)(stage + ((MB + bj) * NS + t) * 1024),
                                           16, 0, 0);
      }
    };
    v4f q[MB][NB][slice_groups(NS)];
    for (int bi = 0; bi < MB; bi++)
      for (int bj = 0; bj < NB; bj++)
        for (int g = 0; g < slice_groups(NS); g++) q[bi][bj][g] = (v4f){0.f, 0.f, 0.f, 0.f};
    int si = T.nid, k0 = 0, K = cs[si].K;
    double sc = cg[si].s;
    lines(si);
    dma(0, K);
    for (;;) {
      __builtin_amdgcn_s_waitcnt(WAIT_VM0);      // this step's chunks are in LDS
      __builtin_amdgcn_sched_barrier(0);
      v8bf as[MB][NS], bs[NB][NS];
      const int lo = 16 * (r16 + 16 * q4);
      for (int t = 0; t < NS; t++) {
        for (int bi = 0; bi < MB; bi++) as[bi][t] = *(const lv8ptr)(stage + (bi * NS + t) * 1024 + lo);
        for (int bj = 0; bj < NB; bj++) bs[bj][t] = *(const lv8ptr)(stage + ((MB + bj) * NS + t) * 1024 + lo);
      }
      const bool newseg = k0 + 32 >= K;
      const int nsi = newseg ? si + 1 : si, nk0 = newseg ? 0 : k0 + 32;
      const bool more = nsi < T.nseg;
      const bool fold = newseg || (k0 + 32) % FOLD == 0;
      int nK = K, erow[MB][4], fcol[NB];
      double nsc = sc;
      if (newseg && more) {
        nK = cs[nsi].K;
        nsc = cg[nsi].s;
        lines(nsi);
      }
      __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);    // ... and in registers: the stage is free
      __builtin_amdgcn_sched_barrier(0);
      if (fold) exps(si, erow, fcol);
      if (more) dma(nk0, nK);
      __builtin_amdgcn_sched_barrier(0);
      if (k0 + 32 > K && k0 + 8 * q4 >= K)   // only the last step of a segment has such lanes
        for (int bi = 0; bi < MB; bi++)
          for (int t = 0; t < NS; t++) as[bi][t] = (v8bf){};
#pragma unroll
      for (int d = 0; d < NS; d++)
#pragma unroll
        for (int t = 0; t <= d; t++)
          for (int bi = 0; bi < MB; bi++)
            for (int bj = 0; bj < NB; bj++)
              q[bi][bj][sgroup<NS>(d)] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(as[bi][t], bs[bj][d - t], q[bi][bj][sgroup<NS>(d)], 0, 0, 0);
      if (fold) {
        for (int bi = 0; bi < MB; bi++)
          for (int bj = 0; bj < NB; bj++)
            for (int r = 0; r < 4; r++) {
              const double x = fold_groups<slice_groups(NS)>(q[bi][bj], r);
              acc[bi][bj][r] += sc * ldexp(x, erow[bi][r] + fcol[bj] - 2 * SLICE_BITS);
            }
        for (int bi = 0; bi < MB; bi++)
          for (int bj = 0; bj < NB; bj++)
            for (int g = 0; g < slice_groups(NS); g++) q[bi][bj][g] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      if (!more) break;
      K = nK;
      sc = nsc;
      si = nsi;
      k0 = nk0;
    }
  }
  double *C = const_cast<double *>(sbase_ptr(T.c_base, bases, psi, y, work, part)) + T.c_off;
  for (int bi = 0; bi < MB; bi++)
    for (int bj = 0; bj < NB; bj++)
      for (int r = 0; r < 4; r++) {
        int i = 16 * bi + 4 * q4 + r, j = 16 * bj + r16;
        if (i < mrem && j < nrem) {
          double *c = T.rowmajor ? C + (int64_t)(T.ci0 + i) * T.ldc + (T.cj0 + j)
                                 : C + (int64_t)(T.ci0 + i) + (int64_t)(T.cj0 + j) * T.ldc;
          *c = T.accumulate ? *c + acc[bi][bj][r] : acc[bi][bj][r];
        }
      }
  // first-stage tiles: exponent of every stripe column they wrote (smallest e
  // with max |value| <= 2^e), combined over tiles with atomicMax
  const SegS Q0 = ssegs[T.seg0];
  if (Q0.t_exp >= 0) {
    int32_t *ex = bufs.exps[SBUF_T] + Q0.t_exp;
    for (int bj = 0; bj < NB; bj++) {
      const int j = 16 * bj + r16;
      double m = 0.0;
      for (int bi = 0; bi < MB; bi++)
        for (int r = 0; r < 4; r++) {
          const int i = 16 * bi + 4 * q4 + r;
          if (i < mrem && j < nrem) m = fmax(m, fabs(acc[bi][bj][r]));
        }
      m = fmax(m, __shfl_xor(m, 16));
      m = fmax(m, __shfl_xor(m, 32));
      if (q4 == 0 && j < nrem && m > 0.0) {
        int e2;
        const double mant = frexp(m, &e2);
        atomicMax(ex + (T.cj0 + j) % Q0.t_nb, mant == 0.5 ? e2 - 1 : e2);
      }
    }
  }
}

// Wavefront tiles: every wavefront takes its next tile from the per-XCD
// queues (one lane takes it, the index is wave-uniform).
// waves of a work group: 25 KiB of LDS each at s = 5, so three work groups of
// two fit a CU, where one of four did
constexpr int SPLIT_WAVES = 2;
template <int NS>
__device__ __forceinline__ void items_split(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,
                                            const SegS *__restrict__ ssegs, const XcdQueues &q,
                                            int32_t *__restrict__ counters,
                                            int32_t *__restrict__ next_counters, int chunk,
                                            const double *const *__restrict__ bases, const double *__restrict__ psi,
                                            double *__restrict__ y, double *__restrict__ work,
                                            double *__restrict__ part, const SliceBufs &bufs) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;
  __shared__ __attribute__((aligned(1024))) char lds[SPLIT_WAVES * stage_bytes(NS)];
  char *stage = lds + wave * stage_bytes(NS);
  clear_counters(next_counters);
  WorkQueue wq(q, counters, (int)(blockIdx.x / NXCD) * SPLIT_WAVES + wave, (int)(gridDim.x / NXCD) * SPLIT_WAVES, chunk);
  do {
    for (; wq.t < wq.tend; wq.t += wq.step) {
      if (wq.last()) wq.request(lane == 0);
      const Tile T = tiles[__builtin_amdgcn_readfirstlane(wq.t)];
      if (T.mb == 1) item_split<1, NS>(T, segs, ssegs, bases, psi, y, work, part, bufs, stage, r16, q4);
      else if (T.mb == 4) item_split<4, NS>(T, segs, ssegs, bases, psi, y, work, part, bufs, stage, r16, q4);
      else item_split<2, NS>(T, segs, ssegs, bases, psi, y, work, part, bufs, stage, r16, q4);
    }
  } while (wq.next(lane));
}

// ------------------------------------------------------------ work-group tiles
// A 64 x 64 output tile computed by the four wavefronts of a work group: wave
// w owns the 32 x 32 quarter (w >> 1, w & 1).  Each 32-wide K step of the
// operands (A: 4 row blocks of 16 rows, B: 4 column blocks of 16 columns, NS
// slices each) goes from global memory straight into one of two LDS stages --
// wave w loads row block w and column block w, 16 bytes per lane and slice,
// in the MFMA operand layout -- and after one barrier every wave reads the two
// row blocks and two column blocks of its quarter.  The loads of the next step
// (across segment boundaries) are issued before this step's MFMAs, so each
// operand byte is fetched once per work group instead of once per wavefront,
// and the stage's waves overlap their loads with the other work group's MFMAs
// (two work groups per CU).
constexpr int mstage_bytes(int ns) { return 8 * ns * 1024; }

template <int NS>
__device__ __forceinline__ void macro_split(const Tile &T, const Seg *__restrict__ segs,
                                            const SegS *__restrict__ ssegs, const double *const *bases,
                                            const double *psi, double *y, double *work, double *part,
                                            const SliceBufs &bufs, char *lds, int wave, int lane) {
  constexpr int MB = 2, NB = 2;
  constexpr int STAGE = mstage_bytes(NS);
  constexpr int FOLD = split_fold_k(NS);
  static_assert(FOLD % 32 == 0, "the K loop folds after whole 32-wide steps");
  const int r16 = lane & 15, q4 = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;
  const int i0 = T.i0 + 32 * wr, j0 = T.j0 + 32 * wc;     // this wave's quarter
  const int mrem = T.m - i0, nrem = T.n - j0;              // <= 0: quarter outside the output
  // operand line this lane loads (row block `wave` of A, column block `wave` of
  // B); lines past the output read the last one (never stored)
  const uint32_t lrow = (uint32_t)min(T.i0 + 16 * wave + r16, T.m - 1);
  const uint32_t lcol = (uint32_t)min(T.j0 + 16 * wave + r16, T.n - 1);
  v4d acc[MB][NB];
  for (int a = 0; a < MB; a++)
    for (int b = 0; b < NB; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
  // identity left operators: exact FP64 additions of the FP64 operand
  for (int si = 0; si < T.nseg; si++) {
    if (ssegs[T.seg0 + si].K != 0) continue;
    const Seg S = segs[T.seg0 + si];
    const double *B = sbase_ptr(S.b_base, bases, psi, y, work, part) + S.b_off;
    for (int bi = 0; bi < MB; bi++)
      for (int bj = 0; bj < NB; bj++) {
        const int jj = 16 * bj + r16;
        if (jj >= nrem) continue;
        const int n = j0 + jj;
        const int pn = n / S.b_nb;
        const int64_t bo = (int64_t)pn * S.b_pn + (int64_t)(n - pn * S.b_nb) * S.b_n;
        for (int r = 0; r < 4; r++) {
          const int i = 16 * bi + 4 * q4 + r;
          if (i < mrem) {
            const int k = i0 + i;
            const int pk = k / S.b_kb;
            acc[bi][bj][r] += S.s * B[(int64_t)pk * S.b_pk + (int64_t)(k - pk * S.b_kb) * S.b_k + bo];
          }
        }
      }
  }
  int si = 0;
  while (si < T.nseg && ssegs[T.seg0 + si].K == 0) si++;
  // every wave has finished reading the LDS stages of its previous tile
  __syncthreads();
  if (si < T.nseg) {
    // scale exponents of this lane's outputs (clamped inside the output)
    auto exps = [&](const SegS &Q, int (*er)[4], int *fc) {
      const int32_t *ea = bufs.exps[Q.a_buf] + Q.a_exp;
      const int32_t *eb = bufs.exps[Q.b_buf] + Q.b_exp;
      for (int bi = 0; bi < MB; bi++)
        for (int r = 0; r < 4; r++) er[bi][r] = ea[min(i0 + 16 * bi + 4 * q4 + r, T.m - 1)];
      for (int bj = 0; bj < NB; bj++) fc[bj] = eb[min(j0 + 16 * bj + r16, T.n - 1)];
    };
    // one K step of segment Q at k0 into LDS stage b (K is a multiple of 8 and
    // lines are zero-padded to it: the chunk of 8 at min(k, K - 8) is inside
    // the operand; lanes whose chunk starts at or past K are zeroed at the MFMA)
    auto issue = [&](const SegS &Q, int k0, int b) {
      const char *A = (const char *)(bufs.data[Q.a_buf] + Q.a_off * NS);   // panels, see item_split
      const char *B = (const char *)(bufs.data[Q.b_buf] + Q.b_off * NS);
      const uint32_t kc = (uint32_t)min(k0 + 8 * q4, Q.K - 8) / 8;
      uint32_t ah, bh;
      A += line_offset<NS>(Q.a_line0 + lrow, Q.a_nl, (uint32_t)Q.a_ld, ah);
      B += line_offset<NS>(Q.b_line0 + lcol, Q.b_nl, (uint32_t)Q.b_ld, bh);
      A += (uint64_t)(NS * (Q.a_k0 / 8 + kc)) * ah;
      B += (uint64_t)(NS * (Q.b_k0 / 8 + kc)) * bh;
      char *st = lds + b * STAGE;
      for (int t = 0; t < NS; t++) {
        __builtin_amdgcn_global_load_lds((gvptr)(A + t * ah), (lvptr)(st + (wave * NS + t) * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gvptr)(B + t * bh), (lvptr)(st + ((4 + wave) * NS + t) * 1024), 16, 0, 0);
      }
    };
    v4f q[MB][NB][slice_groups(NS)];
    for (int bi = 0; bi < MB; bi++)
      for (int bj = 0; bj < NB; bj++)
        for (int g = 0; g < slice_groups(NS); g++) q[bi][bj][g] = (v4f){0.f, 0.f, 0.f, 0.f};
    SegS Q = ssegs[T.seg0 + si];
    double sc = segs[T.seg0 + si].s;
    int erow[MB][4], fcol[NB];
    exps(Q, erow, fcol);
    issue(Q, 0, 0);
    int k0 = 0, b = 0;
    for (;;) {
      __builtin_amdgcn_s_waitcnt(WAIT_VM0);      // this wave's chunks of the step are in LDS ...
      __syncthreads();                          // ... and every other wave's; the other stage is free
      int nsi = si, nk0 = k0 + 32;
      const bool newseg = nk0 >= Q.K;
      if (newseg) {
        nk0 = 0;
        nsi++;
        while (nsi < T.nseg && ssegs[T.seg0 + nsi].K == 0) nsi++;
      }
      const bool more = nsi < T.nseg;
      SegS NQ = Q;
      double nsc = sc;
      int nerow[MB][4], nfcol[NB];
      if (more && newseg) {
        NQ = ssegs[T.seg0 + nsi];
        nsc = segs[T.seg0 + nsi].s;
      }
      // this step's operands: LDS -> registers, all reads complete (and the
      // next segment's descriptors in) before the next step's loads into the
      // other stage are issued, so no wait below depends on those loads
      v8bf as[MB][NS], bs[NB][NS];
      const char *st = lds + b * STAGE;
      for (int t = 0; t < NS; t++) {
        for (int bi = 0; bi < MB; bi++) as[bi][t] = *(const lv8ptr)(st + ((2 * wr + bi) * NS + t) * 1024 + 16 * lane);
        for (int bj = 0; bj < NB; bj++)
          bs[bj][t] = *(const lv8ptr)(st + ((4 + 2 * wc + bj) * NS + t) * 1024 + 16 * lane);
      }
      __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        issue(NQ, nk0, b ^ 1);
        if (newseg) exps(NQ, nerow, nfcol);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (k0 + 32 > Q.K && k0 + 8 * q4 >= Q.K)   // only the last step of a segment has such lanes
        for (int bi = 0; bi < MB; bi++)
          for (int t = 0; t < NS; t++) as[bi][t] = (v8bf){};
#pragma unroll
      for (int d = 0; d < NS; d++)
#pragma unroll
        for (int t = 0; t <= d; t++)
          for (int bi = 0; bi < MB; bi++)
            for (int bj = 0; bj < NB; bj++)
              q[bi][bj][sgroup<NS>(d)] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(as[bi][t], bs[bj][d - t], q[bi][bj][sgroup<NS>(d)], 0, 0, 0);
      if (newseg || (k0 + 32) % FOLD == 0) {
        for (int bi = 0; bi < MB; bi++)
          for (int bj = 0; bj < NB; bj++)
            for (int r = 0; r < 4; r++) {
              const double x = fold_groups<slice_groups(NS)>(q[bi][bj], r);
              acc[bi][bj][r] += sc * ldexp(x, erow[bi][r] + fcol[bj] - 2 * SLICE_BITS);
            }
        for (int bi = 0; bi < MB; bi++)
          for (int bj = 0; bj < NB; bj++)
            for (int g = 0; g < slice_groups(NS); g++) q[bi][bj][g] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      if (!more) break;
      if (newseg) {
        Q = NQ;
        sc = nsc;
        si = nsi;
        for (int bi = 0; bi < MB; bi++)
          for (int r = 0; r < 4; r++) erow[bi][r] = nerow[bi][r];
        for (int bj = 0; bj < NB; bj++) fcol[bj] = nfcol[bj];
      }
      k0 = nk0;
      b ^= 1;
    }
  }
  double *C = const_cast<double *>(sbase_ptr(T.c_base, bases, psi, y, work, part)) + T.c_off;
  const int ci0 = T.ci0 + 32 * wr, cj0 = T.cj0 + 32 * wc;
  for (int bi = 0; bi < MB; bi++)
    for (int bj = 0; bj < NB; bj++)
      for (int r = 0; r < 4; r++) {
        const int i = 16 * bi + 4 * q4 + r, j = 16 * bj + r16;
        if (i < mrem && j < nrem) {
          double *c = T.rowmajor ? C + (int64_t)(ci0 + i) * T.ldc + (cj0 + j)
                                 : C + (int64_t)(ci0 + i) + (int64_t)(cj0 + j) * T.ldc;
          *c = T.accumulate ? *c + acc[bi][bj][r] : acc[bi][bj][r];
        }
      }
  // first-stage tiles: exponent of every stripe column written (see item_split)
  const SegS Q0 = ssegs[T.seg0];
  if (Q0.t_exp >= 0) {
    int32_t *ex = bufs.exps[SBUF_T] + Q0.t_exp;
    for (int bj = 0; bj < NB; bj++) {
      const int j = 16 * bj + r16;
      double m = 0.0;
      for (int bi = 0; bi < MB; bi++)
        for (int r = 0; r < 4; r++) {
          const int i = 16 * bi + 4 * q4 + r;
          if (i < mrem && j < nrem) m = fmax(m, fabs(acc[bi][bj][r]));
        }
      m = fmax(m, __shfl_xor(m, 16));
      m = fmax(m, __shfl_xor(m, 32));
      if (q4 == 0 && j < nrem && m > 0.0) {
        int e2;
        const double mant = frexp(m, &e2);
        atomicMax(ex + (cj0 + j) % Q0.t_nb, mant == 0.5 ? e2 - 1 : e2);
      }
    }
  }
}

template <int NS>
__device__ __forceinline__ void macro_items(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,
                                            const SegS *__restrict__ ssegs, const XcdQueues &q,
                                            int32_t *__restrict__ counters,
                                            int32_t *__restrict__ next_counters,
                                            const double *const *__restrict__ bases, const double *__restrict__ psi,
                                            double *__restrict__ y, double *__restrict__ work,
                                            double *__restrict__ part, const SliceBufs &bufs) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // all of the LDS holds the two operand stages (two work groups per CU); the
  // index of the next tile reaches the wavefronts through the second one, which
  // a tile writes only after the first barrier of its K loop
  __shared__ __attribute__((aligned(1024))) char lds[2 * mstage_bytes(NS)];
  clear_counters(next_counters);
  WorkQueue wq(q, counters, (int)(blockIdx.x / NXCD), (int)(gridDim.x / NXCD), 1);
  for (bool more = true; more;) {
    for (; wq.t < wq.tend; wq.t += wq.step) {
      if (wave == 0 && wq.last()) wq.request(lane == 0);
      const Tile T = tiles[__builtin_amdgcn_readfirstlane(wq.t)];
      macro_split<NS>(T, segs, ssegs, bases, psi, y, work, part, bufs, lds, wave, lane);
    }
    __syncthreads();   // everyone has read the last LDS stage
    if (wave == 0) {
      const int v = wq.next(lane) ? wq.t : -1;
      if (lane == 0) *(volatile int *)(lds + mstage_bytes(NS)) = v;
    }
    __syncthreads();
    wq.t = __builtin_amdgcn_readfirstlane(*(volatile int *)(lds + mstage_bytes(NS)));
    more = wq.t >= 0;
    wq.tend = wq.t + 1;
    wq.step = 1;
  }
}

#define MACRO_KERNELS(NS)                                                                                   \
  __global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))                 \
  stage1_msplit##NS##_kernel(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,                  \
                             const SegS *__restrict__ ssegs, XcdQueues q, int32_t *__restrict__ counters,   \
                             int32_t *__restrict__ next_counters,\
                             const double *const *__restrict__ bases, const double *__restrict__ psi,       \
                             double *__restrict__ y, double *__restrict__ work, double *__restrict__ part,   \
                             SliceBufs bufs) {                                                              \
    macro_items<NS>(tiles, segs, ssegs, q, counters, next_counters, bases, psi, y, work, part, bufs);                      \
  }                                                                                                         \
  __global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))                 \
  stage2_msplit##NS##_kernel(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,                  \
                             const SegS *__restrict__ ssegs, XcdQueues q, int32_t *__restrict__ counters,   \
                             int32_t *__restrict__ next_counters,\
                             const double *const *__restrict__ bases, const double *__restrict__ psi,       \
                             double *__restrict__ y, double *__restrict__ work, double *__restrict__ part,   \
                             SliceBufs bufs) {                                                              \
    macro_items<NS>(tiles, segs, ssegs, q, counters, next_counters, bases, psi, y, work, part, bufs);                      \
  }

MACRO_KERNELS(3)
MACRO_KERNELS(4)
MACRO_KERNELS(5)
MACRO_KERNELS(6)
MACRO_KERNELS(7)

// ------------------------------------------------------------ wide work-group tiles
// A 128 x 128 output tile (WIDE_MB) computed by the eight wavefronts of a
// work group, two per SIMD, in blocks of v_mfma_f32_32x32x16_bf16: the blocks
// that lie inside the output (up to 16) are dealt to the waves, so a part-filled
// tile costs what its blocks cost (outputs of 48 to 127 lines; 42 % of the wide
// tiles' products at L = 54, D = 768 fell outside).  Lane l holds output column l % 32 of a block and its rows wrow(r) = 8 (r / 4) + 4 (l / 32)
// + r % 4, so the accesses of 32 lanes to the row-major stripes (first-stage
// stores, identity segments) are contiguous 256-byte runs, and a column's
// exponent takes one exchange between lanes.  Each 32-wide K step of
// the operands (A: 4 row blocks of 32 lines, B: 4 column blocks, two K halves
// of 16, NS slices; 1 KiB per block, half and slice) goes from global memory
// through registers into one of two LDS stages -- wave w loads row block
// w % 4 and column block w % 4 of K half w / 4 -- while the step before runs
// on the other stage.  The stages are two separate LDS objects, so the
// compiler knows that the stores into one never alias the reads of the other.
constexpr int wstage_bytes(int ns) { return 16 * ns * 1024; }
__device__ __forceinline__ int wrow(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

template <int NS>
__device__ __forceinline__ void wide_split(const Tile &T, const Seg *__restrict__ segs,
                                           const SegS *__restrict__ ssegs, const double *const *bases,
                                           const double *psi, double *y, double *work, double *part,
                                           const SliceBufs &bufs, char *lds0, char *lds1, int wave, int lane) {
  constexpr int FOLD = split_fold_k(NS);
  static_assert(FOLD % 32 == 0, "the K loop folds after whole 32-wide steps");
  typedef float v16f __attribute__((ext_vector_type(16)));
  // the tile and segment descriptors do not change during the launch: read
  // through the constant address space they are scalar loads (scalar cache,
  // no vector memory wait on the K loop's path)
  const CSegS *cs = (const CSegS *)ssegs;
  const CSeg *cg = (const CSeg *)segs;
  // the lane index passes through an empty asm per tile: the per-lane column
  // offsets derived from it are recomputed per tile instead of being hoisted
  // out of the tile loop into registers that the K loop needs
  asm volatile("" : "+v"(lane));
  const int c32 = lane & 31, h = lane >> 5;
  // the 32 x 32 blocks inside the output, row by row: the first nblk - 8 waves
  // take two neighbours each, the others one
  const int nc = min(4, (T.n - T.j0 + 31) >> 5), nblk = nc * min(4, (T.m - T.i0 + 31) >> 5);
  const int two = max(0, nblk - WIDE_WAVES);
  const int nb = wave < two ? 2 : wave < nblk ? 1 : 0;
  int br[2], bc[2];
  for (int b = 0; b < 2; b++) {
    const int id = min(wave < two ? 2 * wave + b : two + wave, nblk - 1);
    br[b] = id / nc;
    bc[b] = id - br[b] * nc;
  }
  // operand lines this lane loads: row block / column block wave % 4, K half
  // wave / 4 (see issue)
  const int lb = wave & 3, lkh = wave >> 2;
  double acc[2][16];
  for (int b = 0; b < 2; b++)
    for (int r = 0; r < 16; r++) acc[b][r] = 0.0;
  // identity left operators: exact FP64 additions of the FP64 operand
  for (int si = 0; si < T.nseg; si++) {
    if (cs[T.seg0 + si].K != 0) continue;
    CSeg &S = cg[T.seg0 + si];
    const double *B = sbase_ptr(S.b_base, bases, psi, y, work, part) + S.b_off;
    for (int b = 0; b < 2; b++) {
      const int n = T.j0 + 32 * bc[b] + c32, i0 = T.i0 + 32 * br[b];
      if (b >= nb || n >= T.n) continue;
      const int pn = n / S.b_nb;
      const int64_t bo = (int64_t)pn * S.b_pn + (int64_t)(n - pn * S.b_nb) * S.b_n;
      for (int r = 0; r < 16; r++) {
        const int k = i0 + wrow(r, h);
        if (k < T.m) {
          const int pk = k / S.b_kb;
          acc[b][r] += S.s * B[(int64_t)pk * S.b_pk + (int64_t)(k - pk * S.b_kb) * S.b_k + bo];
        }
      }
    }
  }
  int si = 0;
  while (si < T.nseg && cs[T.seg0 + si].K == 0) si++;
  // every wave has finished reading the LDS stages of its previous tile
  __syncthreads();
  if (si < T.nseg) {
    // one operand's NS chunks of a K step of segment qi at k0 (operand 0: the A
    // lines of row block wave % 4, 1: the B lines of column block wave % 4; K
    // half wave / 4) into registers.  K is a multiple of 8 and lines are
    // zero-padded to it: the chunk of 8 at min(k, K - 8) is inside the operand;
    // lanes whose chunk starts at or past K are zeroed at the MFMA.  Plain
    // vector loads: under load they complete about 2.5 times sooner than
    // loads straight into LDS.
    typedef unsigned int v4u __attribute__((ext_vector_type(4)));
    auto load = [&](int qi, int k0, int op, v4u *pre) {
      if (32 * lb >= (op ? T.n - T.j0 : T.m - T.i0)) return;   // block outside the output
      CSegS &Q = cs[T.seg0 + qi];
      const int buf = op ? Q.b_buf : Q.a_buf;
      const char *X = (const char *)(bufs.data[buf] + (op ? Q.b_off : Q.a_off) * NS);   // see item_split
      // the lane index is recomputed here (volatile: not kept in a register
      // across the K loop); lines past the output read the last one (never stored)
      int ln;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
      const uint32_t line = (uint32_t)(op ? Q.b_line0 + min(T.j0 + 32 * lb + (ln & 31), T.n - 1)
                                          : Q.a_line0 + min(T.i0 + 32 * lb + (ln & 31), T.m - 1));
      const uint32_t kc = (uint32_t)((op ? Q.b_k0 : Q.a_k0) + min(k0 + 16 * lkh + 8 * (ln >> 5), Q.K - 8)) / 8;
      uint32_t hs;
      X += line_offset<NS>(line, op ? Q.b_nl : Q.a_nl, (uint32_t)(op ? Q.b_ld : Q.a_ld), hs);
      X += (uint64_t)(NS * kc) * hs;
      for (int t = 0; t < NS; t++) pre[t] = *(const v4u *)(X + t * hs);
    };
    // ... and from registers into LDS stage st, in the MFMA operand layout
    auto store = [&](int op, const v4u *pre, char *st) {
      if (32 * lb >= (op ? T.n - T.j0 : T.m - T.i0)) return;
      int ln;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
      for (int t = 0; t < NS; t++)
        *(v4u *)(st + (8 * NS * op + (2 * lb + lkh) * NS + t) * 1024 + 16 * ln) = pre[t];
    };
    v16f q[2][slice_groups(NS)];
    for (int b = 0; b < 2; b++)
      for (int g = 0; g < slice_groups(NS); g++) q[b][g] = (v16f){};
    // one K half kh of this step's products from stage st: per block the row
    // block's A slices (those of the block before if it is the same), then
    // the column block's B slices one at a time (slice u
    // meets A slices t <= NS - 1 - u), the next one read while the MFMAs of
    // the current one run; so only five A and two B operands are in registers
    auto compute = [&](const char *st, int k0, int K, int kh) {
      v8bf a[NS];
#pragma unroll
      for (int b = 0; b < 2; b++) {
        if (b >= nb) continue;
        if (b == 0 || br[1] != br[0]) {
          for (int t = 0; t < NS; t++) a[t] = *(const lv8ptr)(st + ((2 * br[b] + kh) * NS + t) * 1024 + 16 * lane);
          if (k0 + 32 > K && k0 + 16 * kh + 8 * h >= K)   // only a segment's last step has such lanes
            for (int t = 0; t < NS; t++) a[t] = (v8bf){};
        }
        const char *bs = st + (8 * NS + (2 * bc[b] + kh) * NS) * 1024 + 16 * lane;
        v8bf x = *(const lv8ptr)bs;
#pragma unroll
        for (int u = 0; u < NS; u++) {
          const v8bf xn = u + 1 < NS ? *(const lv8ptr)(bs + (u + 1) * 1024) : x;
#pragma unroll
          for (int t = 0; t + u < NS; t++)
            q[b][sgroup<NS>(t + u)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], x, q[b][sgroup<NS>(t + u)], 0, 0, 0);
          x = xn;
        }
      }
    };
    // segment descriptors are read where needed (wave-uniform, scalar loads)
    // rather than copied, so that they never sit in scratch memory
    // fold into FP64 with the scale exponents of this lane's column and 16 rows
    // per block, read here (the exponent arrays hold WIDE_EDGE spare entries, so
    // the lines past the output read in bounds; their outputs are never
    // stored).  Exponents are in [-1100, 1100] or the all-zero sentinel, which
    // only meets zero sums: int16 keeps every sum of two in range.
    auto fold = [&]() {
      CSegS &Q = cs[T.seg0 + si];
      const double sc = cg[T.seg0 + si].s;
#pragma unroll
      for (int b = 0; b < 2; b++) {
        if (b >= nb) continue;
        const int32_t *ea = bufs.exps[Q.a_buf] + Q.a_exp + (T.i0 + 32 * br[b] + 4 * h);
        const int f = (int16_t)bufs.exps[Q.b_buf][Q.b_exp + (T.j0 + 32 * bc[b] + c32)];
        for (int r = 0; r < 16; r++) {
          const int er = (int16_t)ea[8 * (r >> 2) + (r & 3)];
          const double x = fold_groups<slice_groups(NS)>(q[b], r);
          acc[b][r] += sc * ldexp(x, er + f - 2 * SLICE_BITS);
        }
        for (int g = 0; g < slice_groups(NS); g++) q[b][g] = (v16f){};
      }
    };
    {
      v4u pa[NS], pb[NS];
      load(si, 0, 0, pa);
      load(si, 0, 1, pb);
      store(0, pa, lds0);
      store(1, pb, lds0);
    }
    int k0 = 0;
    // one step on stage cur; the next one (across segment boundaries) goes
    // through registers into nxt, its loads in flight during the whole step.
    // Returns false after the tile's last step.
    auto step = [&](const char *cur, char *nxt) -> bool {
      __syncthreads();   // every wave's chunks of this step are in cur; nxt is free
      const int K = cs[T.seg0 + si].K;
      int nsi = si, nk0 = k0 + 32;
      const bool newseg = nk0 >= K;
      if (newseg) {
        nk0 = 0;
        nsi++;
        while (nsi < T.nseg && cs[T.seg0 + nsi].K == 0) nsi++;
      }
      const bool more = nsi < T.nseg;
      v4u pa[NS], pb[NS];
      if (more) {
        load(nsi, nk0, 0, pa);
        load(nsi, nk0, 1, pb);
      }
      compute(cur, k0, K, 0);
      compute(cur, k0, K, 1);
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        store(0, pa, nxt);
        store(1, pb, nxt);
      }
      if (newseg || (k0 + 32) % FOLD == 0) fold();
      si = nsi;
      k0 = nk0;
      return more;
    };
    while (step(lds0, lds1) && step(lds1, lds0)) {
    }
  }
  double *C = const_cast<double *>(sbase_ptr(T.c_base, bases, psi, y, work, part)) + T.c_off;
  for (int b = 0; b < nb; b++) {
    const int i0 = T.i0 + 32 * br[b], j = T.j0 + 32 * bc[b] + c32;
    const int ci0 = T.ci0 + 32 * br[b], cj = T.cj0 + 32 * bc[b] + c32;
    for (int r = 0; r < 16; r++) {
      const int i = wrow(r, h);
      if (i0 + i < T.m && j < T.n) {
        double *c = T.rowmajor ? C + (int64_t)(ci0 + i) * T.ldc + cj : C + (int64_t)(ci0 + i) + (int64_t)cj * T.ldc;
        *c = T.accumulate ? *c + (b ? acc[1][r] : acc[0][r]) : b ? acc[1][r] : acc[0][r];
      }
    }
  }
  // first-stage tiles: exponent of every stripe column written (see item_split)
  CSegS &Q0 = cs[T.seg0];
  if (Q0.t_exp >= 0) {
    int32_t *ex = bufs.exps[SBUF_T] + Q0.t_exp;
    for (int b = 0; b < nb; b++) {
      const int i0 = T.i0 + 32 * br[b], j = T.j0 + 32 * bc[b] + c32;
      double m = 0.0;
      for (int r = 0; r < 16; r++)
        if (i0 + wrow(r, h) < T.m && j < T.n) m = fmax(m, fabs(b ? acc[1][r] : acc[0][r]));
      m = fmax(m, __shfl_xor(m, 32));
      if (h == 0 && j < T.n && m > 0.0) {
        int e2;
        const double mant = frexp(m, &e2);
        atomicMax(ex + (T.cj0 + 32 * bc[b] + c32) % Q0.t_nb, mant == 0.5 ? e2 - 1 : e2);
      }
    }
  }
}

template <int NS>
__device__ __forceinline__ void wide_items(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,
                                           const SegS *__restrict__ ssegs, const XcdQueues &q,
                                           int32_t *__restrict__ counters,
                                            int32_t *__restrict__ next_counters,
                                           const double *const *__restrict__ bases, const double *__restrict__ psi,
                                           double *__restrict__ y, double *__restrict__ work,
                                           double *__restrict__ part, const SliceBufs &bufs) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the two operand stages fill the LDS (one work group of eight wavefronts
  // per CU); the next tile's index passes through the second as in macro_items
  __shared__ __attribute__((aligned(1024))) char lds0[wstage_bytes(NS)];
  __shared__ __attribute__((aligned(1024))) char lds1[wstage_bytes(NS)];
  clear_counters(next_counters);
  WorkQueue wq(q, counters, (int)(blockIdx.x / NXCD), (int)(gridDim.x / NXCD), 1);
  for (bool more = true; more;) {
    for (; wq.t < wq.tend; wq.t += wq.step) {
      if (wave == 0 && wq.last()) wq.request(lane == 0);
      const Tile T = tiles[__builtin_amdgcn_readfirstlane(wq.t)];
      wide_split<NS>(T, segs, ssegs, bases, psi, y, work, part, bufs, lds0, lds1, wave, lane);
    }
    __syncthreads();   // everyone has read the last LDS stage
    if (wave == 0) {
      const int v = wq.next(lane) ? wq.t : -1;
      if (lane == 0) *(volatile int *)lds1 = v;
    }
    __syncthreads();
    wq.t = __builtin_amdgcn_readfirstlane(*(volatile int *)lds1);
    more = wq.t >= 0;
    wq.tend = wq.t + 1;
    wq.step = 1;
  }
}

#define WIDE_KERNELS(NS)                                                                                    \
  __global__ void __launch_bounds__(64 * WIDE_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))           \
  stage1_wsplit##NS##_kernel(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,                  \
                             const SegS *__restrict__ ssegs, XcdQueues q, int32_t *__restrict__ counters,   \
                             int32_t *__restrict__ next_counters,\
                             const double *const *__restrict__ bases, const double *__restrict__ psi,       \
                             double *__restrict__ y, double *__restrict__ work, double *__restrict__ part,   \
                             SliceBufs bufs) {                                                              \
    wide_items<NS>(tiles, segs, ssegs, q, counters, next_counters, bases, psi, y, work, part, bufs);                       \
  }                                                                                                         \
  __global__ void __launch_bounds__(64 * WIDE_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))           \
  stage2_wsplit##NS##_kernel(const Tile *__restrict__ tiles, const Seg *__restrict__ segs,                  \
                             const SegS *__restrict__ ssegs, XcdQueues q, int32_t *__restrict__ counters,   \
                             int32_t *__restrict__ next_counters,\
                             const double *const *__restrict__ bases, const double *__restrict__ psi,       \
                             double *__restrict__ y, double *__restrict__ work, double *__restrict__ part,   \
                             SliceBufs bufs) {                                                              \
    wide_items<NS>(tiles, segs, ssegs, q, counters, next_counters, bases, psi, y, work, part, bufs);                       \
  }

WIDE_KERNELS(3)
WIDE_KERNELS(4)
WIDE_KERNELS(5)

#define SPLIT_KERNELS(NS)                                                                                   \
  __global__ void __launch_bounds__(64 * SPLIT_WAVES, 2) stage1_split##NS##_kernel(                                  \
      const Tile *__restrict__ tiles, const Seg *__restrict__ segs, const SegS *__restrict__ ssegs,         \
      XcdQueues q, int32_t *__restrict__ counters, int32_t *__restrict__ next_counters, int chunk,               \
      const double *const *__restrict__ bases,                 \
      const double *__restrict__ psi, double *__restrict__ y, double *__restrict__ work,                    \
      double *__restrict__ part, SliceBufs bufs) {                                                          \
    items_split<NS>(tiles, segs, ssegs, q, counters, next_counters, chunk, bases, psi, y, work, part, bufs);                      \
  }                                                                                                         \
  __global__ void __launch_bounds__(64 * SPLIT_WAVES, 2) stage2_split##NS##_kernel(                                  \
      const Tile *__restrict__ tiles, const Seg *__restrict__ segs, const SegS *__restrict__ ssegs,         \
      XcdQueues q, int32_t *__restrict__ counters, int32_t *__restrict__ next_counters, int chunk,               \
      const double *const *__restrict__ bases,                 \
      const double *__restrict__ psi, double *__restrict__ y, double *__restrict__ work,                    \
      double *__restrict__ part, SliceBufs bufs) {                                                          \
    items_split<NS>(tiles, segs, ssegs, q, counters, next_counters, chunk, bases, psi, y, work, part, bufs);                      \
  }

SPLIT_KERNELS(3)
SPLIT_KERNELS(4)
SPLIT_KERNELS(5)
SPLIT_KERNELS(6)
SPLIT_KERNELS(7)

void launch_macro_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles, double flops,
                        const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                        const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream) {
  if (ntiles <= 0) return;
  hipStream_t s = (hipStream_t)stream;
  // two work groups resident per CU (80 KiB of LDS each at s = 5); every work
  // group takes tiles until all queues are empty
  const int grid = std::max(8, std::min((ntiles + 7) / 8 * 8, MACRO_GRID));
  const XcdQueues dq = deal(q, grid / NXCD, heavy_tiles(ntiles, flops));
#define MLAUNCH(NS)                                                                                         \
  if (nslices == NS) {                                                                                      \
    if (stage == 1)                                                                                         \
      hipLaunchKernelGGL(stage1_msplit##NS##_kernel, dim3(grid), dim3(64 * WAVES), 0, s, tiles, segs, ssegs,  \
                         dq, qs.cur(), qs.other(), bases, psi, y, work, part, bufs);           \
    else                                                                                                    \
      hipLaunchKernelGGL(stage2_msplit##NS##_kernel, dim3(grid), dim3(64 * WAVES), 0, s, tiles, segs, ssegs,  \
                         dq, qs.cur(), qs.other(), bases, psi, y, work, part, bufs);           \
    qs.launch++;                                                                                            \
    return;                                                                                                 \
  }
  MLAUNCH(3)
  MLAUNCH(4)
  MLAUNCH(5)
  MLAUNCH(6)
  MLAUNCH(7)
#undef MLAUNCH
}

void launch_wide_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles, double flops,
                       const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                       const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream) {
  if (ntiles <= 0) return;
  hipStream_t s = (hipStream_t)stream;
  // one work group per CU (the two stages take all 160 KiB of LDS at s = 5)
  const int grid = std::max(8, std::min((ntiles + 7) / 8 * 8, WIDE_GRID));
  const XcdQueues dq = deal(q, grid / NXCD, heavy_tiles(ntiles, flops));
#define WLAUNCH(NS)                                                                                         \
  if (nslices == NS) {                                                                                      \
    if (stage == 1)                                                                                         \
      hipLaunchKernelGGL(stage1_wsplit##NS##_kernel, dim3(grid), dim3(64 * WIDE_WAVES), 0, s, tiles, segs,  \
                         ssegs, dq, qs.cur(), qs.other(), bases, psi, y, work, part, bufs);    \
    else                                                                                                    \
      hipLaunchKernelGGL(stage2_wsplit##NS##_kernel, dim3(grid), dim3(64 * WIDE_WAVES), 0, s, tiles, segs,  \
                         ssegs, dq, qs.cur(), qs.other(), bases, psi, y, work, part, bufs);    \
    qs.launch++;                                                                                            \
    return;                                                                                                 \
  }
  WLAUNCH(3)
  WLAUNCH(4)
  WLAUNCH(5)
#undef WLAUNCH
}

void launch_tiles_split(int stage, const Tile *tiles, const Seg *segs, const SegS *ssegs, int ntiles,
                        double flops, const XcdQueues &q, QueueSets &qs, int nslices, const double *const *bases,
                        const double *psi, double *y, double *work, double *part, SliceBufs bufs, void *stream) {
  if (ntiles <= 0) return;
  hipStream_t s = (hipStream_t)stream;
  // work groups that the LDS stages let run at once
  const int resident = 256 * std::max(1, LDS_BYTES / (SPLIT_WAVES * stage_bytes(nslices)));
  const int grid = wave_grid(ntiles, resident, SPLIT_WAVES), chunk = wave_chunk(ntiles, flops);
  const XcdQueues dq = deal(q, grid / NXCD * SPLIT_WAVES, false);
#define LAUNCH(NS)                                                                                          \
  if (nslices == NS) {                                                                                      \
    if (stage == 1)                                                                                         \
      hipLaunchKernelGGL(stage1_split##NS##_kernel, dim3(grid), dim3(64 * SPLIT_WAVES), 0, s, tiles, segs, ssegs,   \
                         dq, qs.cur(), qs.other(), chunk, bases, psi, y, work, part, bufs);           \
    else                                                                                                    \
      hipLaunchKernelGGL(stage2_split##NS##_kernel, dim3(grid), dim3(64 * SPLIT_WAVES), 0, s, tiles, segs, ssegs,   \
                         dq, qs.cur(), qs.other(), chunk, bases, psi, y, work, part, bufs);           \
    qs.launch++;                                                                                            \
    return;                                                                                                 \
  }
  LAUNCH(3)
  LAUNCH(4)
  LAUNCH(5)
  LAUNCH(6)
  LAUNCH(7)
#undef LAUNCH
}

}  // namespace dmrg
