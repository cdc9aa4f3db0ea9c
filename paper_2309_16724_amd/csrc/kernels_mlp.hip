// Learned Davidson preconditioner: forward, backward and Adam kernels of the
// 3-layer perceptron g = w3 . relu(W2 relu(W1 x + b1) + b2) + b3 (FP32
// storage; reductions of the backward pass accumulate in FP64 in a fixed
// order, so every result is reproducible bit for bit).
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include "mlp.hpp"

namespace dmrg {

namespace {

constexpr int NT = 256;     // threads per block

struct POff {
  int64_t W1, b1, W2, b2, w3, b3;
};
__host__ __device__ inline POff poff(int W) {
  POff o;
  o.W1 = 0;
  o.b1 = (int64_t)MLP_IN * W;
  o.W2 = o.b1 + W;
  o.b2 = o.W2 + (int64_t)W * W;
  o.w3 = o.b2 + W;
  o.b3 = o.w3 + W;
  return o;
}

__device__ inline double floored(double den, double fl) {
  return fabs(den) < fl ? (den < 0.0 ? -fl : fl) : den;
}

__device__ inline int seg_of(const int64_t *off, int nseg, int64_t i) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

typedef float v4f __attribute__((ext_vector_type(4)));

// Output row (within a wavefront's 16) of accumulator element r held by lane
// group q = lane / 16 in v_mfma_f32_16x16x4f32; the column is lane % 16.
// Operands: A[lane % 16][lane / 16], B[lane / 16][lane % 16].
__device__ constexpr int mfma_row(int q, int r) { return 4 * q + r; }

// Features (x0, x1) and, in MODE 1, the diagonal step td of row i.
template <int MODE>
__device__ inline void row_inputs(const FwdArgs &A, const FwdSegs &S, int64_t i, float &f0, float &f1, double &td) {
  f0 = f1 = 0.0f;
  td = 0.0;
  if (i >= A.n) return;
  if (MODE == 0) {
    f0 = A.x[i * MLP_IN];
    f1 = A.x[i * MLP_IN + 1];
  } else {
    double theta, sigma, floor_, feature;
    if (A.theta) {
      const int s = seg_of(A.seg_off, A.nseg, i);
      theta = A.theta[s];
      sigma = A.sigma[s];
      floor_ = A.floor_[s];
      feature = A.f1[s];
    } else {
      int s = 0;
      for (int k = 1; k < A.nseg; k++) s += i >= S.off[k];
      theta = S.theta[s];
      sigma = S.sigma[s];
      floor_ = S.floor_[s];
      feature = S.f1[s];
    }
    const double den = A.d[i] - theta;
    td = -A.r[i] / floored(den, floor_);
    f0 = (float)asinh(den / sigma);
    f1 = (float)feature;
  }
}

// pre-activation of layer 1 (the backward pass computes it again)
__device__ __forceinline__ float layer1(float b1, float w10, float w11, float f0, float f1) {
  return fmaf(f1, w11, fmaf(f0, w10, b1));
}

// MODE 0: rows from x[n][2], g out, optional activations z2 (training).
// MODE 1: rows from Davidson vectors; t[i] = td_i (1 + g_i), td = -r/(d - theta).
//
// Four wavefronts as 4 / CS row groups of 16 rows and CS column groups of
// W / CS columns.  Lane l computes layer 1 of row l % 16 at k = 4j + l / 16, the
// A operand of step j of layer 2, when that step comes (two multiply-adds from
// W1 and b1 in LDS: kept for all k they took W / 4 registers and three global
// loads each); layer 2 runs on v_mfma_f32_16x16x4f32 with W2 going through
// registers into one of two LDS chunks of 16 rows while the chunk before is
// used (row stride W + 16: the four rows an operand read touches lie in
// different banks).  Layer 3 sums a row's columns in 16 lanes, each every
// sixteenth column in rising order, then over the lanes; column groups hand
// their layer-2 outputs over in LDS for it, so that a row's result does not
// depend on the rows beside it (with a sum per column group the gradient of
// 4096 rows at width 64 was 4.96e-8 off, 4.84e-8 this way, at the same time).
// Bound: the FP32 matrix rate.  CS = 4 is for few rows: at 4096 rows, width 256,
// CS = 1 is 64 work groups on 256 CUs, 33 us, CS = 4 is 256 of them, 17 us.
template <int W, int MODE, int CS>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) mlp_fwd_kernel(const FwdArgs A, const FwdSegs S) {
  constexpr int NB = W / 16 / CS, KC = 16, LD = W + 16, RG = 4 / CS, ROWS = 16 * RG;
  static_assert(W % (16 * CS) == 0 && (KC * W / 4) % NT == 0 || W < 64, "whole chunks");
  static_assert(CS == 1 || (CS == 4 && W / KC % 2 == 0), "16 rows a work group, the last chunk is chunk 1");
  __shared__ float w2c[2][KC][LD];
  __shared__ float l1[3][W];
  const POff o = poff(W);
  const float *__restrict__ p = A.params;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, q = lane >> 4;
  const int rg = wave / CS, cg = wave % CS;
  const int64_t base = (int64_t)blockIdx.x * ROWS + rg * 16;
  const int c0 = cg * (W / CS);
  constexpr int V = KC * W / 4;                    // float4 per chunk
  constexpr int PER = (V + NT - 1) / NT;
  v4f pre[PER];
  auto load = [&](int k0) {
#pragma unroll
    for (int e = 0; e < PER; e++) {
      const int v = tid + e * NT;
      if (V % NT == 0 || v < V) {
        const float *s = p + o.W2 + (int64_t)k0 * W + 4 * v;   // W2 starts at a multiple of 4 floats only for
        pre[e] = (v4f){s[0], s[1], s[2], s[3]};                // 3 W % 4 == 0: four loads, merged when aligned
      }
    }
  };
  auto store = [&](int b) {
#pragma unroll
    for (int e = 0; e < PER; e++) {
      const int v = tid + e * NT;
      if (V % NT == 0 || v < V) *(v4f *)&w2c[b][4 * v / W][4 * v % W] = pre[e];
    }
  };
  load(0);
  for (int e = tid; e < W; e += NT) {
    l1[0][e] = p[o.b1 + e];
    l1[1][e] = p[o.W1 + e];
    l1[2][e] = p[o.W1 + W + e];
  }
  float f0, f1;
  double td;
  row_inputs<MODE>(A, S, base + l16, f0, f1, td);
  store(0);
  v4f acc[NB];
#pragma unroll
  for (int bj = 0; bj < NB; bj++) acc[bj] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < W; k0 += KC) {
    const int b = (k0 / KC) & 1;
    __syncthreads();   // chunk b is in LDS, the other one is free
    if (k0 + KC < W) load(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      const int k = k0 + kk + q;
      const float a = fmaxf(layer1(l1[0][k], l1[1][k], l1[2][k], f0, f1), 0.0f);
#pragma unroll
      for (int bj = 0; bj < NB; bj++)
        acc[bj] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w2c[b][kk + q][c0 + 16 * bj + l16], acc[bj], 0, 0, 0);
    }
    if (k0 + KC < W) store(1 - b);
  }
  // layer 3
  const float b3 = p[o.b3];
  float w3s[CS > 1 ? W / 16 : 1];
  if (CS > 1) {
#pragma unroll
    for (int e = 0; e < W / 16; e++) w3s[CS > 1 ? e : 0] = p[o.w3 + 16 * e + l16];   // in flight until the barrier
  }
  float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int bj = 0; bj < NB; bj++) {
    const int c = c0 + 16 * bj + l16;
    const float bb = p[o.b2 + c], w3 = p[o.w3 + c];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const float z = acc[bj][r] + bb;
      const int64_t orow = base + mfma_row(q, r);
      if (MODE == 0 && A.z2 && orow < A.n) A.z2[orow * W + c] = z;
      // (the last K step read chunk 1: chunk 0 is free)
      if (CS > 1) w2c[0][mfma_row(q, r)][c] = fmaxf(z, 0.0f);
      else part[r] = fmaf(fmaxf(z, 0.0f), w3, part[r]);
    }
  }
  if (CS > 1) {
    // wavefront w sums rows 4 w + q over all columns as CS = 1 does
    __syncthreads();
    const int row = 4 * wave + q;
#pragma unroll
    for (int e = 0; e < W / 16; e++) part[0] = fmaf(w2c[0][row][16 * e + l16], w3s[CS > 1 ? e : 0], part[0]);
    for (int m = 8; m > 0; m >>= 1) part[0] += __shfl_xor(part[0], m, 16);
    const double tdr = MODE == 1 ? __shfl(td, row) : 0.0;
    const int64_t orow = base + row;
    if (l16 != 0 || orow >= A.n) return;
    const float g = part[0] + b3;
    if (MODE == 0) A.g[orow] = g;
    else A.t[orow] = tdr * (1.0 + (double)g);
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; r++)
    for (int m = 8; m > 0; m >>= 1) part[r] += __shfl_xor(part[r], m, 16);
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int64_t orow = base + mfma_row(q, r);
    const double tdr = MODE == 1 ? __shfl(td, mfma_row(q, r)) : 0.0;   // held by the lane of that row
    if (l16 != 0 || orow >= A.n) continue;
    const float g = part[r] + b3;
    if (MODE == 0) A.g[orow] = g;
    else A.t[orow] = tdr * (1.0 + (double)g);
  }
}

// dg_i = 2 e_i a_i / n, e_i = a_i (1 + g_i) - b_i; per-block partial sums of e^2
__global__ void __launch_bounds__(NT) out_grad_kernel(const float *__restrict__ g, const float *__restrict__ a,
                                                      const float *__restrict__ b, int64_t n,
                                                      float *__restrict__ dg, double *__restrict__ lpart) {
  __shared__ double red[NT];
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  double e2 = 0.0;
  if (i < n) {
    const float e = a[i] * (1.0f + g[i]) - b[i];
    dg[i] = 2.0f * e * a[i] / (float)n;
    e2 = (double)e * (double)e;
  }
  red[threadIdx.x] = e2;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) lpart[blockIdx.x] = red[0];
}

typedef double v4d __attribute__((ext_vector_type(4)));

// gradient of the layer-2 pre-activation
__device__ __forceinline__ float dz2_of(float z2, float dg, float w3) { return z2 > 0.0f ? dg * w3 : 0.0f; }

// dz1[i][k] = (sum_j dz2[i][j] W2[k][j]) [z1[i][k] > 0], products and sums in
// FP64 on the matrix cores (v_mfma_f64_16x16x4: A[l%16][l/16], B[l/16][l%16],
// D[l/16 + 4r][l%16]).  A wavefront computes 16 rows x CB blocks of 16 columns;
// lane group l / 16 takes j = 16 s + 4 (l / 16) + e in step e, so that every
// lane reads four consecutive j of both operands at once.
template <int W>
__global__ void __launch_bounds__(NT) dz1_kernel(const float *__restrict__ params, const float *__restrict__ x,
                                                 const float *__restrict__ dg, const float *__restrict__ z2,
                                                 int64_t n, float *__restrict__ dz1) {
  constexpr int CB = W >= 64 ? 4 : W / 16, CG = W / (16 * CB);   // column groups
  const POff o = poff(W);
  const float *W2 = params + o.W2, *w3 = params + o.w3;
  const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t i0 = w / CG * 16;
  const int c0 = (int)(w % CG) * 16 * CB;
  if (i0 >= n) return;
  const int64_t row = min(i0 + l16, n - 1);
  const float dgi = dg[row];
  v4d acc[CB];
#pragma unroll
  for (int b = 0; b < CB; b++) acc[b] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int s = 0; s < W; s += 16) {
    const int j = s + 4 * q;
    float a[4], bw[CB][4];
#pragma unroll
    for (int e = 0; e < 4; e++) a[e] = dz2_of(z2[row * W + j + e], dgi, w3[j + e]);
#pragma unroll
    for (int b = 0; b < CB; b++)
#pragma unroll
      for (int e = 0; e < 4; e++) bw[b][e] = W2[(int64_t)(c0 + 16 * b + l16) * W + j + e];
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int b = 0; b < CB; b++)
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[e], (double)bw[b][e], acc[b], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int64_t i = i0 + q + 4 * r;
    if (i >= n) continue;
    const float f0 = x[i * MLP_IN], f1 = x[i * MLP_IN + 1];
#pragma unroll
    for (int b = 0; b < CB; b++) {
      const int k = c0 + 16 * b + l16;
      const float z1 = layer1(params[o.b1 + k], params[o.W1 + k], params[o.W1 + W + k], f0, f1);
      dz1[i * W + k] = z1 > 0.0f ? (float)acc[b][r] : 0.0f;
    }
  }
}

// Row splits of the gradient's sums over rows: at most 64 of dW2 (a multiple of
// 16 rows, at least 256) and 256 of the column sums (at least 64 rows).
struct Splits {
  int64_t rows2;
  int n2;
  int64_t rowsv;
  int nv;
};
__host__ __device__ inline Splits splits_of(int64_t n) {
  Splits s;
  s.rows2 = (n + 63) / 64;
  s.rows2 = s.rows2 < 256 ? 256 : (s.rows2 + 15) / 16 * 16;
  s.n2 = (int)((n + s.rows2 - 1) / s.rows2);
  s.rowsv = (n + 255) / 256;
  s.rowsv = s.rowsv < 64 ? 64 : s.rowsv;
  s.nv = (int)((n + s.rowsv - 1) / s.rowsv);
  return s;
}
// partial sums: [n2][W][W] of dW2, then [nv][5 W + 1]: dW1 (2 W), db1, db2, dw3, db3

// Partial sums over row splits, FP64 throughout.  Blocks [0, nb2): dW2 =
// relu(z1)^T dz2, a 32 x 32 tile of one split per wavefront on the FP64 matrix
// cores, four K steps (16 rows) loaded at a time; the other blocks: column
// sums, one thread per column.  With one work group per 32 x 32 tile walking
// all rows in FP64 vector code this took 6 x 353 us at 4096 rows.
template <int W>
__global__ void __launch_bounds__(NT) grad_part_kernel(const float *__restrict__ params, const float *__restrict__ x,
                                                       const float *__restrict__ dg, const float *__restrict__ z2,
                                                       const float *__restrict__ dz1, int64_t n, int nb2,
                                                       double *__restrict__ part) {
  const POff o = poff(W);
  const Splits sp = splits_of(n);
  if ((int)blockIdx.x < nb2) {
    constexpr int T = W / 32;
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const int w = (int)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= sp.n2 * T * T) return;
    const int split = w / (T * T), m0 = w / T % T * 32, j0 = w % T * 32;
    const int64_t r0 = split * sp.rows2, r1 = min(n, r0 + sp.rows2);
    float b1[2], w10[2], w11[2], w3[2];
#pragma unroll
    for (int b = 0; b < 2; b++) {
      const int m = m0 + 16 * b + l16;
      b1[b] = params[o.b1 + m];
      w10[b] = params[o.W1 + m];
      w11[b] = params[o.W1 + W + m];
      w3[b] = params[o.w3 + j0 + 16 * b + l16];
    }
    v4d acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int b = 0; b < 2; b++) acc[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
    float f0[4], f1[4], d[4], z[4][2];
    auto load = [&](int64_t i0) {   // rows past the end read the last one
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int64_t i = i0 + 4 * e + q, ic = min(i, r1 - 1);
        f0[e] = x[ic * MLP_IN];
        f1[e] = x[ic * MLP_IN + 1];
        d[e] = dg[ic];
#pragma unroll
        for (int b = 0; b < 2; b++) z[e][b] = z2[ic * W + j0 + 16 * b + l16];
      }
    };
    load(r0);
    for (int64_t i0 = r0; i0 < r1; i0 += 16) {
      double av[4][2], bv[4][2];
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int b = 0; b < 2; b++) {
          av[e][b] = (double)fmaxf(layer1(b1[b], w10[b], w11[b], f0[e], f1[e]), 0.0f);
          bv[e][b] = (double)dz2_of(z[e][b], d[e], w3[b]);
        }
      // ... and are zeros in both operands: zero times what the last row holds
      // would make an infinite sum a NaN
      if (i0 + 16 > r1) {
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int b = 0; b < 2; b++)
            if (i0 + 4 * e + q >= r1) av[e][b] = bv[e][b] = 0.0;
      }
      load(min(i0 + 16, r1 - 1));
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
          for (int b = 0; b < 2; b++)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[e][a], bv[e][b], acc[a][b], 0, 0, 0);
    }
    double *out = part + (int64_t)split * W * W;
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
      for (int b = 0; b < 2; b++)
#pragma unroll
        for (int r = 0; r < 4; r++)
          out[(int64_t)(m0 + 16 * a + q + 4 * r) * W + j0 + 16 * b + l16] = acc[a][b][r];
    return;
  }
  const int split = (int)blockIdx.x - nb2;
  const int64_t r0 = split * sp.rowsv, r1 = min(n, r0 + sp.rowsv);
  double *out = part + (int64_t)sp.n2 * W * W + (int64_t)split * (5 * W + 1);
  for (int c = threadIdx.x; c < W; c += NT) {
    const float w3 = params[o.w3 + c];
    double s0 = 0.0, s1 = 0.0, sb1 = 0.0, sb2 = 0.0, sw3 = 0.0, sb3 = 0.0;
#pragma unroll 8
    for (int64_t i = r0; i < r1; i++) {
      const float d = dg[i], z = z2[i * W + c], e = dz1[i * W + c];
      s0 += (double)x[i * MLP_IN] * (double)e;
      s1 += (double)x[i * MLP_IN + 1] * (double)e;
      sb1 += (double)e;
      sb2 += (double)dz2_of(z, d, w3);
      sw3 += (double)d * (double)fmaxf(z, 0.0f);
      sb3 += (double)d;
    }
    out[c] = s0;
    out[W + c] = s1;
    out[2 * W + c] = sb1;
    out[3 * W + c] = sb2;
    out[4 * W + c] = sw3;
    if (c == 0) out[5 * W] = sb3;
  }
}

// gradient = sum of the partial sums in split order
template <int W>
__global__ void __launch_bounds__(NT) grad_sum_kernel(const double *__restrict__ part, int64_t n,
                                                      float *__restrict__ grad) {
  const POff o = poff(W);
  const Splits sp = splits_of(n);
  const int e = blockIdx.x * NT + threadIdx.x;
  if (e < W * W) {
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < sp.n2; k++) s += part[(int64_t)k * W * W + e];
    grad[o.W2 + e] = (float)s;
    return;
  }
  const int v = e - W * W;
  if (v > 5 * W) return;
  const double *pv = part + (int64_t)sp.n2 * W * W + v;
  double s = 0.0;
#pragma unroll 8
  for (int k = 0; k < sp.nv; k++) s += pv[(int64_t)k * (5 * W + 1)];
  const int64_t at = v < 2 * W ? o.W1 + v : v < 3 * W ? o.b1 + v - 2 * W : v < 4 * W ? o.b2 + v - 3 * W
                   : v < 5 * W ? o.w3 + v - 4 * W : o.b3;
  grad[at] = (float)s;
}

// p -= lr mhat / (sqrt(vhat) + eps), mhat = m c1, vhat = v c2
__global__ void __launch_bounds__(NT) adam_kernel(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                                  const float *__restrict__ gr, int64_t n, float lr, float b1,
                                                  float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (i >= n) return;
  const float g = gr[i];
  const float mi = b1 * m[i] + (1.0f - b1) * g;
  const float vi = b2 * v[i] + (1.0f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// SplitMix64 (Steele, Lea & Flood 2014) as a counter-based index generator
__device__ inline uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// minibatch gather: row j of the batch is sample splitmix64(seed + step * 2^32 + j) mod n
__global__ void __launch_bounds__(NT) gather_kernel(const float *__restrict__ x, const float *__restrict__ a,
                                                    const float *__restrict__ b, int64_t n, uint64_t seed,
                                                    uint64_t step, int batch, float *__restrict__ xb,
                                                    float *__restrict__ ab, float *__restrict__ bb) {
  const int j = blockIdx.x * NT + threadIdx.x;
  if (j >= batch) return;
  const int64_t i = (int64_t)(splitmix64(seed + (step << 32) + (uint64_t)j) % (uint64_t)n);
  xb[j * MLP_IN] = x[i * MLP_IN];
  xb[j * MLP_IN + 1] = x[i * MLP_IN + 1];
  ab[j] = a[i];
  bb[j] = b[i];
}

// training rows of one recorded iteration: ts = psi* c - u (c = 1/<u|psi*>),
// x = (asinh((d - theta)/sigma), f1), a = td s, b = ts s, s = sqrt(n)/||ts||,
// both scaled by MLP_A_MAX/|a| where |a| exceeds MLP_A_MAX
__global__ void __launch_bounds__(NT) collect_kernel(const double *__restrict__ d, const double *__restrict__ r,
                                                     const double *__restrict__ ts, int64_t n, double theta,
                                                     double sigma, double f1, double s, double floor_,
                                                     float *__restrict__ x, float *__restrict__ a,
                                                     float *__restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (i >= n) return;
  const double den = d[i] - theta;
  x[i * MLP_IN] = (float)asinh(den / sigma);
  x[i * MLP_IN + 1] = (float)f1;
  const double av = -r[i] / floored(den, floor_) * s;
  const double w = fabs(av) > MLP_A_MAX ? MLP_A_MAX / fabs(av) : 1.0;
  a[i] = (float)(av * w);
  b[i] = (float)(ts[i] * s * w);
}

__global__ void __launch_bounds__(NT) exact_corr_kernel(const double *__restrict__ psi, const double *__restrict__ u,
                                                        int64_t n, double c, double *__restrict__ ts) {
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (i < n) ts[i] = psi[i] * c - u[i];
}

inline dim3 grid1(int64_t n) { return dim3((unsigned)((n + NT - 1) / NT)); }

}  // namespace

bool mlp_width_ok(int W) { return W == 32 || W == 64 || W == 128 || W == 256; }

void launch_mlp_forward(int W, int mode, const FwdArgs &A, const FwdSegs &S, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  // column groups where 64-row work groups would not give every CU two.  (Width
  // 256: 4096 rows 17 us against 33 without, 20000 rows 43 against 48, 32768 rows
  // 57 against 49: beyond some 25000 rows the line could lie lower.)
  const bool few = W >= 64 && A.n <= 64 * 512;
  const dim3 grid((unsigned)(few ? (A.n + 15) / 16 : (A.n + 63) / 64));
#define FWD(w, cs)                                                                                     \
  {                                                                                                    \
    if (mode == 0) hipLaunchKernelGGL((mlp_fwd_kernel<w, 0, cs>), grid, dim3(NT), 0, s, A, S);         \
    else hipLaunchKernelGGL((mlp_fwd_kernel<w, 1, cs>), grid, dim3(NT), 0, s, A, S);                   \
  }
  switch (W) {
    case 32: FWD(32, 1) break;
    case 64: if (few) FWD(64, 4) else FWD(64, 1) break;
    case 128: if (few) FWD(128, 4) else FWD(128, 1) break;
    case 256: if (few) FWD(256, 4) else FWD(256, 1) break;
    default: break;
  }
#undef FWD
}

int64_t mlp_part_elems(int W, int64_t n) {
  // splits_of grows with n up to its limits (64 and 256)
  const int64_t n2 = std::min<int64_t>(64, (n + 255) / 256), nv = std::min<int64_t>(256, (n + 63) / 64);
  return n2 * W * W + nv * (5 * W + 1);
}

void launch_mlp_backward(int W, const float *params, const float *x, const float *a, const float *b, int64_t n,
                         const float *g, const float *z2, float *dg, float *dz1, double *lpart, double *part,
                         float *grad, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const Splits sp = splits_of(n);
  hipLaunchKernelGGL(out_grad_kernel, grid1(n), dim3(NT), 0, s, g, a, b, n, dg, lpart);
  const int t = W / 32, nb2 = (sp.n2 * t * t + 3) / 4;
  const int64_t waves1 = (n + 15) / 16 * (W >= 64 ? W / 64 : 1);
#define BWD(w)                                                                                             \
  case w:                                                                                                  \
    hipLaunchKernelGGL(dz1_kernel<w>, dim3((unsigned)((waves1 + 3) / 4)), dim3(NT), 0, s, params, x, dg, z2, n, dz1); \
    hipLaunchKernelGGL(grad_part_kernel<w>, dim3((unsigned)(nb2 + sp.nv)), dim3(NT), 0, s, params, x, dg, z2, dz1, n, \
                       nb2, part);                                                                         \
    hipLaunchKernelGGL(grad_sum_kernel<w>, dim3((w * w + 5 * w + 1 + NT - 1) / NT), dim3(NT), 0, s, part, n, grad);   \
    break;
  switch (W) { BWD(32) BWD(64) BWD(128) BWD(256) default: break; }
#undef BWD
}

void launch_adam(float *p, float *m, float *v, const float *gr, int64_t n, float lr, float b1, float b2, float eps,
                 float c1, float c2, void *stream) {
  hipLaunchKernelGGL(adam_kernel, grid1(n), dim3(NT), 0, (hipStream_t)stream, p, m, v, gr, n, lr, b1, b2, eps, c1,
                     c2);
}

void launch_gather(const float *x, const float *a, const float *b, int64_t n, uint64_t seed, uint64_t step, int batch,
                   float *xb, float *ab, float *bb, void *stream) {
  hipLaunchKernelGGL(gather_kernel, grid1(batch), dim3(NT), 0, (hipStream_t)stream, x, a, b, n, seed, step, batch,
                     xb, ab, bb);
}

void launch_exact_corr(const double *psi, const double *u, int64_t n, double c, double *ts, void *stream) {
  hipLaunchKernelGGL(exact_corr_kernel, grid1(n), dim3(NT), 0, (hipStream_t)stream, psi, u, n, c, ts);
}

void launch_collect(const double *d, const double *r, const double *ts, int64_t n, double theta, double sigma,
                    double f1, double s, double floor_, float *x, float *a, float *b, void *stream) {
  hipLaunchKernelGGL(collect_kernel, grid1(n), dim3(NT), 0, (hipStream_t)stream, d, r, ts, n, theta, sigma, f1, s,
                     floor_, x, a, b);
}

}  // namespace dmrg
