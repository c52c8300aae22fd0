// gptq.hip -- the GPTQ quantizer the paper applies to every expert (Sec. 3.1:
// Hessian H = 2 X^T X of the layer-wise squared error, columns quantized in
// order with each column's error compensated on the columns after it), on
// the packed format of the Sec. 3.1 group quantizer.  All arithmetic fp64.
//
// Three steps, each its own entry point:
//   hessian   H (+)= 2 X^T X from bf16 calibration inputs X [N][K];
//   factor    dead inputs (H_kk = 0 -> H_kk = 1), damping H += damp * mean(diag
//             H) * I, and U, the upper Cholesky factor of H^-1 (H^-1 = U^T U);
//   quantize  for k = 0 .. K-1: at a group start the Sec. 3.1 scale/zero of
//             the fp32 rounding of the group's current values; q_k = nearest
//             level of fp32(w_k); e_k = (w_k - s (q_k - z)) / U_kk; w_j -= e_k
//             U_kj for j > k.  Codes and scale/zero go straight into the
//             layer's packed storage.
//
// U without forming H^-1: with J the index reversal, J H J = L L^T (lower
// Cholesky) gives H = V V^T with V = J L J upper triangular, so H^-1 =
// V^-T V^-1 and U = V^-1 = J L^-1 J.  The factor step therefore runs one
// blocked Cholesky and one recursive triangular inverse on the reversed matrix.
//
// Kernels: fp64 MFMA GEMMs on 64 x 64 tiles carry the Hessian (lower tiles,
// mirrored), the Cholesky trailing updates and the inverse's corner blocks;
// GPTQ's deferred updates run one column after the other with every product
// and subtraction rounded, which no MFMA does, on a register-tiled fp64 kernel;
// the sequential parts are one workgroup (64 x 64 Cholesky) and four lanes per
// row (panel solve, GPTQ column loop).
#include <type_traits>

#include "mc_internal.hpp"

namespace mc {

constexpr int kNb = 64;            // Cholesky / inverse block, GEMM tile
constexpr int kOb = 256;           // columns of a Cholesky panel between trailing updates
constexpr int kQb = 128;           // GPTQ column block
constexpr int kQo = 512;           // columns quantized between updates of the columns after them
constexpr int kQRows = 64;         // rows of a GPTQ workgroup (four wavefronts)

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// D += A B on 16 x 16 x 4: lane l holds A[l % 16][l / 16], B[l / 16][l % 16]
// and, in register i, D[4 i + l / 16][l % 16].
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- GEMMs --
// C (=, +=) alpha A B on 64 x 64 tiles of fp64 matrices, M, N and Kc multiples
// of 64: A(m, k) = A[m * lda + k]; B(k, n) = B[k * ldb + n], or B[n * ldb + k]
// with BT.  Four waves, 32 x 32 outputs each (four MFMA tiles); 16 columns of
// the reduction at a time go through LDS, the next 16 are loaded meanwhile.
// The MFMAs' sums are added to the totals (C's values to begin with, when they
// accumulate) every 64 columns: sums over a whole 256-column panel doubled the
// factor's error.
struct GemmF64 {
  const double* A;
  const double* B;
  double* C;
  long long lda, ldb, ldc;
  double alpha;
};

constexpr int kGemmK = 16;
constexpr int kGemmLd = kNb + 4;   // rows of the staged tiles start 4 doubles apart

// ACCUM: C += (else C =).
template <bool BT, bool ACCUM>
__device__ __forceinline__ void gemm_tile_f64(const GemmF64& g, int m0, int n0, int k_begin, int k_end) {
  __shared__ double As[kGemmK][kGemmLd];
  __shared__ double Bs[kGemmK][kGemmLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = 32 * (wave >> 1), wn = 32 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
  // k-fast operands: rows tid / 8 and +32, columns 2 (tid % 8) and +1 (a
  // 128-byte row piece per 8 lanes); n-fast: row tid / 16, columns 4 (tid % 16)
  const int kr = tid >> 3, kc = 2 * (tid & 7), nr = tid >> 4, nc = 4 * (tid & 15);
  f64x2 a[2], b[2];
  auto load = [&](int k0) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const double* pa = g.A + (long long)(m0 + kr + 32 * p) * g.lda + k0 + kc;
      a[p] = f64x2{pa[0], pa[1]};
      const double* pb = BT ? g.B + (long long)(n0 + kr + 32 * p) * g.ldb + k0 + kc
                            : g.B + (long long)(k0 + nr) * g.ldb + n0 + nc + 2 * p;
      b[p] = f64x2{pb[0], pb[1]};
    }
  };
  auto out = [&](int i, int j, int r) {
    return g.C + (long long)(m0 + wm + 16 * i + 4 * r + lk) * g.ldc + n0 + wn + 16 * j + lr;
  };
  f64x4 acc[2][2], tot[2][2];
  if (k_begin < k_end) load(k_begin);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r) tot[i][j][r] = ACCUM ? *out(i, j, r) : 0.0;
    }
  for (int k0 = k_begin; k0 < k_end; k0 += kGemmK) {
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      As[kc][kr + 32 * p] = a[p][0];
      As[kc + 1][kr + 32 * p] = a[p][1];
      if (BT) {
        Bs[kc][kr + 32 * p] = b[p][0];
        Bs[kc + 1][kr + 32 * p] = b[p][1];
      } else {
        Bs[nr][nc + 2 * p] = b[p][0];
        Bs[nr][nc + 2 * p + 1] = b[p][1];
      }
    }
    __syncthreads();
    if (k0 + kGemmK < k_end) load(k0 + kGemmK);
#pragma unroll
    for (int kk = 0; kk < kGemmK; kk += 4) {
      double af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = As[kk + lk][wm + 16 * i + lr];
        bf[i] = Bs[kk + lk][wn + 16 * i + lr];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(af[i], bf[j], acc[i][j]);
    }
    if (((k0 + kGemmK - k_begin) & (kNb - 1)) == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) tot[i][j][r] += g.alpha * acc[i][j][r];
          acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) *out(i, j, r) = tot[i][j][r];
}

// C += alpha A B^T (both k-fast) on the tiles with tm >= tn (C's diagonal at
// its origin): the Cholesky updates.  Grid (N / 64, M / 64).
__global__ void __launch_bounds__(256) gemm_lower_kernel(GemmF64 g, int Kc) {
  if (blockIdx.x > blockIdx.y) return;
  gemm_tile_f64<true, true>(g, blockIdx.y * kNb, blockIdx.x * kNb, 0, Kc);
}

// ---------------------------------------------------------------- factor --
// mean of the diagonal with dead entries counted as 1 (fixed order), times damp.
__global__ void __launch_bounds__(1024) gptq_diag_kernel(const double* __restrict__ H, int K, double damp,
                                                         uint8_t* __restrict__ dead, double* __restrict__ aux) {
  __shared__ double red[16];
  double s = 0.0;
  for (int k = threadIdx.x; k < K; k += 1024) {
    const double h = H[(size_t)k * K + k];
    dead[k] = h == 0.0 ? 1 : 0;
    s += h == 0.0 ? 1.0 : h;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w];
    aux[0] = damp * (t / K);
  }
}

// Row i = blockIdx.x of A[i][j] = H[K-1-i][K-1-j], dead diagonal entries 1,
// plus the damping; the lower triangle and the rest of its 64-column blocks.
__global__ void __launch_bounds__(256) gptq_reverse_kernel(const double* __restrict__ H, int K,
                                                           const double* __restrict__ aux, double* __restrict__ A) {
  const int i = blockIdx.x;
  const double add = aux[0];
  const double* h = H + (size_t)(K - 1 - i) * K + (K - 1);
  for (int j = threadIdx.x; j <= (i | (kNb - 1)); j += 256) {
    double v = h[-j];
    if (i == j) v = (v == 0.0 ? 1.0 : v) + add;
    A[(size_t)i * K + j] = v;
  }
}

// In-place Cholesky of the 64 x 64 diagonal block kb (lower triangle), 16
// columns at a time: one wave factors them (lane i holds row i in registers,
// the column's values of later rows by readlane), then all four update the
// columns after them.  (With the whole block in LDS and three barriers a
// column it took 90 us; this takes 16.)
constexpr int kDb = 16;

__global__ void __launch_bounds__(256) chol_diag_kernel(double* __restrict__ A, int K, int kb) {
  __shared__ __attribute__((aligned(16))) double a[kNb][kNb + 2];
  double* blk = A + (size_t)kb * kNb * K + (size_t)kb * kNb;
  const int tid = threadIdx.x, lane = tid & 63;
  for (int idx = tid; idx < kNb * kNb; idx += 256) a[idx >> 6][idx & 63] = blk[(size_t)(idx >> 6) * K + (idx & 63)];
  __syncthreads();
  for (int s = 0; s < kNb; s += kDb) {
    if (tid < 64) {
      double c[kDb];
#pragma unroll
      for (int j = 0; j < kDb; ++j) c[j] = a[lane][s + j];
#pragma unroll
      for (int j = 0; j < kDb; ++j) {
        // d = sqrt(p) and the column over d, from 1 / sqrt(p) by two Newton
        // steps, each result with a last correction
        const double p = readlane_f64(c[j], s + j);
        double r = __builtin_amdgcn_rsq(p);
        r = __fma_rn(0.5 * r, __fma_rn(-p * r, r, 1.0), r);
        r = __fma_rn(0.5 * r, __fma_rn(-p * r, r, 1.0), r);
        double d = p * r;
        d = __fma_rn(__fma_rn(-d, d, p), 0.5 * r, d);
        double x = c[j] * r;
        x = __fma_rn(__fma_rn(-x, d, c[j]), r, x);
        c[j] = lane == s + j ? d : x;
#pragma unroll
        for (int i = j + 1; i < kDb; ++i) c[i] = __fma_rn(-c[j], readlane_f64(c[j], s + i), c[i]);
      }
#pragma unroll
      for (int j = 0; j < kDb; ++j)
        if (lane >= s + j) a[lane][s + j] = c[j];
    }
    __syncthreads();
    // columns after s + 16: four threads a row, every fourth column
    const int row = tid >> 2;
    if (row >= s + kDb) {
      double l[kDb];
#pragma unroll
      for (int k = 0; k < kDb; ++k) l[k] = a[row][s + k];
      for (int c = s + kDb + (tid & 3); c <= row; c += 4) {
        double v = a[row][c];
#pragma unroll
        for (int k = 0; k < kDb; ++k) v = __fma_rn(-l[k], a[c][s + k], v);
        a[row][c] = v;
      }
    }
    __syncthreads();
  }
  for (int idx = tid; idx < kNb * kNb; idx += 256) {
    const int i = idx >> 6, c = idx & 63;
    if (i >= c) blk[(size_t)i * K + c] = a[i][c];
  }
}

// Lane C of each four lanes' value, in all four (DPP quad permutation).
template <int C>
__device__ __forceinline__ double quad_bcast(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x55 * C, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x55 * C, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}

// Panel below block kb: each row x of A[r][kb*64 .. +64] solves x L_kk^T = a.
// 64 rows a workgroup, four lanes a row: lane `sub` holds columns 4 t + sub.
// Quotients from the reciprocal with one correction.
constexpr int kLtStride = kNb / 4 + 2;   // doubles between the lanes' shares of a column of L (banks)

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) chol_panel_kernel(double* __restrict__ A, int K, int kb) {
  __shared__ __attribute__((aligned(16))) double Lt[kNb * 4 * kLtStride];   // [m][j % 4][j / 4]: L_kk[j][m]
  __shared__ double inv[kNb];
  const double* blk = A + (size_t)kb * kNb * K + (size_t)kb * kNb;
  const int lane = threadIdx.x & 63, sub = lane & 3;
  double* a = A + ((size_t)(kb + 1) * kNb + (size_t)blockIdx.x * kNb + (threadIdx.x >> 2)) * K + (size_t)kb * kNb;
  double v[kNb / 4];
#pragma unroll
  for (int t = 0; t < kNb / 4; ++t) v[t] = a[4 * t + sub];
#pragma unroll
  for (int p = 0; p < kNb * kNb / 256; ++p) {
    const int j = (threadIdx.x >> 6) + 4 * p, m = lane;
    const double l = m <= j ? blk[(size_t)j * K + m] : 0.0;
    Lt[(m * 4 + (j & 3)) * kLtStride + (j >> 2)] = l;
    if (m == j) inv[m] = 1.0 / l;
  }
  __syncthreads();
  const double* ls = Lt + sub * kLtStride;
#pragma unroll
  for (int m = 0; m < kNb; ++m) {
    const int c = m & 3, tm = m >> 2;
    const double r = c == 0 ? quad_bcast<0>(v[tm]) : c == 1 ? quad_bcast<1>(v[tm])
                   : c == 2 ? quad_bcast<2>(v[tm]) : quad_bcast<3>(v[tm]);
    const double im = inv[m];
    double x = r * im;
    x = __fma_rn(__fma_rn(-x, Lt[(m * 4 + c) * kLtStride + tm], r), im, x);
    const double u = __fma_rn(-x, ls[m * 4 * kLtStride + tm], v[tm]);   // L's zeros keep the solved columns
    v[tm] = sub == c ? x : u;
#pragma unroll
    for (int t = tm + 1; t < kNb / 4; ++t) v[t] = __fma_rn(-x, ls[m * 4 * kLtStride + t], v[t]);
  }
#pragma unroll
  for (int t = 0; t < kNb / 4; ++t) a[4 * t + sub] = v[t];
}

// Mi[ib][ib] = inverse of the lower 64 x 64 block L_ii (zeros above its
// diagonal), a workgroup per block ib.  16 wavefronts, 4 columns each; lane i
// holds row i.
__global__ void __launch_bounds__(1024) tri_inv_diag_kernel(const double* __restrict__ A, int K,
                                                            double* __restrict__ Mi) {
  const int ib = blockIdx.x;
  __shared__ double Lt[kNb][kNb];      // Lt[m][i] = L_ii[i][m]
  const double* blk = A + (size_t)ib * kNb * K + (size_t)ib * kNb;
  for (int idx = threadIdx.x; idx < kNb * kNb; idx += 1024) {
    const int i = idx >> 6, m = idx & 63;
    Lt[m][i] = i >= m ? blk[(size_t)i * K + m] : 0.0;
  }
  __syncthreads();
  const int l = threadIdx.x & 63, w = (int)(threadIdx.x >> 6);
  double* out = Mi + (size_t)ib * kNb * K + (size_t)ib * kNb;
  for (int t = 0; t < 4; ++t) {
    const int c = 4 * w + t;
    double r = l == c ? 1.0 : 0.0, y = 0.0;
    for (int m = c; m < kNb; ++m) {
      const double ym = readlane_f64(r, m) / Lt[m][m];
      if (l == m) y = ym;
      if (l > m) r -= Lt[m][l] * ym;
    }
    out[(size_t)l * K + c] = l >= c ? y : 0.0;
  }
}

// Row i = blockIdx.x of U[i][j] = Mi[K-1-i][K-1-j] on and above the diagonal, 0 below.
__global__ void __launch_bounds__(256) gptq_unreverse_kernel(const double* __restrict__ Mi, int K,
                                                             double* __restrict__ U) {
  const int i = blockIdx.x;
  const double* m = Mi + (size_t)(K - 1 - i) * K + (K - 1);
  for (int j = threadIdx.x; j < K; j += 256) U[(size_t)i * K + j] = j >= i ? m[-j] : 0.0;
}

// One merge level of the triangular inverse: with L = [[P, 0], [Q, S]] (P of
// h rows, S of the next min(h, what is left)), L^-1 = [[P^-1, 0], [-S^-1 Q P^-1,
// S^-1]].  Node blockIdx.z starts at row 2 h z; STEP 0 forms X = Q P^-1 in the
// scratch (node z at z h^2), STEP 1 the corner -S^-1 X.  Blocks of the inverses
// above their diagonals are not read.
template <int STEP>
__global__ void __launch_bounds__(256) tri_merge_kernel(const double* __restrict__ L, double* __restrict__ Mi,
                                                        double* __restrict__ X, int K, int h) {
  const int off = 2 * h * blockIdx.z;
  const int n2 = (K - off - h) < h ? (K - off - h) : h;
  const int m0 = blockIdx.y * kNb, n0 = blockIdx.x * kNb;
  if (m0 >= n2) return;
  double* x = X + (size_t)blockIdx.z * h * h;
  GemmF64 g;
  if (STEP == 0) {
    g = GemmF64{L + (size_t)(off + h) * K + off, Mi + (size_t)off * K + off, x, K, K, h, 1.0};
    gemm_tile_f64<false, false>(g, m0, n0, n0, h);            // P^-1 is lower triangular
  } else {
    g = GemmF64{Mi + (size_t)(off + h) * K + off + h, x, Mi + (size_t)(off + h) * K + off, K, h, K, -1.0};
    gemm_tile_f64<false, false>(g, m0, n0, 0, m0 + kNb);      // so is S^-1
  }
}

// Workspace of the factor: the reversed matrix and its Cholesky factor (in
// place), the inverse, the merges' products (nodes of h rows: at most
// h (K - h) <= K^2 / 4 values) and one scalar.
size_t gptq_factor_bytes(int K) {
  const size_t n = (size_t)K * K;
  return 2 * n * sizeof(double) + n / 4 * sizeof(double) + 256;
}

// ---------------------------------------------------------------- Hessian --
// H (+)= 2 X^T X: a 64 x 64 tile of the lower triangle per workgroup (and its
// mirror image; the two sums are the same bits), 32 calibration rows at a time
// through LDS as bf16, widened as the MFMAs take them.  (K = 4096, 8192 rows:
// 9.5 ms for every tile with vector fp64, 2.7 ms.)
constexpr int kHsRows = 32;
constexpr int kHsLd = kNb + 8;     // LDS row stride (bf16): 16-byte aligned

template <bool VEC>
__global__ void __launch_bounds__(256) gptq_hessian_kernel(const uint16_t* __restrict__ x, int N, int K,
                                                           double* __restrict__ H, bool accumulate) {
  __shared__ __attribute__((aligned(16))) uint16_t As[kHsRows][kHsLd];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[kHsRows][kHsLd];
  // tile (tm, tn), tn <= tm, of the linear index tm (tm + 1) / 2 + tn
  int tm = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
  while (tm * (tm + 1) / 2 > (int)blockIdx.x) --tm;
  while ((tm + 1) * (tm + 2) / 2 <= (int)blockIdx.x) ++tm;
  const int tn = (int)blockIdx.x - tm * (tm + 1) / 2;
  const int m0 = tm * kNb, n0 = tn * kNb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = 32 * (wave >> 1), wn = 32 * (wave & 1);
  const int lr = lane & 15, lk = lane >> 4;
  const int sr = tid >> 3, sc = 8 * (tid & 7);                // staged row and first of 8 columns
  auto load = [&](int t, int c) -> u32x4 {
    if (t >= N) return u32x4{0u, 0u, 0u, 0u};
    const uint16_t* p = x + (size_t)t * K + c;
    if (VEC) return *reinterpret_cast<const u32x4*>(p);
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
    return v;
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  u32x4 a = load(sr, m0 + sc), b = load(sr, n0 + sc);
  for (int t0 = 0; t0 < N; t0 += kHsRows) {
    __syncthreads();
    *reinterpret_cast<u32x4*>(&As[sr][sc]) = a;
    *reinterpret_cast<u32x4*>(&Bs[sr][sc]) = b;
    __syncthreads();
    if (t0 + kHsRows < N) {
      a = load(t0 + kHsRows + sr, m0 + sc);
      b = load(t0 + kHsRows + sr, n0 + sc);
    }
#pragma unroll
    for (int kk = 0; kk < kHsRows; kk += 4) {
      double af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = (double)bf16_bits_to_float(As[kk + lk][wm + 16 * i + lr]);
        bf[i] = (double)bf16_bits_to_float(Bs[kk + lk][wn + 16 * i + lr]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(af[i], bf[j], acc[i][j]);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const size_t m = m0 + wm + 16 * i + 4 * r + lk, n = n0 + wn + 16 * j + lr;
        const double v = 2.0 * acc[i][j][r];
        H[m * K + n] = accumulate ? H[m * K + n] + v : v;
        if (tm != tn) H[n * K + m] = accumulate ? H[n * K + m] + v : v;
      }
}

hipError_t launch_gptq_hessian(const uint16_t* x, int N, int K, double* H, bool accumulate, hipStream_t st) {
  const int nt = K / kNb;
  const dim3 grid((unsigned)(nt * (nt + 1) / 2));
  timing_begin(st, kSiteGptqHessian);
  if (reinterpret_cast<uintptr_t>(x) % 16 == 0)
    hipLaunchKernelGGL(gptq_hessian_kernel<true>, grid, dim3(256), 0, st, x, N, K, H, accumulate);
  else
    hipLaunchKernelGGL(gptq_hessian_kernel<false>, grid, dim3(256), 0, st, x, N, K, H, accumulate);
  timing_end(st, kSiteGptqHessian);
  return hipGetLastError();
}

// A22 -= P P^T on the lower tiles of rows >= r0 and columns [r0, r0 + cols), P
// the columns [c0, c0 + Kc).
static void chol_update(double* A, int K, int r0, int cols, int c0, int Kc, hipStream_t st) {
  if (cols <= 0) return;
  const double* P = A + (size_t)r0 * K + c0;
  const GemmF64 g{P, P, A + (size_t)r0 * K + r0, K, K, K, -1.0};
  hipLaunchKernelGGL(gemm_lower_kernel, dim3(cols / kNb, (K - r0) / kNb), dim3(256), 0, st, g, Kc);
}

hipError_t launch_gptq_factor(const double* H, int K, double damp, double* U, uint8_t* dead, void* ws,
                              hipStream_t st) {
  double* A = static_cast<double*>(ws);
  double* Mi = A + (size_t)K * K;
  double* X = Mi + (size_t)K * K;
  double* aux = X + (size_t)K * K / 4;
  const int nb = K / kNb;
  timing_begin(st, kSiteGptqFactor);
  hipLaunchKernelGGL(gptq_diag_kernel, dim3(1), dim3(1024), 0, st, H, K, damp, dead, aux);
  hipLaunchKernelGGL(gptq_reverse_kernel, dim3(K), dim3(256), 0, st, H, K, aux, A);
  // panels of 256 columns: each 64-column block updates the rest of its panel,
  // the finished panel the matrix after it
  for (int o = 0; o < K; o += kOb) {
    const int oe = o + kOb < K ? o + kOb : K;
    for (int c = o; c < oe; c += kNb) {
      const int kb = c / kNb;
      hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(256), 0, st, A, K, kb);
      if (kb + 1 < nb) hipLaunchKernelGGL(chol_panel_kernel, dim3(nb - kb - 1), dim3(256), 0, st, A, K, kb);
      chol_update(A, K, c + kNb, oe - c - kNb, c, kNb, st);
    }
    if (oe < K) chol_update(A, K, oe, K - oe, o, oe - o, st);
  }
  hipLaunchKernelGGL(tri_inv_diag_kernel, dim3(nb), dim3(1024), 0, st, A, K, Mi);
  for (int h = kNb; h < K; h *= 2) {
    const dim3 grid(h / kNb, h / kNb, (K - h + 2 * h - 1) / (2 * h));
    hipLaunchKernelGGL(tri_merge_kernel<0>, grid, dim3(256), 0, st, A, Mi, X, K, h);
    hipLaunchKernelGGL(tri_merge_kernel<1>, grid, dim3(256), 0, st, A, Mi, X, K, h);
  }
  hipLaunchKernelGGL(gptq_unreverse_kernel, dim3(K), dim3(256), 0, st, Mi, K, U);
  timing_end(st, kSiteGptqFactor);
  return hipGetLastError();
}

// -------------------------------------------------------------- quantize --
// Workspace: the compensated weights [R][K] (a block's columns hold its errors
// e_k once it is quantized) and the codes.
size_t gptq_quantize_bytes(int R, int K) {
  return (size_t)R * K * sizeof(double) + (((size_t)R * K + 255) / 256) * 256;
}

// A row per workgroup at a time: fp64 weights, dead inputs 0; the row's loss
// starts at 0.  The grid is capped: 2^24 rows of 256 threads are one more than
// a launch holds.
constexpr int kPrepRows = 1 << 20;

__global__ void __launch_bounds__(256) gptq_prep_kernel(const float* __restrict__ W, const uint8_t* __restrict__ dead,
                                                        int R, int K, double* __restrict__ Ww,
                                                        double* __restrict__ loss) {
  for (int r = blockIdx.x; r < R; r += gridDim.x) {
    const size_t o = (size_t)r * K;
    for (int k = threadIdx.x; k < K; k += 256) Ww[o + k] = dead[k] ? 0.0 : (double)W[o + k];
    if (loss && threadIdx.x == 0) loss[r] = 0.0;
  }
}

__device__ __forceinline__ void quad_min_max(float& mn, float& mx) {
  mn = fminf(mn, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mn), 0xb1, 0xf, 0xf, false)));
  mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0xb1, 0xf, 0xf, false)));
  mn = fminf(mn, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mn), 0x4e, 0xf, 0xf, false)));
  mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mx), 0x4e, 0xf, 0xf, false)));
}

// A block of 128 columns [b0, b0 + 128): four lanes a row, 16 rows a wave;
// lane `sub` of a row holds columns b0 + 4 i + sub.  The sequential chain of a
// row (decide column k, divide, compensate) is the same for its four lanes,
// which share the block's compensations out; a wave per row, as before, repeated
// the chain's fp64 arithmetic in 64 lanes (494 us a block of 14336 rows, now
// 62 us).  The values move down one register every four columns, so that the
// loop over columns needs no register indexing.
constexpr int kUbStride = 34;      // doubles between the lanes' shares of a row of U (banks)

template <int B>
struct QuantGroup {
  float t[(1 << B) - 1];           // code thresholds
  double lev[1 << B];              // levels s (j - z)
};

// a / b correctly rounded, y = 1 / b correctly rounded: two corrections of
// a y by the exact remainder (Markstein 1990: the first gives a faithful
// quotient, the second the rounded one).  b finite and not tiny; the fix-up
// puts the quotients of infinities, NaN and zeros in place (the corrections
// would make a NaN of an infinite a).
__device__ __forceinline__ double quotient(double a, double b, double y) {
  double q = a * y;
  q = __fma_rn(__fma_rn(-q, b, a), y, q);
  return __builtin_amdgcn_div_fixup(__fma_rn(__fma_rn(-q, b, a), y, q), b, a);
}

// Columns 4 i .. 4 i + 3 of the block; v[t] is column 4 (i + t) + sub, N of them
// live at most.  ub: this lane's share of U (row k at k * 4 * kUbStride).
template <int B, int G, int N>
__device__ __forceinline__ void quant_step(double (&v)[kQb / 4], int i, int sub, const double* ub, const double* ud,
                                           const double* uinv, QuantGroup<B>& grp, uint32_t* sz_row, double& lsum, double& e,
                                           uint32_t& codes) {
  if (4 * i % G == 0) {
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int t = 0; t < G / 4; ++t) {
      if (t < N) {
        const float f = (float)v[t];
        mn = fminf(mn, f);
        mx = fmaxf(mx, f);
      }
    }
    quad_min_max(mn, mx);
    const uint32_t word = group_sz_word(mn, mx, B);
    code_thresholds<B>(grp.t, word);
    const double gs = (double)half_bits_to_float(word & 0xffffu);
    const double gz = (double)half_bits_to_float(word >> 16);
#pragma unroll
    for (int j = 0; j < (1 << B); ++j) grp.lev[j] = gs * ((double)j - gz);
    if (sub == 0) sz_row[(4 * i / G) * 16] = word;
  }
  codes = 0u;
  auto column = [&](auto cc) {
    constexpr int C = decltype(cc)::value;
    const double* uk = ub + (4 * i + C) * 4 * kUbStride + i;
    const double ukk = ud[(4 * i + C) * 4 * kUbStride + C * kUbStride + i], inv = uinv[4 * i + C];
    double u[N];                   // on its way during the column's chain
#pragma unroll
    for (int t = 0; t < N; ++t) u[t] = uk[t];
    const double wk = quad_bcast<C>(v[0]);
    double lev;
    const uint32_t code = threshold_level<B>((float)wk, grp.t, grp.lev, lev);
    const double err = quotient(wk - lev, ukk, inv);
    lsum += err * err / 2.0;
    codes |= code << (8 * C);
    e = sub == C ? err : e;
    // columns up to k are done: their values are no longer read.  Eight
    // products, then their differences: left to itself the compiler puts every
    // difference right behind its product and waits for it
#pragma unroll
    for (int t0 = 0; t0 < N; t0 += 8) {
      double p[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) p[t] = __dmul_rn(err, u[t0 + t]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (C < 3)
          v[t0 + t] = __dsub_rn(v[t0 + t], p[t]);
        else if (t0 + t > 0)
          v[t0 + t - 1] = __dsub_rn(v[t0 + t], p[t]);
      }
      // these values are made here, and the next column's reads stay behind
      // them (sunk below the four columns' chains, they would wait for it with
      // every operand in a register)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int x = t0 + t - (C < 3 ? 0 : 1);
        if (x >= 0) asm volatile("" : "+v"(v[x]) : : "memory");
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  column(std::integral_constant<int, 0>{});
  column(std::integral_constant<int, 1>{});
  column(std::integral_constant<int, 2>{});
  column(std::integral_constant<int, 3>{});
}

template <int B, int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gptq_block_kernel(double* __restrict__ Ww, const double* __restrict__ U, int R,
                                                         int K, int b0, uint8_t* __restrict__ q,
                                                         uint32_t* __restrict__ sz, double* __restrict__ loss) {
  // U's block: [k][column % 4][column / 4], zero before the diagonal; a step
  // reads up to 7 entries past a row's end (values it drops)
  __shared__ __attribute__((aligned(16))) double Ub[kQb * 4 * kUbStride + 8];
  __shared__ double uinv[kQb];     // 1 / U_kk
#pragma unroll 16
  for (int idx = threadIdx.x; idx < kQb * kQb; idx += 256) {
    const int k = idx >> 7, j = idx & 127;
    Ub[(k * 4 + (j & 3)) * kUbStride + (j >> 2)] = j >= k ? U[(size_t)(b0 + k) * K + b0 + j] : 0.0;
  }
  for (int idx = threadIdx.x; idx < kQb * 4 * (kUbStride - 32); idx += 256)   // the padding
    Ub[(idx / (kUbStride - 32)) * kUbStride + 32 + idx % (kUbStride - 32)] = 0.0;
  if (threadIdx.x < 8) Ub[kQb * 4 * kUbStride + threadIdx.x] = 0.0;
  if (threadIdx.x < kQb) uinv[threadIdx.x] = 1.0 / U[(size_t)(b0 + threadIdx.x) * K + b0 + threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63, sub = lane & 3;
  const int row = blockIdx.x * kQRows + 16 * wave_id() + (lane >> 2);
  if (row >= R) return;            // R is a multiple of 16: whole waves
  double* w = Ww + (size_t)row * K + b0;
  double v[kQb / 4];
#pragma unroll
  for (int i = 0; i < kQb / 4; ++i) v[i] = w[4 * i + sub];
  uint32_t* sz_row = sz + ((size_t)(row / 16) * (K / G) + b0 / G) * 16 + row % 16;
  uint32_t* q4 = reinterpret_cast<uint32_t*>(q + (size_t)row * K + b0);
  const double* ub = Ub + sub * kUbStride;
  QuantGroup<B> grp;
  double lsum = 0.0, e = 0.0;
  uint32_t codes = 0u, keep = 0u;
  auto phase = [&](auto nn, int i0) {
    constexpr int N = decltype(nn)::value;
#pragma unroll 1
    for (int i = i0; i < i0 + 8; ++i) {
      quant_step<B, G, N>(v, i, sub, ub, Ub, uinv, grp, sz_row, lsum, e, codes);
      w[4 * i + sub] = e;
      if ((i & 3) == sub) keep = codes;
      if ((i & 3) == 3) q4[i - 3 + sub] = keep;
    }
  };
  phase(std::integral_constant<int, 32>{}, 0);
  phase(std::integral_constant<int, 24>{}, 8);
  phase(std::integral_constant<int, 16>{}, 16);
  phase(std::integral_constant<int, 8>{}, 24);
  if (sub == 0 && loss) loss[row] += lsum;
}

// C[m][n] -= A(m, k) B(k, n), one k after the other with the product and the
// difference rounded each time (the order and roundings of applying GPTQ's
// per-column updates one column at a time), A(m, k) = A[m * ld + k], B(k, n) =
// B[k * ld + n], C[m * ld + n]; N and Kc multiples of 128, M of 16.  A tile of
// 16 T x 16 T outputs per workgroup, T x T per thread in pairs of rows and
// columns; bound by the two fp64 vector operations per multiply-subtract (at
// R = 14336, K = 4096 they issue in 77 % of the cycles, and the clock is down to
// 2.07 GHz: 11.3 ms with 4 x 4 outputs a thread and a pass over the columns
// after every 128, 9.5 ms).
template <int T>
__global__ void __launch_bounds__(256, 2) gptq_update_kernel(int M, int Kc, const double* __restrict__ A,
                                                             const double* __restrict__ B, double* __restrict__ C,
                                                             long long ld) {
  constexpr int TM = 16 * T, KS = 16, P = T / 2;
  __shared__ __attribute__((aligned(16))) double As[2][KS][TM + 4];
  __shared__ __attribute__((aligned(16))) double Bs[2][KS][TM];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
  const int kr = tid >> 3, kc = 2 * (tid & 7);
  f64x2 a[P], b[P];
  auto load = [&](int k0) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int m = m0 + kr + 32 * p;
      const double* pa = A + (long long)(m < M ? m : M - 1) * ld + k0 + kc;
      a[p] = f64x2{pa[0], pa[1]};
      const double* pb = B + (long long)(k0 + ty) * ld + n0 + 2 * tx + 32 * p;
      b[p] = f64x2{pb[0], pb[1]};
    }
  };
  load(0);
  double acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int m = m0 + 2 * ty + (i & 1) + 32 * (i >> 1);
#pragma unroll
    for (int j = 0; j < T; j += 2) {
      const double* c = C + (long long)(m < M ? m : M - 1) * ld + n0 + 2 * tx + 16 * j;
      acc[i][j] = c[0];
      acc[i][j + 1] = c[1];
    }
  }
  auto store = [&](int buf) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      As[buf][kc][kr + 32 * p] = a[p][0];
      As[buf][kc + 1][kr + 32 * p] = a[p][1];
      *reinterpret_cast<f64x2*>(&Bs[buf][ty][2 * tx + 32 * p]) = b[p];
    }
  };
  store(0);
  __syncthreads();
  for (int k0 = 0, buf = 0; k0 < Kc; k0 += KS, buf ^= 1) {
    const bool more = k0 + KS < Kc;
    if (more) load(k0 + KS);
#pragma unroll 2
    for (int kk = 0; kk < KS; ++kk) {
      f64x2 av[P], bv[P];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        av[p] = *reinterpret_cast<const f64x2*>(&As[buf][kk][2 * ty + 32 * p]);
        bv[p] = *reinterpret_cast<const f64x2*>(&Bs[buf][kk][2 * tx + 32 * p]);
      }
      // a row's products, then its differences: left to itself the compiler
      // puts every difference right behind its product, which it waits for
#pragma unroll
      for (int i = 0; i < T; ++i) {
        double p[T];
#pragma unroll
        for (int j = 0; j < T; ++j) p[j] = __dmul_rn(av[i >> 1][i & 1], bv[j >> 1][j & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = __dsub_rn(acc[i][j], p[j]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) {
      store(buf ^ 1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int m = m0 + 2 * ty + (i & 1) + 32 * (i >> 1);
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < T; j += 2) {
      double* c = C + (long long)m * ld + n0 + 2 * tx + 16 * j;
      c[0] = acc[i][j];
      c[1] = acc[i][j + 1];
    }
  }
}

// Columns [n0, n1) take the updates of the errors of columns [k0, k1).
static void gptq_update(double* Ww, const double* U, int R, int K, int k0, int k1, int n0, int n1, hipStream_t st) {
  if (n0 >= n1) return;
  const double* A = Ww + k0;
  const double* B = U + (size_t)k0 * K + n0;
  double* C = Ww + n0;
  const int big = ((R + 127) / 128) * ((n1 - n0) / 128);
  if (big >= 256)   // 128 x 128 tiles where they fill the CUs, else 64 x 64
    hipLaunchKernelGGL(gptq_update_kernel<8>, dim3((n1 - n0) / 128, (R + 127) / 128), dim3(256), 0, st, R, k1 - k0, A,
                       B, C, (long long)K);
  else
    hipLaunchKernelGGL(gptq_update_kernel<4>, dim3((n1 - n0) / 64, (R + 63) / 64), dim3(256), 0, st, R, k1 - k0, A, B,
                       C, (long long)K);
}

// Codes [R][K] -> the packed words of one matrix (same layout as the pack
// kernel): one thread per (16 x 128 tile, lane), the width a compile-time
// constant so that every code lands at a fixed bit position.
template <int B>
__global__ void __launch_bounds__(256) pack_codes_u8_kernel(const uint8_t* __restrict__ q, int R, int K,
                                                            uint32_t* __restrict__ words) {
  const long long tid = (long long)blockIdx.x * 256 + threadIdx.x;
  if (tid >= (long long)R * K / 32) return;
  const int lane = (int)(tid & 63);
  const long long tile = tid >> 6;
  const int tiles_per_row = K / kTileCols;
  const int trow = (int)(tile / tiles_per_row), tcol = (int)(tile % tiles_per_row);
  const int n = trow * kTileRows + (lane & 15), kq = lane >> 4;
  uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int k0 = tcol * kTileCols + 32 * u + 8 * kq;
    const uint2 v = *reinterpret_cast<const uint2*>(q + (size_t)n * K + k0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t code = ((j < 4 ? v.x : v.y) >> (8 * (j & 3))) & 0xffu;
      place_code(w, code, 4 * u + (j >> 1), j & 1, B);
    }
  }
  uint32_t* dst = words + ((size_t)tile * 64 + lane) * B;
#pragma unroll
  for (int p = 0; p < B; ++p) dst[p] = w[p];
}

template <int B, int G>
static void quantize_blocks(double* Ww, const double* U, int R, int K, uint8_t* q, uint32_t* words, uint32_t* sz,
                            double* loss, hipStream_t st) {
  for (int o = 0; o < K; o += kQo) {
    const int oe = o + kQo < K ? o + kQo : K;
    for (int b0 = o; b0 < oe; b0 += kQb) {
      hipLaunchKernelGGL((gptq_block_kernel<B, G>), dim3((R + kQRows - 1) / kQRows), dim3(256), 0, st, Ww, U, R, K, b0,
                         q, sz, loss);
      gptq_update(Ww, U, R, K, b0, b0 + kQb, b0 + kQb, oe, st);
    }
    gptq_update(Ww, U, R, K, o, oe, oe, K, st);
  }
  hipLaunchKernelGGL(pack_codes_u8_kernel<B>, dim3((unsigned)(((long long)R * K / 32 + 255) / 256)), dim3(256), 0, st,
                     q, R, K, words);
}

hipError_t launch_gptq_quantize(const float* W, const double* U, const uint8_t* dead, int R, int K, int bits, int G,
                                uint32_t* words, uint32_t* sz, double* loss, void* ws, hipStream_t st) {
  double* Ww = static_cast<double*>(ws);
  uint8_t* q = reinterpret_cast<uint8_t*>(Ww + (size_t)R * K);
  timing_begin(st, kSiteGptqQuantize);
  hipLaunchKernelGGL(gptq_prep_kernel, dim3(R < kPrepRows ? R : kPrepRows), dim3(256), 0, st, W, dead, R, K, Ww, loss);
#define MC_QUANT(B)                                                        \
  if (G == 32) quantize_blocks<B, 32>(Ww, U, R, K, q, words, sz, loss, st); \
  else if (G == 64) quantize_blocks<B, 64>(Ww, U, R, K, q, words, sz, loss, st); \
  else quantize_blocks<B, 128>(Ww, U, R, K, q, words, sz, loss, st)
  if (bits == 1) {
    MC_QUANT(1);
  } else if (bits == 2) {
    MC_QUANT(2);
  } else {
    MC_QUANT(3);
  }
#undef MC_QUANT
  timing_end(st, kSiteGptqQuantize);
  return hipGetLastError();
}

}  // namespace mc
