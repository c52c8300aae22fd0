// pack.hip -- the quantize + pack kernel and the dequant/code export kernels.
//
// Quantizer (paper Sec. 3.1: uniform asymmetric, group-wise, values mapped onto
// the integer grid 0..2^b-1; widths 1/2/3 from the PMQ allocation of Eq. 4).
// Per group of G inputs of one row, L = 2^b - 1:
//   s = fp16(fp32(max - min) / L) (1.0 if it rounds to zero), z = fp16(-min / s),
//   code = nearest level s*(j - z), ties to the even j, decided exactly in fp64.
// Sign binarization (appendix A.2, Eq. 7-9; 1-bit experts that ask for it):
// code = 1 where w >= 0, else 0, and every group of the matrix gets
// s = fp16(2 * ||W||_1 / (rows * cols)), z = 1/2, so that s*(code - z) =
// +-||W||_1 / (rows * cols) -- the binarized weight times its scale, in the same
// packed format (the kernels' product is then Eq. 10's add/subtract form).
#include "mc_internal.hpp"

namespace mc {

// ------------------------------------------------------- scale/zero + codes --
// One pass over the weights (HBM-bound: 4 bytes in per weight, about b/8 + 4/G
// out).  A wave takes one packed tile (16 rows x 128 columns): lane l holds the
// 32 weights of row l % 16 whose codes go into its own b words, so the groups'
// minima and maxima need two cross-lane steps (the four lanes of a row) and the
// weights are read once.  The 1.41 G weights of a Mixtral layer (2.5 bits, G =
// 128) take 1.17 ms, 5.2 TB/s of reads and writes; two passes, one for the
// scale/zero words and one for the codes, with every midpoint compared in fp64,
// took 4.94 ms.

// The minimum and maximum over the four lanes of a row (l % 16 equal).
__device__ __forceinline__ void row_min_max(float& mn, float& mx) {
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
    mn = fminf(mn, __shfl_xor(mn, off));
    mx = fmaxf(mx, __shfl_xor(mx, off));
  }
}

// Tile `tile` of one matrix at width B: GPC groups per 128 columns.
template <int B, int GPC>
__device__ __forceinline__ void pack_tile(const float4 (&v)[8], bool sign, int lane, uint32_t* __restrict__ words,
                                          uint32_t* __restrict__ sz) {
  constexpr int UPG = 4 / GPC;                         // 32-column steps of a group
  uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
  for (int g = 0; g < GPC; ++g) {
    float t[(1 << B) - 1];
    if (sign) {
      t[0] = fp32_below(0.0f);                         // w >= 0
    } else {
      float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
      for (int i = 2 * UPG * g; i < 2 * UPG * (g + 1); ++i) {
        mn = fminf(mn, fminf(fminf(v[i].x, v[i].y), fminf(v[i].z, v[i].w)));
        mx = fmaxf(mx, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
      }
      row_min_max(mn, mx);
      const uint32_t szw = group_sz_word(mn, mx, B);
      if (lane >> 4 == g) sz[16 * g + (lane & 15)] = szw;
      code_thresholds<B>(t, szw);
    }
#pragma unroll
    for (int u = UPG * g; u < UPG * (g + 1); ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float4& q = v[2 * u + (j >> 2)];
        const float x = (j & 3) == 0 ? q.x : (j & 3) == 1 ? q.y : (j & 3) == 2 ? q.z : q.w;
        place_code(w, threshold_code<B>(x, t), 4 * u + (j >> 1), j & 1, B);
      }
  }
#pragma unroll
  for (int p = 0; p < B; ++p) words[(size_t)lane * B + p] = w[p];
}

constexpr int kPackWaves = 4;

// grid (tiles of a matrix / kPackWaves, 3E matrices); d and ffn are multiples
// of 128, so a matrix has a multiple of 8 tiles.
template <int GPC>
__global__ void __launch_bounds__(64 * kPackWaves) pack_kernel(const float* __restrict__ wg,
                                                               const float* __restrict__ wu,
                                                               const float* __restrict__ wd, LayerArgs L,
                                                               uint32_t* __restrict__ words_out,
                                                               uint32_t* __restrict__ sz_out) {
  const int lane = threadIdx.x & 63;
  const uint32_t tile = blockIdx.x * kPackWaves + wave_id();
  const int e = blockIdx.y / 3, m = blockIdx.y % 3;
  const int K = (m < 2) ? L.d : L.ffn;
  const uint32_t per_row = (uint32_t)K / kTileCols;
  const uint32_t trow = tile / per_row, tcol = tile - trow * per_row;
  const float* W = (m == 0) ? wg : (m == 1) ? wu : wd;
  const float* src = W + (size_t)e * L.d * L.ffn + (size_t)(trow * kTileRows + (lane & 15)) * K + tcol * kTileCols +
                     8 * (lane >> 4);
  float4 v[8];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    v[2 * u] = reinterpret_cast<const float4*>(src + 32 * u)[0];
    v[2 * u + 1] = reinterpret_cast<const float4*>(src + 32 * u)[1];
  }
  const int b = L.cum_bits[e + 1] - L.cum_bits[e];
  const bool sign = expert_is_sign(L, e);
  uint32_t* words = words_out + layer_word_offset(L, e, m) + (size_t)tile * 64 * b;
  uint32_t* sz = sz_out + layer_sz_offset(L, e, m) + (size_t)tile * GPC * 16;   // groups of a row block are consecutive
  if (b == 1)
    pack_tile<1, GPC>(v, sign, lane, words, sz);
  else if (b == 2)
    pack_tile<2, GPC>(v, false, lane, words, sz);
  else
    pack_tile<3, GPC>(v, false, lane, words, sz);
}

// ------------------------------------------------------- sign binarization --
// ||W||_1 of every sign-binarized matrix: kSignParts partial sums in fp64 per
// matrix (each over a contiguous slice, fixed order inside the block), kept
// in the matrix's own scale/zero words (overwritten by the finish kernel).
constexpr int kSignThreads = 256;

__host__ __device__ inline int sign_parts(long long groups_per_matrix) {
  // partials (8 bytes = 2 words each) fit in the matrix's scale/zero words
  const long long cap = groups_per_matrix / 2;
  return (int)(cap < 1 ? 1 : (cap < 1024 ? cap : 1024));
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kSignThreads / 64; ++w) t += red[w];
  return t;
}

// grid (parts, 3E matrices); matrices of other experts exit at once.
__global__ void __launch_bounds__(kSignThreads) sign_l1_kernel(const float* __restrict__ wg,
                                                               const float* __restrict__ wu,
                                                               const float* __restrict__ wd, LayerArgs L,
                                                               uint32_t* __restrict__ sz) {
  __shared__ double red[kSignThreads / 64];
  const int e = blockIdx.y / 3, m = blockIdx.y % 3;
  if (!expert_is_sign(L, e)) return;
  const long long n4 = (long long)L.d * L.ffn / 4;                    // float4 pieces
  const long long gpm = (long long)L.d * L.ffn / L.G;
  const int parts = sign_parts(gpm);
  const int part = blockIdx.x;
  if (part >= parts) return;
  const long long per = (n4 + parts - 1) / parts;
  const long long b0 = part * per, b1 = (b0 + per) < n4 ? (b0 + per) : n4;
  const float* W = ((m == 0) ? wg : (m == 1) ? wu : wd) + (size_t)e * L.d * L.ffn;
  double acc = 0.0;
  for (long long i = b0 + threadIdx.x; i < b1; i += kSignThreads) {
    const float4 v = reinterpret_cast<const float4*>(W)[i];
    acc += (double)fabsf(v.x) + (double)fabsf(v.y) + (double)fabsf(v.z) + (double)fabsf(v.w);
  }
  const double t = block_sum_f64(acc, red);
  if (threadIdx.x == 0) {             // two 32-bit words (the buffer is only 4-byte aligned)
    const unsigned long long b = __double_as_longlong(t);
    uint32_t* dst = sz + layer_sz_offset(L, e, m) + 2 * (size_t)part;
    dst[0] = (uint32_t)b;
    dst[1] = (uint32_t)(b >> 32);
  }
}

// One workgroup per matrix of a binarized expert: adds the partials in order,
// then writes the scale/zero word of every group.
__global__ void __launch_bounds__(kSignThreads) sign_finish_kernel(LayerArgs L, uint32_t* __restrict__ sz) {
  __shared__ double red[kSignThreads / 64];
  const int e = blockIdx.x / 3, m = blockIdx.x % 3;
  if (!expert_is_sign(L, e)) return;
  const long long gpm = (long long)L.d * L.ffn / L.G;
  const int parts = sign_parts(gpm);
  uint32_t* dst = sz + layer_sz_offset(L, e, m);
  double acc = 0.0;
  const int per = (parts + kSignThreads - 1) / kSignThreads;
  for (int i = threadIdx.x * per; i < (threadIdx.x + 1) * per && i < parts; ++i)
    acc += __longlong_as_double((long long)(((unsigned long long)dst[2 * i + 1] << 32) | dst[2 * i]));
  const double l1 = block_sum_f64(acc, red);             // every partial read before any write
  double s2 = 2.0 * (l1 / ((double)L.d * (double)L.ffn));
  if (s2 > 65504.0) s2 = 65504.0;
  const uint32_t word = (uint32_t)double_to_half_rne(s2) | (0x3800u << 16);   // z = 1/2
  __syncthreads();
  for (long long i = threadIdx.x; i < gpm; i += kSignThreads) dst[i] = word;
}

// ------------------------------------------------------------------ export --
// One thread per tile lane of one matrix: writes its 32 values.
template <int BITS, bool DEQUANT>
__global__ void __launch_bounds__(256) export_kernel(const uint32_t* __restrict__ words,
                                                    const uint32_t* __restrict__ sz, int R, int K,
                                                    int G, void* __restrict__ out) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long lanes = (long long)R * K / 32;
  if (tid >= lanes) return;
  const int lane = (int)(tid & 63);
  const long long tile = tid >> 6;
  const int tiles_per_row = K / kTileCols;
  const int trow = (int)(tile / tiles_per_row), tcol = (int)(tile % tiles_per_row);
  const int n = trow * kTileRows + (lane & 15);
  const int kq = lane >> 4;
  const int ng = K / G;
  uint32_t w[3] = {0u, 0u, 0u};
  const uint32_t* src = words + ((size_t)tile * 64 + lane) * BITS;
  for (int p = 0; p < BITS; ++p) w[p] = src[p];
  for (int u = 0; u < 4; ++u) {
    const int k0 = tcol * kTileCols + 32 * u + 8 * kq;
    const uint32_t szw = sz[((size_t)(n / 16) * ng + k0 / G) * 16 + (n % 16)];
    const double s = (double)half_bits_to_float(szw & 0xffffu);
    const double z = (double)half_bits_to_float(szw >> 16);
    for (int j = 0; j < 8; ++j) {
      const int code = extract_code<BITS>(w, 4 * u + (j >> 1), j & 1);
      const size_t o = (size_t)n * K + k0 + j;
      if constexpr (DEQUANT) {
        // s*(q - z): q - z needs <= 41 bits, the product <= 52: exact in fp64.
        static_cast<uint16_t*>(out)[o] = double_to_half_rne(s * ((double)code - z));
      } else {
        static_cast<uint8_t*>(out)[o] = (uint8_t)code;
      }
    }
  }
}

// ---------------------------------------------------------------- launchers --

hipError_t launch_pack(const float* wg, const float* wu, const float* wd, const LayerArgs& L,
                       uint32_t* words, uint32_t* sz, bool any_sign, hipStream_t stream) {
  if (any_sign) {
    const int parts = sign_parts((long long)L.d * L.ffn / L.G);
    timing_begin(stream, kSitePackSz);
    hipLaunchKernelGGL(sign_l1_kernel, dim3(parts, 3 * L.E), dim3(kSignThreads), 0, stream, wg, wu, wd, L, sz);
    hipLaunchKernelGGL(sign_finish_kernel, dim3(3 * L.E), dim3(kSignThreads), 0, stream, L, sz);
    timing_end(stream, kSitePackSz);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  const dim3 grid((unsigned)((long long)L.d * L.ffn / (kTileRows * kTileCols) / kPackWaves), 3 * L.E);
  const dim3 block(64 * kPackWaves);
  timing_begin(stream, kSitePackCodes);
  if (L.G == 128)
    hipLaunchKernelGGL(pack_kernel<1>, grid, block, 0, stream, wg, wu, wd, L, words, sz);
  else if (L.G == 64)
    hipLaunchKernelGGL(pack_kernel<2>, grid, block, 0, stream, wg, wu, wd, L, words, sz);
  else
    hipLaunchKernelGGL(pack_kernel<4>, grid, block, 0, stream, wg, wu, wd, L, words, sz);
  timing_end(stream, kSitePackCodes);
  return hipGetLastError();
}

hipError_t launch_export(const uint32_t* words, const uint32_t* sz, int bits, int R, int K, int G,
                         bool dequant, void* out, hipStream_t stream) {
  const long long lanes = (long long)R * K / 32;
  const dim3 grid((unsigned)((lanes + 255) / 256)), block(256);
#define MC_EXPORT_CASE(B)                                                                     \
  if (bits == B) {                                                                            \
    if (dequant)                                                                              \
      hipLaunchKernelGGL((export_kernel<B, true>), grid, block, 0, stream, words, sz, R, K, G, \
                         out);                                                                \
    else                                                                                      \
      hipLaunchKernelGGL((export_kernel<B, false>), grid, block, 0, stream, words, sz, R, K,  \
                         G, out);                                                             \
  }
  timing_begin(stream, kSiteExport);
  MC_EXPORT_CASE(1)
  MC_EXPORT_CASE(2)
  MC_EXPORT_CASE(3)
  timing_end(stream, kSiteExport);
#undef MC_EXPORT_CASE
  return hipGetLastError();
}

}  // namespace mc
