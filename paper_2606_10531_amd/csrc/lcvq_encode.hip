// LC encode: the codes of a dense weight under a map A, b (eq. lc_codebook
// inverted).  Per group g of row r, v = A^-1 (w_g - b) and code_k =
// clip(round(v_k), 0, 3).  For A = s G with G orthogonal (the form eq. init_ab
// gives) the distance ||w_g - A z - b|| = s ||v - z|| separates over the d
// coordinates, so these are the nearest codewords of eq. vq_assign; for other
// maps they are the rounding of A^-1 (w_g - b).
//
// v is evaluated in fp32: A^-1 by Gauss-Jordan elimination with partial
// pivoting (largest |pivot|), the pivot row times the reciprocal of the pivot,
// then row_k = fma(-f, pivot_row, row_k) for every other row k; then
// t_j = w_j - b_j and v_k = sum_j Ainv[k, j] t_j as an fma chain.  The codes
// therefore equal those of the exact v except within that evaluation's
// rounding error of a decision boundary.
// Each block inverts A once: a wave holds one element of A and of the inverse per lane
// and takes rows and columns by shuffles, the same operations on every element as the
// serial elimination, hence the same bits.  (One thread per block, through LDS, had
// kept 4096 blocks waiting for it: 28672 x 8192 bf16 to bytes and packed 200 us, now
// 153, of 150 at the copy rate.)  The rest is one pass: the weight is read once (2 or 4
// bytes per element), the codes written once (1 byte and / or 2 bits per element),
// with about 13 vector instructions per element beside it.
#include <algorithm>

#include "lcvq_prep.hpp"

namespace lcvq {

// Lane D i + j of the calling wave holds element (i, j); lanes past D^2 follow along.
template <int D>
__device__ __forceinline__ float invert_f32(const float *__restrict__ A) {
  const int lane = threadIdx.x & 63, l = lane & (D * D - 1), i = l / D, j = l % D;
  float M = A[l], I = i == j ? 1.0f : 0.0f;
  for (int c = 0; c < D; ++c) {
    int p = c;
    float best = fabsf(__shfl(M, c * D + c, 64));
    for (int r = c + 1; r < D; ++r) {
      const float x = fabsf(__shfl(M, r * D + c, 64));
      if (x > best) {
        best = x;
        p = r;
      }
    }
    const int from = (i == c ? p : i == p ? c : i) * D + j;  // rows c and p exchanged
    M = __shfl(M, from, 64);
    I = __shfl(I, from, 64);
    const float rcp = __fdiv_rn(1.0f, __shfl(M, c * D + c, 64));
    const float f = __shfl(M, i * D + c, 64);
    const float mc = __fmul_rn(__shfl(M, c * D + j, 64), rcp), ic = __fmul_rn(__shfl(I, c * D + j, 64), rcp);
    M = i == c ? mc : fmaf(-f, mc, M);
    I = i == c ? ic : fmaf(-f, ic, I);
  }
  return I;
}

// A thread takes 16 consecutive elements (two groups of 8 or four of 4; groups never
// straddle rows, so the flattened matrix is enough): 16 bytes of byte codes, 4 of packed
// ones.  Grid-stride, the next unit's loads in flight.  codes: m x n bytes (optional);
// packed: m x n/4 bytes in the lcvq_pack2bit layout (optional).
template <int D, typename WT>
__global__ __launch_bounds__(256) void k_encode(const WT *__restrict__ W, int64_t total, const float *__restrict__ A,
                                                const float *__restrict__ b, uint8_t *__restrict__ codes,
                                                uint8_t *__restrict__ packed) {
  constexpr int kL = (int)sizeof(WT);  // 16-byte loads per unit
  __shared__ float Ai[D * D];
  if (threadIdx.x < 64) {
    const float x = invert_f32<D>(A);
    if (threadIdx.x < D * D) Ai[threadIdx.x] = x;
  }
  __syncthreads();
  float inv[D][D], bv[D];  // the same in every lane: scalar registers
#pragma unroll
  for (int k = 0; k < D; ++k) {
    bv[k] = b[k];
#pragma unroll
    for (int j = 0; j < D; ++j)
      inv[k][j] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(Ai[k * D + j])));
  }
  // the D codes of one group, as bytes
  auto group = [&](const float *w, uint32_t *bytes) {
    float t[D], v[D];
#pragma unroll
    for (int j = 0; j < D; ++j) t[j] = __fsub_rn(w[j], bv[j]);
#pragma unroll
    for (int k = 0; k < D; ++k) {
      v[k] = 0.0f;
#pragma unroll
      for (int j = 0; j < D; ++j) v[k] = fmaf(inv[k][j], t[j], v[k]);
    }
#pragma unroll
    for (int h = 0; h < D / 4; ++h) bytes[h] = quant_bytes(v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]);
  };
  const int64_t units = total / 16, stride = (int64_t)gridDim.x * 256;
  const u32x4 *src = reinterpret_cast<const u32x4 *>(W);
  int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  u32x4 cur[kL], nxt[kL];
#pragma unroll
  for (int i = 0; i < kL; ++i) cur[i] = u < units ? src[u * kL + i] : u32x4{0u, 0u, 0u, 0u};
  for (; u < units; u += stride) {
    const int64_t un = u + stride;
#pragma unroll
    for (int i = 0; i < kL; ++i) nxt[i] = un < units ? src[un * kL + i] : u32x4{0u, 0u, 0u, 0u};
    float w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if constexpr (kL == 2) w[e] = (e & 1) ? bf16_hi(cur[e >> 3][(e >> 1) & 3]) : bf16_lo(cur[e >> 3][(e >> 1) & 3]);
      else w[e] = __uint_as_float(cur[e >> 2][e & 3]);
    }
    u32x4 c;
#pragma unroll
    for (int g = 0; g < 16 / D; ++g) {
      uint32_t bytes[D / 4];
      group(w + g * D, bytes);
#pragma unroll
      for (int h = 0; h < D / 4; ++h) c[g * (D / 4) + h] = bytes[h];
    }
    if (codes != nullptr) reinterpret_cast<u32x4 *>(codes)[u] = c;
    if (packed != nullptr)
      reinterpret_cast<uint32_t *>(packed)[u] = bytes_to_2bit(c[0], c[1]) | bytes_to_2bit(c[2], c[3]) << 16;
#pragma unroll
    for (int i = 0; i < kL; ++i) cur[i] = nxt[i];
  }
  // fewer than 16 elements left: whole groups
  const int64_t e0 = units * 16 + (int64_t)threadIdx.x * D;
  if (blockIdx.x == 0 && e0 < total) {
    float w[D];
    uint32_t bytes[D / 4];
#pragma unroll
    for (int e = 0; e < D; ++e) {
      if constexpr (kL == 2) w[e] = bf16_to_f32(W[e0 + e]);
      else w[e] = W[e0 + e];
    }
    group(w, bytes);
#pragma unroll
    for (int h = 0; h < D / 4; ++h) {
      if (codes != nullptr) reinterpret_cast<uint32_t *>(codes + e0)[h] = bytes[h];
      if (packed != nullptr) packed[e0 / 4 + h] = (uint8_t)bytes_to_2bit(bytes[h], 0u);
    }
  }
}

hipError_t launch_encode(const void *W, bool w_bf16, int64_t m, int64_t n, int d, const float *A, const float *b,
                         uint8_t *codes, uint8_t *packed, hipStream_t st) {
  // one round of blocks, eight per compute unit; the loop takes the rest
  const int64_t total = m * n;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(total, 16 * 256), 8 * 256));
  if (d == 8) {
    if (w_bf16) k_encode<8, uint16_t><<<g, 256, 0, st>>>((const uint16_t *)W, total, A, b, codes, packed);
    else k_encode<8, float><<<g, 256, 0, st>>>((const float *)W, total, A, b, codes, packed);
  } else {
    if (w_bf16) k_encode<4, uint16_t><<<g, 256, 0, st>>>((const uint16_t *)W, total, A, b, codes, packed);
    else k_encode<4, float><<<g, 256, 0, st>>>((const float *)W, total, A, b, codes, packed);
  }
  return hipGetLastError();
}

}  // namespace lcvq
