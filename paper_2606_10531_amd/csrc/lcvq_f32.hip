// fp32 mode of the LC-VQ layer: the three products of the bf16 path on the fp32
// matrix instruction v_mfma_f32_16x16x4_f32 (fp32 operands and accumulation, an
// fma per term, so the 1e-5 accuracy of this mode holds).
//
//   mode 0 forward : M = r, N = t, K = c   A = code[r,c]   B = X'[t,c], from X while staging
//   mode 3 forward : the same, X' and s ready in memory
//   mode 1 input   : M = c, N = t, K = r   A = code[r,c]   B = dY[t,r]
//   mode 2 weight  : M = c, N = r, K = t   A = X[t,c]      B = dY[t,r]
//
// Block tile 32 (M) x 16 NB (N).  Every 64-wide K chunk goes through LDS (double
// buffered, the next chunk's loads in flight); wave w multiplies K 16 w .. 16 w + 15
// of each chunk over the whole tile, and the four sums are added in LDS at the
// end.  Splitting K instead of the tile keeps a 32-row slab in one wave: with the
// slab_row order lane L ends with eight consecutive M indices 8 (L / 16) .. + 7 of
// column L % 16, i.e. whole groups, and small layers still give many blocks.
//
// The row sums of dY, and for small layers the activation transform (X' = X
// blockdiag(A), s = X b~), are taken while a chunk is staged: every tile repeats
// them for its own tokens, which saves a launch of its own.
// Bound: the matrix core with the chip full (4096^3: input gradient 114, weight
// gradient 120 of the 153 TFLOP/s that a library product reaches), load latency and
// the launches below that.  Vector-unit products before: 500 tokens of 1376 x 1024
// took 166, 247 and 127 us, now 23 each (kernel trace of passes without a pause); 16
// tokens of 256 x 256 32, 33 and 142 (72 LDS atomics per thread for dA), now 6 to 7 each.
// Relative error against 64 bits, 500 tokens of 1376 x 1024, mean of eight inputs, before /
// now in 1e-7: Y 4.9 / 2.5, dX 5.7 / 2.9, dZ 4.0 / 2.1, dA 6.1 / 3.1, db 5.9 / 3.6 (four
// shorter sums instead of one).
#include "lcvq_prep.hpp"

namespace lcvq {

constexpr int64_t kMaxBufLd = (int64_t)1 << 22;  // 64 rows of 2^22 floats: 2^30 bytes
// One dimension of a grid holds fewer than 2^32 threads: tiles past this many go on in
// the grid's next row (2^35 outputs of the forward are that many).
constexpr int kGridRow = 1 << 23;
constexpr int kFM = 32, kFK = 64;   // tile rows, K chunk
constexpr int kLdK = kFK + 4;       // LDS row of a K-contiguous operand: 16-byte reads of 8 rows meet 8 bank groups
constexpr int kLdM = kFM + 4;       // LDS row (one k) of an M-contiguous operand: k rows four apart are 16 banks apart

// MFMA row of weight-side row `r` of a slab (the inverse of slab_row)
__device__ __forceinline__ int slab_pos(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// Four codes as floats.
__device__ __forceinline__ floatx4 codes4(const floatx4 &z, const Quantizer &qz) {
  floatx4 c;
#pragma unroll
  for (int e = 0; e < 4; ++e) c[e] = quant_code_f(code_value(z[e], qz));
  return c;
}

// Four consecutive floats of a row of length `len` from column c, zeros past its
// end (kVec: len and c are multiples of 4, so they are in or out together).
template <bool kVec>
__device__ __forceinline__ floatx4 load_row4(const float *__restrict__ row, int64_t c, int64_t len) {
  floatx4 v = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (kVec) {
    if (c < len) v = *reinterpret_cast<const floatx4 *>(row + c);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < len) v[e] = row[c + e];
  }
  return v;
}
template <bool kVec>
__device__ __forceinline__ void store_row4(float *__restrict__ row, int64_t c, int64_t len, const floatx4 &v) {
  if constexpr (kVec) {
    if (c < len) *reinterpret_cast<floatx4 *>(row + c) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < len) row[c + e] = v[e];
  }
}

// kVec: m is a multiple of 4 (rows of dY and Y can be moved 16 bytes at a time;
// n is a multiple of D, so rows of Z, X, dX and dZ always can).
template <int kMode, int D, int NB, bool kVec, bool kBuf>
__global__ __launch_bounds__(256) void k_f32(const float *__restrict__ Z, Quantizer qz, const float *__restrict__ X,
                                             const float *__restrict__ dY, const float *__restrict__ A,
                                             const float *__restrict__ bvec, int64_t N, int64_t m, int64_t n, int tiles_n,
                                             int mask_mode, GradEst est, int accumulate, float *__restrict__ out,
                                             float *__restrict__ mapp, const float *__restrict__ svec, int tiles) {
  constexpr int kN = 16 * NB, kLdN = kN + 4;
  constexpr bool kFwd = kMode == 0 || kMode == 3;
  constexpr int kASize = kFwd ? kFM * kLdK : kFK * kLdM;
  constexpr int kBSize = kMode == 2 ? kFK * kLdN : kN * kLdK;
  constexpr int kRed = 4 * 2 * NB * 256;  // four waves' tiles
  constexpr int kLds = 2 * (kASize + kBSize) > kRed ? 2 * (kASize + kBSize) : kRed;
  __shared__ __attribute__((aligned(16))) float lds[kLds];
  __shared__ float srow[kN];  // s of the forward, rowsum(dY) of the input gradient
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (the last grid row may have blocks past the last tile: they find no rows to load or
  // store; leaving at once would wait for `tiles` before anything else, 0.2 us a launch)
  const unsigned tile = blockIdx.y * (unsigned)kGridRow + blockIdx.x;
  const int64_t m0 = (int64_t)(tile / (unsigned)tiles_n) * kFM, n0 = (int64_t)(tile % (unsigned)tiles_n) * kN;
  const int64_t K = kFwd ? n : kMode == 1 ? m : N;
  const int64_t Mlen = kFwd ? m : n, Nlen = kMode == 2 ? m : N;

  float a[D][D], bb[D];
  if constexpr (kMode < 2) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      bb[j] = bvec[j];
#pragma unroll
      for (int k = 0; k < D; ++k) a[j][k] = A[j * D + k];
    }
  }

  // ---- staging: K-contiguous rows as eight floats per thread (eight threads per
  // row), M- or N-contiguous ones as four
  floatx4 ra[2][2], rb[2][NB];  // 16-byte pieces of A and B per thread, of two chunks
  float sacc[NB / 2];
#pragma unroll
  for (int i = 0; i < NB / 2; ++i) sacc[i] = 0.0f;
  // Row operands (K-contiguous): thread -> row tid / 8 (+ 32 i), pieces of four at
  // k = kp(0), kp(1): for the transform one run of eight (a whole group), else 32
  // apart, so that eight threads cover 128 bytes.  Column operands: K row tid / kT
  // (+ 256 / kT per piece), four columns from 4 (tid % kT).
  const int r8 = tid >> 3;
  auto kp = [&](bool group, int h) { return group ? (tid & 7) * 8 + 4 * h : (tid & 7) * 4 + 32 * h; };
  // Loads of a chunk: buffer loads from a base that moves with the chunk, so a
  // thread's offsets stay as they are and the ends of the matrix read as zero
  // (kBuf; offsets of a tile below 2^31), or plain loads with every bound checked.
  auto row_piece = [&](const float *src, int64_t r0, int64_t rows, int64_t len, int row, int64_t k0, int k, bool vec) {
    floatx4 v = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (kBuf) {
      const __amdgpu_buffer_rsrc_t rs =
          make_rsrc(src + r0 * len + k0, ((rows - r0 < kN ? rows - r0 : kN) * len - k0) * 4);  // kN >= kFM
      const uint32_t off = (uint32_t)(row * len + k) * 4u;
      const int left = (int)(len - k0 < kFK ? len - k0 : kFK) - k;  // columns of the row from here
      if (vec) {
        v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(left > 0 ? off : kOffNone), 0, 0));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(left > e ? off + 4u * e : kOffNone), 0, 0));
      }
    } else if (r0 + row < rows) {
      v = load_row4<false>(src + (r0 + row) * len, k0 + k, len);
    }
    return v;
  };
  auto col_piece = [&](const float *src, int64_t c0, int64_t len, int64_t k0, int krow, int c, bool vec) {
    floatx4 v = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (kBuf) {
      const int64_t kl = K - k0 < kFK ? K - k0 : kFK;  // <= 0 past the end: nothing is read
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(src + k0 * len + c0, (kl * len - c0) * 4);
      const uint32_t off = (uint32_t)(krow * len + c) * 4u;
      const int left = (int)(len - c0 < kN ? len - c0 : kN) - c;
      if (vec) {
        v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(left > 0 ? off : kOffNone), 0, 0));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(left > e ? off + 4u * e : kOffNone), 0, 0));
      }
    } else if (k0 + krow < K) {
      v = load_row4<false>(src + (k0 + krow) * len, c0 + c, len);
    }
    return v;
  };
  constexpr int kT = kN / 4;  // threads per K row of the weight gradient's dY
  auto load = [&](int u, int64_t ch) {
    const int64_t k0 = ch * kFK;  // chunks past K read as zeros
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (kFwd) ra[u][i] = row_piece(Z, m0, m, n, r8, k0, kp(false, i), true);
      else ra[u][i] = col_piece(kMode == 1 ? Z : X, m0, n, k0, r8 + 32 * i, (tid & 7) * 4, true);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if constexpr (kFwd) rb[u][i] = row_piece(X, n0, N, n, r8 + 32 * (i >> 1), k0, kp(kMode == 0, i & 1), true);
      else if constexpr (kMode == 1) rb[u][i] = row_piece(dY, n0, N, m, r8 + 32 * (i >> 1), k0, kp(false, i & 1), kVec);
      else rb[u][i] = col_piece(dY, n0, m, k0, tid / kT + (256 / kT) * i, (tid % kT) * 4, kVec);
    }
  };
  auto stage = [&](int buf) {
    float *As = lds + buf * (kASize + kBSize), *Bs = As + kASize;
    if constexpr (kFwd) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<floatx4 *>(As + slab_pos(r8) * kLdK + kp(false, h)) = codes4(ra[buf][h], qz);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        *reinterpret_cast<floatx4 *>(As + (r8 + 32 * i) * kLdM + slab_pos((tid & 7) * 4)) =
            kMode == 1 ? codes4(ra[buf][i], qz) : ra[buf][i];
    }
    if constexpr (kMode == 2) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        *reinterpret_cast<floatx4 *>(Bs + (tid / kT + (256 / kT) * i) * kLdN + (tid % kT) * 4) = rb[buf][i];
    } else {
#pragma unroll
      for (int i = 0; i < NB / 2; ++i) {
        float x[8], y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = rb[buf][2 * i + (e >> 2)][e & 3];
        if constexpr (kMode == 0) {
#pragma unroll
          for (int g = 0; g < 8 / D; ++g)
#pragma unroll
            for (int k = 0; k < D; ++k) {
              float v = 0.0f;
#pragma unroll
              for (int j = 0; j < D; ++j) v = fmaf(x[g * D + j], a[j][k], v);
              y[g * D + k] = v;
            }
#pragma unroll
          for (int e = 0; e < 8; ++e) sacc[i] = fmaf(x[e], bb[e % D], sacc[i]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            y[e] = x[e];
            if constexpr (kMode == 1) sacc[i] += x[e];
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          *reinterpret_cast<floatx4 *>(Bs + (r8 + 32 * i) * kLdK + kp(kMode == 0, h)) =
              floatx4{y[4 * h], y[4 * h + 1], y[4 * h + 2], y[4 * h + 3]};
      }
    }
  };

  floatx4 acc[2][NB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  // the wave's 16 K values of the chunk: instruction j takes k = 4 (L / 16) + j of them
  auto compute = [&](int buf) {
    const float *As = lds + buf * (kASize + kBSize), *Bs = As + kASize;
    const int kw = 16 * wave + 4 * q;
    floatx4 av[2], bv[NB];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (kFwd) {
        av[i] = *reinterpret_cast<const floatx4 *>(As + (16 * i + c16) * kLdK + kw);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) av[i][j] = As[(kw + j) * kLdM + 16 * i + c16];
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if constexpr (kMode != 2) {
        bv[i] = *reinterpret_cast<const floatx4 *>(Bs + (16 * i + c16) * kLdK + kw);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[i][j] = Bs[(kw + j) * kLdN + 16 * i + c16];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][j], bv[nb][j], acc[i][nb], 0, 0, 0);
  };

  // loads run two chunks ahead of the staging (a chunk's products are shorter than
  // a load's latency: one chunk ahead, 1376 x 1024 at 500 tokens took 30 us)
  load(0, 0);
  load(1, 1);
  stage(0);
  load(0, 2);
  const int64_t nch = ceil_div(K, kFK);
  for (int64_t ch = 0; ch < nch; ch += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      __syncthreads();
      compute(u);
      stage(u ^ 1);
      load(u ^ 1, ch + u + 3);
    }
  }

  // ---- the four waves' sums, in wave order; wave w finishes column block nb = w
  __syncthreads();
  floatx4 *red = reinterpret_cast<floatx4 *>(lds);  // [wave][nb][rb][lane]
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 2; ++i) red[((wave * NB + nb) * 2 + i) * 64 + lane] = acc[i][nb];
  if constexpr (kMode < 2) {
#pragma unroll
    for (int i = 0; i < NB / 2; ++i) {
      sacc[i] += __shfl_xor(sacc[i], 1, 64);
      sacc[i] += __shfl_xor(sacc[i], 2, 64);
      sacc[i] += __shfl_xor(sacc[i], 4, 64);
      if ((tid & 7) == 0) srow[r8 + 32 * i] = sacc[i];
    }
  }
  __syncthreads();
  // v[0 .. 7]: M indices mb .. mb + 7 of column `col`
  const int64_t mb = m0 + 8 * q, col = n0 + 16 * wave + c16;
  float v[8] = {};
  if (wave < NB) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      floatx4 s = red[(wave * 2 + i) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) s += red[((w * NB + wave) * 2 + i) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = s[e];
    }
  }
  if constexpr (kFwd) {
    if (wave < NB && col < Nlen) {
      const float s = kMode == 0 ? srow[16 * wave + c16] : svec[col];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        store_row4<kVec>(out + col * m, mb + 4 * h, m,
                         floatx4{v[4 * h] + s, v[4 * h + 1] + s, v[4 * h + 2] + s, v[4 * h + 3] + s});
    }
  } else if constexpr (kMode == 1) {
    // dX[t, g*D + j] = sum_k A[j,k] P[t, g*D + k] + rs[t] b[j]
    if (wave < NB && col < Nlen) {
      const float rst = srow[16 * wave + c16];
      float y[8];
#pragma unroll
      for (int g = 0; g < 8 / D; ++g)
#pragma unroll
        for (int j = 0; j < D; ++j) {
          float x = rst * bb[j];
#pragma unroll
          for (int k = 0; k < D; ++k) x = fmaf(a[j][k], v[g * D + k], x);
          y[g * D + j] = x;
        }
#pragma unroll
      for (int h = 0; h < 2; ++h)
        store_row4<true>(out + col * n, mb + 4 * h, n, floatx4{y[4 * h], y[4 * h + 1], y[4 * h + 2], y[4 * h + 3]});
    }
  } else {
    // dW[r, c] = v; dZ = mask * (dW-group A) (times the estimator's slope); dA, db
    // summed over (r, g)
    const bool live = wave < NB && col < Nlen;
    float code[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) code[e] = 0.0f;
    if (live) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (mb + 4 * h >= Mlen) continue;
        const floatx4 zv = load_row4<true>(Z + col * n, mb + 4 * h, n);
        floatx4 o = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (out != nullptr && accumulate) o = load_row4<true>(out + col * n, mb + 4 * h, n);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float z = code_value(zv[e], qz);
          code[4 * h + e] = quant_code_f(z);
          const int g = (4 * h + e) / D, k = (4 * h + e) % D;
          float x = 0.0f;
#pragma unroll
          for (int j = 0; j < D; ++j) x = fmaf(v[g * D + j], A[j * D + k], x);
          const float gz = ste_pass(z, mask_mode) ? (est.dge ? x * dge_slope(z, est) : x) * qz.scale : 0.0f;
          o[e] = accumulate ? o[e] + gz : gz;
        }
        if (out != nullptr) store_row4<true>(out + col * n, mb + 4 * h, n, o);
      }
    }
    if (mapp == nullptr) return;
    // dA[j, k] = sum over (r, g) of dW[r, g D + j] code[r, g D + k], db[j] = sum of
    // dW[r, g D + j]: products with the groups as K.  The wave's 64 x 8 values go
    // through its own LDS rows; operand row i takes component i % D of the groups
    // whose number / 4 is i / D (mod 16 / D), so of each 16 x 16 result the D x D
    // blocks on the diagonal count.
    __syncthreads();  // the sums have been read
    float *gw = lds + wave * 1024, *gc = gw + 512;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      gw[lane * 8 + e] = live ? v[e] : 0.0f;
      gc[lane * 8 + e] = code[e];
    }
    __syncthreads();
    floatx4 da = floatx4{0.0f, 0.0f, 0.0f, 0.0f}, dbv = da;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int at = ((64 / D) * s + 4 * (c16 / D) + q) * D + c16 % D;
      da = __builtin_amdgcn_mfma_f32_16x16x4f32(gw[at], gc[at], da, 0, 0, 0);
      dbv = __builtin_amdgcn_mfma_f32_16x16x4f32(gw[at], 1.0f, dbv, 0, 0, 0);
    }
    constexpr int kSlots = 16 / D;
    float *sum = lds + 4096;  // [wave][slot][D D + D]
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * q + e;
      float *p = sum + (wave * kSlots + i / D) * (D * D + D);
      if (i / D == c16 / D) p[(i % D) * D + c16 % D] = da[e];
      if (c16 == 0) p[D * D + i % D] = dbv[e];
    }
    __syncthreads();
    if (tid < D * D + D && tile < (unsigned)tiles) {
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < 4 * kSlots; ++w) t += sum[w * (D * D + D) + tid];
      mapp[(int64_t)tid * tiles + tile] = t;  // summed over the blocks by launch_map_combine
    }
  }
}

// 64 columns per tile, or 32 where that leaves fewer than two tiles per compute
// unit (the block's time is its K loop, so more and smaller blocks finish sooner).
static bool wide_cols(int64_t rows, int64_t cols) { return ceil_div(rows, kFM) * ceil_div(cols, 64) >= 512; }
int map_rows_f32(int64_t m, int64_t n) {
  return (int)(ceil_div(n, kFM) * ceil_div(m, wide_cols(n, m) ? 64 : 32));
}

// X' (N x n) and s of the forward; one block per token.
template <int D>
__global__ __launch_bounds__(256) void k_f32_act(const float *__restrict__ X, int64_t n, const float *__restrict__ A,
                                                 const float *__restrict__ b, float *__restrict__ Xp,
                                                 float *__restrict__ s) {
  __shared__ float red[4];
  const int tid = threadIdx.x;
  const int64_t t = blockIdx.x;
  float acc = 0.0f;
  for (int64_t g = tid; g < n / D; g += 256) {
    float x[D], y[D];
#pragma unroll
    for (int j = 0; j < D; j += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4 *>(X + t * n + g * D + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[j + e] = v[e];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
      float v = 0.0f;
#pragma unroll
      for (int j = 0; j < D; ++j) v = fmaf(x[j], A[j * D + k], v);
      y[k] = v;
      acc = fmaf(x[k], b[k], acc);
    }
#pragma unroll
    for (int j = 0; j < D; j += 4)
      *reinterpret_cast<floatx4 *>(Xp + t * n + g * D + j) = floatx4{y[j], y[j + 1], y[j + 2], y[j + 3]};
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) s[t] = (red[0] + red[1]) + (red[2] + red[3]);
}

template <int kMode, int D>
static hipError_t launch(const float *Z, const Quantizer &qz, const float *X, const float *dY, const float *A,
                         const float *b, int64_t N, int64_t m, int64_t n, int mask_mode, const GradEst &est,
                         int accumulate, float *out, float *mapp, const float *svec, hipStream_t st) {
  const int64_t rows = kMode == 0 || kMode == 3 ? m : n, cols = kMode == 2 ? m : N;
  const bool wide = wide_cols(rows, cols), vec = m % 4 == 0;
  const int64_t tm = ceil_div(rows, kFM), tn = ceil_div(cols, wide ? 64 : 32);
  auto k = wide ? (vec ? k_f32<kMode, D, 4, true, true> : k_f32<kMode, D, 4, false, true>)
                : (vec ? k_f32<kMode, D, 2, true, true> : k_f32<kMode, D, 2, false, true>);
  // rows so long that a tile's offsets pass 2^31
  if (m >= kMaxBufLd || n >= kMaxBufLd) k = wide ? k_f32<kMode, D, 4, false, false> : k_f32<kMode, D, 2, false, false>;
  const int64_t tiles = tm * tn;
  const dim3 grid((unsigned)(tiles < kGridRow ? tiles : kGridRow), (unsigned)ceil_div(tiles, kGridRow));
  k<<<grid, 256, 0, st>>>(Z, qz, X, dY, A, b, N, m, n, (int)tn, mask_mode, est, accumulate, out, mapp, svec, (int)tiles);
  return hipGetLastError();
}

// Transforming inside the product repeats the transform for every row tile, about 11
// us per 2^30 products N m n beyond the separate form's (64 tokens of 512 x 512 0,
// 500 of 1376 x 1024 9, 2048^3 92); the separate form costs a launch, 3 to 5 us.
bool f32_fused_act(int64_t N, int64_t m, int64_t n) { return (double)N * (double)m * (double)n < (double)(1 << 28); }

hipError_t launch_act_f32(const float *X, const float *A, const float *b, int d, float *Xp, float *s, int64_t N,
                          int64_t n, hipStream_t st) {
  if (d == 8) k_f32_act<8><<<(unsigned)N, 256, 0, st>>>(X, n, A, b, Xp, s);
  else k_f32_act<4><<<(unsigned)N, 256, 0, st>>>(X, n, A, b, Xp, s);
  return hipGetLastError();
}

hipError_t launch_fwd_f32(const float *Z, const Quantizer &qz, const float *X, const float *s, const float *A,
                          const float *b, int d, float *Y, int64_t N, int64_t m, int64_t n, hipStream_t st) {
  auto go = s != nullptr ? launch<3, 8> : d == 8 ? launch<0, 8> : launch<0, 4>;
  return go(Z, qz, X, nullptr, A, b, N, m, n, 0, GradEst{}, 0, Y, nullptr, s, st);
}

hipError_t launch_dx_f32(const float *Z, const Quantizer &qz, const float *dY, const float *A, const float *b, int d,
                         float *dX, int64_t N, int64_t m, int64_t n, hipStream_t st) {
  return (d == 8 ? launch<1, 8> : launch<1, 4>)(Z, qz, nullptr, dY, A, b, N, m, n, 0, GradEst{}, 0, dX, nullptr, nullptr,
                                                st);
}

hipError_t launch_dz_f32(const float *X, const float *dY, const float *Z, const Quantizer &qz, const float *A, int d,
                         int mask_mode, const GradEst &est, int accumulate, float *dZ, float *mapp, int64_t N, int64_t m,
                         int64_t n, hipStream_t st) {
  return (d == 8 ? launch<2, 8> : launch<2, 4>)(Z, qz, X, dY, A, nullptr, N, m, n, mask_mode, est, accumulate, dZ, mapp,
                                                nullptr, st);
}

}  // namespace lcvq
