// Streaming (HBM-bound) kernels of the LC-VQ layer:
//   * quantise latents into the matrix-core operand layout (+ 2-bit packing)
//   * the activation transform X' = X blockdiag(A), s = X b~   (def. forward_x)
//   * the training pair's saved state, written by the forward prepass from the
//     same reads (codes in the input-gradient layout, X' transposed for the
//     weight gradient, both straight-through masks)
//   * the backward operands: dY transposed for the weight gradient, per-token
//     sums of dY
//   * stand-alone 2-bit packing and dense decode
#include "lcvq_prep.hpp"

namespace lcvq {

// ---- element loads ---------------------------------------------------------

__device__ __forceinline__ void load8(const uint16_t *p, float v[8]) {
  u32x4 w = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = bf16_lo(w[i]);
    v[2 * i + 1] = bf16_hi(w[i]);
  }
}
__device__ __forceinline__ void load8(const float *p, float v[8]) {
  floatx4 a = *reinterpret_cast<const floatx4 *>(p);
  floatx4 b = *reinterpret_cast<const floatx4 *>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[4 + i] = b[i];
  }
}
__device__ __forceinline__ void load4(const uint16_t *p, float v[4]) {
  u32x2 w = *reinterpret_cast<const u32x2 *>(p);
  v[0] = bf16_lo(w[0]); v[1] = bf16_hi(w[0]); v[2] = bf16_lo(w[1]); v[3] = bf16_hi(w[1]);
}
__device__ __forceinline__ void load4(const float *p, float v[4]) {
  floatx4 a = *reinterpret_cast<const floatx4 *>(p);
  v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
}
template <int D, typename T>
__device__ __forceinline__ void loadD(const T *p, float v[D]) {
  if constexpr (D == 8) load8(p, v); else load4(p, v);
}

__device__ __forceinline__ void store4(uint16_t *p, const float v[4]) {
  u32x2 w;
  w[0] = pack_bf16x2(v[0], v[1]);
  w[1] = pack_bf16x2(v[2], v[3]);
  *reinterpret_cast<u32x2 *>(p) = w;
}
__device__ __forceinline__ void store4(float *p, const float v[4]) {
  floatx4 a = {v[0], v[1], v[2], v[3]};
  *reinterpret_cast<floatx4 *>(p) = a;
}
template <int D, typename T>
__device__ __forceinline__ void storeD(T *p, const float v[D]) {
  store4(p, v);
  if constexpr (D == 8) store4(p + 4, v + 4);
}
// The same with the non-temporal cache policy, for the dense decode outputs:
// a stream written once, far larger than the caches and not read back by the
// kernel (28672 x 8192 -> bf16: packed source 105 -> 89 us, bf16 latents 160 ->
// 154 us).  p is aligned to the group (D elements).
template <int D>
__device__ __forceinline__ void storeD_nt(uint16_t *p, const float v[D]) {
  if constexpr (D == 8) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(p));
  } else {
    u32x2 w;
    w[0] = pack_bf16x2(v[0], v[1]);
    w[1] = pack_bf16x2(v[2], v[3]);
    __builtin_nontemporal_store(w, reinterpret_cast<u32x2 *>(p));
  }
}
template <int D>
__device__ __forceinline__ void storeD_nt(float *p, const float v[D]) {
#pragma unroll
  for (int h = 0; h < D / 4; ++h) {
    const floatx4 a = {v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]};
    __builtin_nontemporal_store(a, reinterpret_cast<floatx4 *>(p + 4 * h));
  }
}

// ---- quantise into the operand layouts --------------------------------------
// One block quantises four 64 x 64 tiles of bf16 Z side by side: tile row by
// (rows r), tile columns 4 bq .. 4 bq + 3 (columns c), one tile per wave.  Elements
// beyond Z are quantised from 0 (their products meet zero operands or are not
// stored).  All loads of the tile are issued before the first is used.  Lane 4 i + p
// takes rows slab_row(i) and slab_row(16 + i) of each 32-row slab at columns 8 p and
// 32 + 8 p: neighbouring lanes read neighbouring memory, a lane's four words are its
// whole 16 bytes of the forward operand, and the four lanes of a quad hold the four
// bytes of each mask word and 64 contiguous bits of the packed row, which they put
// together and store one row block and K half each.  (Before, a
// thread made 32 stores of one word and 25 vector instructions per latent instead of
// 17: the saved-state prepass took 232 us at 28672 x 8192 and 4096 tokens, now 202, the
// copy rate, and 21.1 us at 4096 x 4096 and 256 tokens, now 17.2.)
// What it writes depends on kMode:
//   kQuantFwd   the forward product's operand (M axis r, K axis c; tiles at or
//               past gx skipped), and with `packed` the 2-bit codes;
//   kQuantBwd   the input-gradient product's operand (M axis c, K axis r, rows
//               of KBt 64-wide steps), through the LDS tiles `codes`, and with
//               `maskbits` the straight-through mask of mask_mode;
//   kQuantSave  both, plus both masks (rounded into maskbits, latent into
//               maskbits2): the training pair's saved state, from one read of Z.
// Which tiles quantise block q takes: column block bq (256 columns) of row
// band by (64 rows), of gq column blocks and nq blocks in all.  Blocks are
// dispatched round-robin over the eight XCDs.  The four column blocks of a
// band that cover 1024 consecutive columns write the same 128-byte lines of
// the mask bitmaps and the same 256 bytes of each packed row; with block
// indices 8 apart they share an XCD, so those lines are completed in its L2
// instead of being merged from four (measured: the forward prepass with the
// saved state 35.5 -> 33.0 us at 4096^2).  Row-major order when the grid is
// not whole sets of 32 blocks.
__device__ __forceinline__ void quant_tile_of_block(int q, int gq, int nq, int &bq, int &by) {
  if ((gq & 3) == 0 && (nq & 31) == 0) {
    const int line = (q >> 5) * 8 + (q & 7), g4 = gq >> 2;
    bq = 4 * (line % g4) + ((q >> 3) & 3);
    by = line / g4;
  } else {
    bq = q % gq;
    by = q / gq;
  }
}

typedef uint8_t CodeTile[64][64 + 8];  // rows of 72 bytes keep 8-byte stores aligned
constexpr int kQuantFwd = 0, kQuantBwd = 1, kQuantSave = 2;
template <int kMode>
__device__ __forceinline__ void quant_block(int bq, int by, int gx, const uint16_t *__restrict__ Z, int64_t m,
                                            int64_t n, const Quantizer &qz, uint32_t *__restrict__ frag, int KB,
                                            uint8_t *__restrict__ packed, CodeTile *codes,
                                            uint32_t *__restrict__ frag_t = nullptr, int KBt = 0,
                                            uint64_t *__restrict__ maskbits = nullptr, int64_t nbc = 0,
                                            int mask_mode = 0, uint64_t *__restrict__ maskbits2 = nullptr) {
  constexpr bool kFwd = kMode != kQuantBwd, kTrans = kMode != kQuantFwd;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, p = lane & 3, i16 = lane >> 2;
  const int64_t r0 = (int64_t)by * 64, bx = 4 * bq + wave;  // the wave's tile
  const int row16 = 8 * (i16 >> 2) + (i16 & 3);             // slab_row(i16); + 4 for MFMA row 16 + i16
  u32x4 v[2][2][2];  // [slab][row block][K half]
#pragma unroll
  for (int sl = 0; sl < 2; ++sl)
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int64_t r = r0 + 32 * sl + row16 + 4 * rb, c = bx * 64 + 32 * kk + 8 * p;
        v[sl][rb][kk] = u32x4{0u, 0u, 0u, 0u};
        if (r < m && c < n) v[sl][rb][kk] = *reinterpret_cast<const u32x4 *>(Z + r * n + c);
      }
  // OR over the four lanes of a quad (DPP quad permutes 1, 0, 3, 2 and 2, 3, 0, 1)
  auto quad_or = [](uint32_t x) {
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, true);
    return x | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, true);
  };
  auto pick = [&](const uint32_t (&w)[2][2]) { return p == 0 ? w[0][0] : p == 1 ? w[0][1] : p == 2 ? w[1][0] : w[1][1]; };
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    uint32_t nib[2][2], mr[2][2], ml[2][2], plo[2][2], phi[2][2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int rr = 32 * sl + row16 + 4 * rb;
        const int64_t r = r0 + rr, c = bx * 64 + 32 * kk + 8 * p;
        const bool in = r < m && c < n;  // n is a multiple of 8: the eight columns are in or out together
        float z[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z[2 * e] = code_value(bf16_lo(v[sl][rb][kk][e]), qz);
          z[2 * e + 1] = code_value(bf16_hi(v[sl][rb][kk][e]), qz);
        }
        const uint32_t lo = quant_bytes(z[0], z[1], z[2], z[3]), hi = quant_bytes(z[4], z[5], z[6], z[7]);
        nib[rb][kk] = bytes_to_nibbles(lo, hi);
        if constexpr (kTrans) {
          // tile column pos holds M column slab_row(pos) of its 32-column slab:
          // columns 8a + 4b + e sit at 16 b + 4 a + e, so the eight codes go out as
          // two runs of four
          uint8_t *row = &codes[wave][rr][32 * kk + 4 * p];
          *reinterpret_cast<uint32_t *>(row) = lo;
          *reinterpret_cast<uint32_t *>(row + 16) = hi;
        }
        // masks: byte 4 kk + p of the row's 64-bit word, the quad's four bytes together
        auto mask_word = [&](const MaskRange &range) {
          return quad_or(in ? mask_byte(z, range) << (8 * p) : 0u);
        };
        if constexpr (kMode == kQuantBwd) {
          if (maskbits != nullptr) mr[rb][kk] = mask_word(mask_range(mask_mode));
        } else if constexpr (kMode == kQuantSave) {
          mr[rb][kk] = mask_word(mask_range(0));
          ml[rb][kk] = mask_word(mask_range(1));
        }
        if (kFwd && packed != nullptr) {
          // 2-bit codes: 16 bits per lane, 64 contiguous bits per quad
          const uint32_t b2 = bytes_to_2bit(lo, hi);
          if ((n & 31) == 0) {
            const uint32_t w = b2 << (16 * (p & 1));
            plo[rb][kk] = quad_or(p < 2 ? w : 0u);
            phi[rb][kk] = quad_or(p < 2 ? 0u : w);
          } else if (in) {
            *reinterpret_cast<uint16_t *>(packed + r * (n / 4) + c / 4) = (uint16_t)b2;
          }
        }
      }
    // K = columns: the lane's four words are its 16 bytes of the forward operand
    if (kFwd && bx < gx)
      *reinterpret_cast<u32x4 *>(frag + frag_dword_index(by * 2 + sl, (int)bx, KB, 16 * p + i16, 0)) =
          u32x4{nib[0][0], nib[0][1], nib[1][0], nib[1][1]};
    // lane p of a quad stores the word of row block p / 2, K half p % 2
    const int rr = 32 * sl + row16 + 4 * (p >> 1);
    if (r0 + rr < m) {
      const int64_t at = ((((int64_t)by * nbc + bq) * 64 + rr) * 4 + wave) * 2 + (p & 1);
      if constexpr (kMode == kQuantBwd) {
        if (maskbits != nullptr) reinterpret_cast<uint32_t *>(maskbits)[at] = pick(mr);
      } else if constexpr (kMode == kQuantSave) {
        reinterpret_cast<uint32_t *>(maskbits)[at] = pick(mr);
        reinterpret_cast<uint32_t *>(maskbits2)[at] = pick(ml);
      }
      if (kFwd && packed != nullptr && (n & 31) == 0) {
        const int64_t c = bx * 64 + 32 * (p & 1);
        if (c < n) *reinterpret_cast<u32x2 *>(packed + (r0 + rr) * (n / 4) + c / 4) = u32x2{pick(plo), pick(phi)};
      }
    }
  }
  if constexpr (!kTrans) return;  // the operand words are stored above
  // the transposed operand has KBt 64-row steps (rows padded to 128); the
  // forward's grid may hold further row tiles, which have nothing to store here
  if (by >= KBt) return;
  __syncthreads();
  // K = rows: the eight codes of an operand dword are a column of the tile
  // (rows kloc .. kloc + 7).  The transposing LDS read gathers them: in each
  // 16-lane group, source lane 2 k + h names row k of its eight rows, tile
  // positions 8 h .. 8 h + 7 of the 16-position half (16 mb ..) of the slab, and
  // output lane 8 h + c receives byte c of all eight rows, i.e. MFMA row
  // 16 mb + 8 h + c, whose column the tile holds at that position.  Lane L of
  // group L / 16 reads rows 32 (dw % 2) + 8 (L / 16) + 0..7 for dword dw; a lane
  // stores its four dwords together.
  const int g16 = lane >> 4, j16 = lane & 15;
#pragma unroll
  for (int slab = 0; slab < 2; ++slab) {
    typedef int int2v __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) int2v lds_int2v;
    u32x4 w;
#pragma unroll
    for (int dw = 0; dw < 4; ++dw) {
      const int kloc = 32 * (dw & 1) + 8 * g16 + (j16 >> 1), ploc = 16 * (dw >> 1) + 8 * (j16 & 1);
      const int2v t = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_int2v *)(&codes[wave][kloc][slab * 32 + ploc]));
      w[dw] = bytes_to_nibbles((uint32_t)t[0], (uint32_t)t[1]);
    }
    *reinterpret_cast<u32x4 *>(frag_t + frag_dword_index((int)bx * 2 + slab, by, KBt, lane, 0)) = w;
  }
}

// ---- backward operands of the weight-gradient product ----------------------
// Transposed store of one 64-token x 64-feature sub-tile from the LDS tile
// into the token-K fragment layout of v_mfma_f32_16x16x32_bf16 (zero-padded to
// KBt steps and to whole 256-feature tiles): block (f0 / 32 + fb, bt) holds
// four 1 KiB fragments phi = 2 fh + kk2; in fragment phi lane L holds tokens
// 32 kk2 + 8 (L / 16) + 0..7 of feature sel(16 fh + L % 16), sel = slab_row
// for in-features (M side) and the identity for out-features (N side).
// The column reads use the transposing LDS read: in each 16-lane group, lane
// 4 e + q addresses token e (+ 4 for the second read) and four consecutive
// features F(q) .. F(q) + 3, and output lane 4 q + w receives feature F(q) + w
// of the four tokens.  F places those features where sel puts them.
template <bool kMside>
__device__ __forceinline__ void tile_store_t(int bt, int64_t f0, int KBt, uint16_t *__restrict__ dst,
                                             uint16_t (&tile)[64][64 + 8]) {
  const int tid = threadIdx.x;
  const int L = tid & 63, g = L >> 4, e = (L >> 2) & 3, q = L & 3;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = tid + 256 * i, fb = id >> 8, phi = (id >> 6) & 3, fh = phi >> 1, kk2 = phi & 1;
    const int F = kMside ? 8 * q + 4 * fh : 16 * fh + 4 * q;
    const int t = 32 * kk2 + 8 * g + e;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&tile[t][fb * 32 + F]);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&tile[t + 4][fb * 32 + F]);
    const u32x4 w = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    const int64_t blk = (f0 >> 5) + fb;
    *reinterpret_cast<u32x4 *>(dst + (((blk * KBt + bt) * 4 + phi) * 64 + L) * 8) = w;
  }
}

// ---- activation transform, bf16, straight into the B-operand fragments -----
// Block (bt, kc): tokens 64 bt .. 64 bt + 63 and the 64-wide K steps of chunk
// kc.  Per step the block covers one 64-token x 64-K tile in eight 1 KiB
// B-operand fragments: wave w, pass i takes fragment f = 2 w + i (32-token
// half f / 4 = w / 2, fragment f % 4 = 2 th + kk2 with th = w % 2, kk2 = i), in
// which lane L owns token 64 bt + 16 w + L % 16 at K = 64 kb + 32 i + 8 (L / 16)
// + 0..7 -- one whole group (d = 8) or two (d = 4).  The lane loads those 16
// bytes, forms X' = X A per group in fp32 (rounded to bf16) and stores them as
// its 16-byte slice of the fragment.  Tokens >= N and K >= n give zeros.
// s[t] = sum_c X[t, c] b[c % D]: a lane sums its token's products over the
// chunk in a fixed order, the four lanes of a token (L / 16) are added, and
// lanes L < 16 write chunk kc's part of s for tokens 64 bt + 16 w + L
// (sp[kc * Np + t]).  With xt, the steps' X' tiles also go to LDS and from
// there, transposed, into the weight-gradient operand (the training pair's
// saved state); the last chunk then runs on to KBx steps (features padded to
// 256), whose tiles are zeros.  Steps are taken in pairs (one barrier pair per
// two tiles), with the next pair's loads in flight.
template <int D, bool kSave>
__device__ __forceinline__ void act_block(int64_t bt, int kc, const uint16_t *__restrict__ X, int64_t N, int64_t n,
                                          const float *__restrict__ A, const float *__restrict__ b,
                                          uint16_t *__restrict__ Xp, int KB, int spc, int nkc, int64_t Np,
                                          float *__restrict__ sp, uint16_t *__restrict__ xt, int KBx, int KBt,
                                          uint16_t (*tile)[64][64 + 8]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t rows = N - bt * 64;  // > 0 only for blocks that hold real tokens
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + bt * 64 * n, rows > 0 ? (rows < 64 ? rows : 64) * n * 2 : 0);
  float a[D][D], bb[D];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    bb[j] = b[j];
#pragma unroll
    for (int k = 0; k < D; ++k) a[j][k] = A[j * D + k];
  }
  const int tl = 16 * wave + (lane & 15);  // this lane's token within the block
  const int kb0 = kc * spc;
  // whole pairs of steps: KB, KBx and spc are even
  const int kb1 = kSave && kc == nkc - 1 ? KBx : min(kb0 + spc, KB);
  // the lane's 16 bytes of steps kb, kb + 1 (index 2 s + i: step kb + s, K half i)
  auto load = [&](u32x4 (&xv)[4], int kb) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int64_t k = (int64_t)(kb + s2) * 64 + 32 * i + 8 * (lane >> 4);
        const uint32_t off = (kb + s2 < kb1 && k < n) ? (uint32_t)((tl * n + k) * 2) : kOffNone;
        xv[2 * s2 + i] = __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0);
      }
  };
  float acc_s = 0.0f;
  u32x4 cur[4], nxt[4];
  load(cur, kb0);
  for (int kb = kb0; kb < kb1; kb += 2) {
    load(nxt, kb + 2);  // one pair ahead
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const u32x4 &xv = cur[2 * s2 + i];
        float x[8], y[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[2 * e] = bf16_lo(xv[e]);
          x[2 * e + 1] = bf16_hi(xv[e]);
        }
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
        for (int e = 0; e < 8; ++e) acc_s = fmaf(x[e], bb[e % D], acc_s);
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(y[2 * e], y[2 * e + 1]);
        if (kb + s2 < KB) {
          const int64_t tb32 = bt * 2 + (wave >> 1);
          const int fr = 2 * (wave & 1) + i;
          *reinterpret_cast<u32x4 *>(Xp + (((tb32 * KB + kb + s2) * 4 + fr) * 64 + lane) * 8) = w;
        }
        if constexpr (kSave) *reinterpret_cast<u32x4 *>(&tile[s2][tl][32 * i + 8 * (lane >> 4)]) = w;
      }
    if constexpr (kSave) {
      __syncthreads();
      tile_store_t<true>((int)bt, (int64_t)kb * 64, KBt, xt, tile[0]);
      tile_store_t<true>((int)bt, (int64_t)(kb + 1) * 64, KBt, xt, tile[1]);
      __syncthreads();  // the tiles are rewritten by the next pair
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) cur[i] = nxt[i];
  }
  // over the token's four K groups (lanes L % 16 + 16 g)
  acc_s += __shfl_xor(acc_s, 16, 64);
  acc_s += __shfl_xor(acc_s, 32, 64);
  if (lane < 16) sp[(int64_t)kc * Np + bt * 64 + tl] = acc_s;
}

// ---- forward prepass, bf16: one launch for both operands ---------------------
// Blocks [0, nq): quantise blocks of Z (four 64 x 64 tiles each, block
// (id % gq, id / gq), K = columns), with the 2-bit pack when `packed` is set;
// blocks [nq, nq + nbt * nkc): the activation transform, block (bt, kc) =
// ((id - nq) % nbt, (id - nq) / nbt).  kSave also writes the training pair's
// saved state: the input-gradient operand of the codes (frag_t, KBq steps),
// both straight-through masks, and X' in the weight-gradient operand (xt).
template <int D, bool kSave>
__global__ __launch_bounds__(256) void k_fwd_prep(const uint16_t *__restrict__ Z, int64_t m, int64_t n, Quantizer qz,
                                                   uint32_t *__restrict__ frag, uint8_t *__restrict__ packed, int gq,
                                                   int nq, const uint16_t *__restrict__ X, int64_t N,
                                                   const float *__restrict__ A, const float *__restrict__ b,
                                                   uint16_t *__restrict__ Xp, int KB, int spc, int nkc, int64_t Np,
                                                   float *__restrict__ sp, uint32_t *__restrict__ frag_t, int KBq,
                                                   uint64_t *__restrict__ mask_r, uint64_t *__restrict__ mask_l,
                                                   int64_t nbc, uint16_t *__restrict__ xt, int KBx) {
  // LDS only for the saved state: the quantise blocks' code tiles and the
  // activation blocks' X' tile (one launch holds both kinds of block)
  __shared__ __attribute__((aligned(16))) uint8_t lds[kSave ? 4 * sizeof(CodeTile) : 16];
  static_assert(!kSave || 4 * sizeof(CodeTile) >= 2 * 64 * (64 + 8) * sizeof(uint16_t), "X' tiles fit");
  const int id = blockIdx.x;
  if (id < nq) {
    int bq, by;
    quant_tile_of_block(id, gq, nq, bq, by);
    if constexpr (kSave)
      quant_block<kQuantSave>(bq, by, KB, Z, m, n, qz, frag, KB, packed, reinterpret_cast<CodeTile *>(lds), frag_t,
                              KBq, mask_r, nbc, 0, mask_l);
    else
      quant_block<kQuantFwd>(bq, by, KB, Z, m, n, qz, frag, KB, packed, nullptr);
  } else {
    const int j = id - nq, nbt = (int)(Np / 64);
    act_block<D, kSave>(j % nbt, j / nbt, X, N, n, A, b, Xp, KB, spc, nkc, Np, sp, xt, KBx, (int)(Np / 64),
                        reinterpret_cast<uint16_t (*)[64][64 + 8]>(lds));
  }
}

// ---- stand-alone 2-bit packing ----------------------------------------------
// Thread -> one 32-bit word of 16 consecutive codes of the flattened m x n
// matrix (rows are n/4 bytes, so the flattened layout is the row layout).
template <typename ST, bool kFromU8>
__global__ __launch_bounds__(256) void k_pack2bit(const ST *__restrict__ src, int64_t total,
                                                   uint8_t *__restrict__ packed, Quantizer qz) {
  const int64_t words = total / 16;
  for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < words; w += (int64_t)gridDim.x * 256) {
    uint32_t bits = 0;
    if constexpr (kFromU8) {
      u32x4 q = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint8_t *>(src) + w * 16);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        uint32_t c = (q[i >> 2] >> (8 * (i & 3))) & 0xffu;
        bits |= (c > 3u ? 3u : c) << (2 * i);
      }
    } else {
      float v[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        load8(src + w * 16 + 8 * h, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = code_value(v[i], qz);
        bits |= bytes_to_2bit(quant_bytes(v[0], v[1], v[2], v[3]), quant_bytes(v[4], v[5], v[6], v[7])) << (16 * h);
      }
    }
    *reinterpret_cast<uint32_t *>(packed + w * 4) = bits;
  }
  // tail: fewer than 16 codes left (total % 4 == 0, so whole bytes)
  const int64_t done = words * 16;
  if (blockIdx.x == 0 && (int64_t)threadIdx.x < (total - done) / 4) {
    const int64_t e0 = done + 4 * threadIdx.x;
    uint32_t byte = 0;
    for (int i = 0; i < 4; ++i) {
      uint32_t c;
      if constexpr (kFromU8) {
        c = reinterpret_cast<const uint8_t *>(src)[e0 + i];
        c = c > 3u ? 3u : c;
      } else if constexpr (sizeof(ST) == 2) {
        c = quant_code(code_value(bf16_to_f32(reinterpret_cast<const uint16_t *>(src)[e0 + i]), qz));
      } else {
        c = quant_code(code_value(reinterpret_cast<const float *>(src)[e0 + i], qz));
      }
      byte |= c << (2 * i);
    }
    packed[e0 / 4] = (uint8_t)byte;
  }
}

// ---- stand-alone dense decode (def. forward) from latents -------------------
// Thread -> one group of D latents -> D outputs W_hat[r, g*D + j].  Groups never
// straddle rows (n % D == 0), so the flattened group index is enough.
template <int D, typename ZT, typename OT>
__global__ __launch_bounds__(256) void k_dequant(const ZT *__restrict__ src, int64_t groups,
                                                  const float *__restrict__ A,
                                                  const float *__restrict__ b, OT *__restrict__ W) {
  float a[D][D], bb[D];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    bb[j] = b[j];
#pragma unroll
    for (int k = 0; k < D; ++k) a[j][k] = A[j * D + k];
  }
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < groups; q += (int64_t)gridDim.x * 256) {
    float z[D], c[D], y[D];
    loadD<D>(src + q * D, z);
#pragma unroll
    for (int k = 0; k < D; ++k) c[k] = quant_code_f(z[k]);
#pragma unroll
    for (int j = 0; j < D; ++j) {
      float v = bb[j];
#pragma unroll
      for (int k = 0; k < D; ++k) v = fmaf(a[j][k], c[k], v);
      y[j] = v;
    }
    storeD_nt<D>(W + q * D, y);
  }
}

// ---- dense decode from byte or packed codes ---------------------------------
// The source is read in 1 KiB wave chunks with one 16-byte load per lane
// (coalesced: the wave reads 1 KiB of contiguous memory), staged in the wave's
// own LDS slice, and decoded group by group: lane L takes groups L, L + 64,
// L + 128, ... of the chunk, so each store instruction of the wave writes
// contiguous memory (for bf16 at d = 8, 16 bytes per lane, 1 KiB per
// instruction).  A group is D / 4 packed bytes (kSrc 2, lcvq_pack2bit layout) or
// D bytes (kSrc 1; values above 3 are taken as 3); groups never straddle rows,
// so the flattened m x n layout is enough.  Two chunks per wave are loaded
// before either is decoded.  The map is A, b (device), or with kScalar the
// diagonal map W = fma(scale, code, shift), the fp32 result of A = scale I,
// b = shift bit for bit (the other terms add 0 * code).
//
// Packed codes with a general map (kTable) take the map from two tables the
// block builds in LDS first, one per half-group of four codes (one packed
// byte): lo[i][j] = b[j] + sum_{k<4} A[j, k] c_k(i) and hi[i][j] = sum_{k<4}
// A[j, 4 + k] c_k(i), c_k(i) = (i >> 2k) & 3 (d = 4: lo alone).  A group's
// W_hat row is then lo[byte 0] + hi[byte 1]: four 16-byte LDS reads and D adds
// instead of D^2 fma, which would otherwise make the kernel VALU-bound.  The
// sum is grouped differently from the plain fma chain, so the fp32 result can
// differ from it in the last bits.  Groups past the last whole chunk are
// decoded by block 0 from direct loads.
template <int D, int kSrc, typename OT, bool kScalar>
__global__ __launch_bounds__(256) void k_decode_codes(const uint8_t *__restrict__ src, int64_t chunks,
                                                       int64_t groups, const float *__restrict__ A,
                                                       const float *__restrict__ b, float scale, float shift,
                                                       OT *__restrict__ W) {
  constexpr int kBytes = kSrc == 2 ? D / 4 : D;        // source bytes per group
  constexpr int kGroups = 1024 / kBytes;               // groups per wave chunk
  constexpr bool kTable = kSrc == 2 && !kScalar;
  __shared__ __attribute__((aligned(16))) uint8_t stage[4][2][1024];
  __shared__ __attribute__((aligned(16))) float tab[kTable ? 2 : 1][kTable ? 256 : 1][kTable ? D : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float a[D][D], bb[D];
  if constexpr (!kScalar) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      bb[j] = b[j];
#pragma unroll
      for (int k = 0; k < D; ++k) a[j][k] = A[j * D + k];
    }
  }
  if constexpr (kTable) {  // thread i builds row i of both tables
    const int i = threadIdx.x;
#pragma unroll
    for (int h = 0; h < D / 4; ++h)
#pragma unroll
      for (int j = 0; j < D; ++j) {
        float v = h == 0 ? bb[j] : 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) v = fmaf(a[j][4 * h + k], (float)((i >> (2 * k)) & 3), v);
        tab[h][i][j] = v;
      }
    __syncthreads();
  }
  auto code_at = [&](uint32_t bits, int k) -> float {  // code k of a group's source bits
    uint32_t c;
    if constexpr (kSrc == 2) {
      c = (bits >> (2 * k)) & 3u;
    } else {
      c = (bits >> (8 * (k & 3))) & 0xffu;
      c = c > 3u ? 3u : c;
    }
    return (float)c;
  };
  auto map_store = [&](const float (&c)[D], OT *dst) {
    float y[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      if constexpr (kScalar) {
        y[j] = fmaf(scale, c[j], shift);
      } else {
        float v = bb[j];
#pragma unroll
        for (int k = 0; k < D; ++k) v = fmaf(a[j][k], c[k], v);
        y[j] = v;
      }
    }
    storeD_nt<D>(dst, y);
  };
  auto decode = [&](const uint8_t *st, int64_t ch) {
#pragma unroll
    for (int i = 0; i < kGroups / 64; ++i) {
      const int gl = i * 64 + lane;
      float c[D];
      if constexpr (kTable && kBytes == 1) {  // d = 4: one byte, b folded into the table row
        const floatx4 y4 = *reinterpret_cast<const floatx4 *>(tab[0][st[gl]]);
        const float y[4] = {y4[0], y4[1], y4[2], y4[3]};
        storeD_nt<D>(W + (ch * kGroups + gl) * D, y);
        continue;
      } else if constexpr (kBytes == 1) {
        const uint32_t v = st[gl];
#pragma unroll
        for (int k = 0; k < D; ++k) c[k] = code_at(v, k);
      } else if constexpr (kTable) {  // d = 8: lo of byte 0 plus hi of byte 1
        const uint32_t v = *reinterpret_cast<const uint16_t *>(st + 2 * gl);
        const floatx4 *lo = reinterpret_cast<const floatx4 *>(tab[0][v & 0xffu]);
        const floatx4 *hi = reinterpret_cast<const floatx4 *>(tab[1][v >> 8]);
        const floatx4 y0 = lo[0] + hi[0], y1 = lo[1] + hi[1];
        const float y[8] = {y0[0], y0[1], y0[2], y0[3], y1[0], y1[1], y1[2], y1[3]};
        storeD_nt<D>(W + (ch * kGroups + gl) * D, y);
        continue;
      } else if constexpr (kBytes == 2) {
        const uint32_t v = *reinterpret_cast<const uint16_t *>(st + 2 * gl);
#pragma unroll
        for (int k = 0; k < D; ++k) c[k] = code_at(v, k);
      } else if constexpr (kBytes == 4) {
        const uint32_t v = *reinterpret_cast<const uint32_t *>(st + 4 * gl);
#pragma unroll
        for (int k = 0; k < D; ++k) c[k] = code_at(v, k);
      } else {
        const u32x2 v = *reinterpret_cast<const u32x2 *>(st + 8 * gl);
#pragma unroll
        for (int k = 0; k < D; ++k) c[k] = code_at(v[k >> 2], k);
      }
      map_store(c, W + (ch * kGroups + gl) * D);
    }
  };
  // A wave reads back what its own lanes staged: a wave-scope release / acquire
  // around the wave barrier orders the LDS writes before the reads, and the
  // reads before the next trip's writes.
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const u32x4 *s16 = reinterpret_cast<const u32x4 *>(src);
  uint8_t *st0 = stage[wave][0], *st1 = stage[wave][1];
  const int64_t stride = (int64_t)gridDim.x * 4;
  int64_t ch = (int64_t)blockIdx.x * 4 + wave;
  for (; ch + stride < chunks; ch += 2 * stride) {
    const u32x4 v0 = s16[ch * 64 + lane], v1 = s16[(ch + stride) * 64 + lane];
    wave_sync();
    *reinterpret_cast<u32x4 *>(st0 + 16 * lane) = v0;
    *reinterpret_cast<u32x4 *>(st1 + 16 * lane) = v1;
    wave_sync();
    decode(st0, ch);
    decode(st1, ch + stride);
  }
  if (ch < chunks) {
    const u32x4 v0 = s16[ch * 64 + lane];
    wave_sync();
    *reinterpret_cast<u32x4 *>(st0 + 16 * lane) = v0;
    wave_sync();
    decode(st0, ch);
  }
  if (blockIdx.x != 0) return;
  for (int64_t g = chunks * kGroups + threadIdx.x; g < groups; g += 256) {  // fewer than kGroups
    if constexpr (kTable) {
      const floatx4 *lo = reinterpret_cast<const floatx4 *>(tab[0][src[g * kBytes]]);
      float y[D];
      if constexpr (D == 8) {
        const floatx4 *hi = reinterpret_cast<const floatx4 *>(tab[1][src[g * kBytes + 1]]);
        const floatx4 y0 = lo[0] + hi[0], y1 = lo[1] + hi[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) { y[j] = y0[j]; y[4 + j] = y1[j]; }
      } else {
#pragma unroll
        for (int j = 0; j < D; ++j) y[j] = lo[0][j];
      }
      storeD_nt<D>(W + g * D, y);
      continue;
    }
    float c[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const int64_t e = g * D + k;
      uint32_t code;
      if constexpr (kSrc == 2) {
        code = (src[e >> 2] >> (2 * (e & 3))) & 3u;
      } else {
        code = src[e];
        code = code > 3u ? 3u : code;
      }
      c[k] = (float)code;
    }
    map_store(c, W + g * D);
  }
}

// Loads of up to four 64 x 64 sub-tiles (columns 64 (sf0 + q), q < nsub) of a
// row-major bf16 matrix with F columns, rows t0 .. t0 + 63 (only rows < `rows`
// are read): thread -> rows tid / 8 and tid / 8 + 32, 8 columns at (tid % 8) * 8.
__device__ __forceinline__ void load_subtiles4(u32x4 (&v)[4][2], const uint16_t *__restrict__ src, int64_t F,
                                               int64_t t0, int64_t rows, int sf0, int nsub) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int id = tid + 256 * i, row = id >> 3, ch = id & 7;
      const int64_t t = t0 + row, f = (int64_t)(sf0 + q) * 64 + ch * 8;
      v[q][i] = u32x4{0u, 0u, 0u, 0u};
      if (q < nsub && t < rows && f < F) v[q][i] = *reinterpret_cast<const u32x4 *>(src + t * F + f);
    }
}

// X block (bt, fx4): tokens 64 bt .. + 63, in-features 256 fx4 .. + 255.  Rows
// become X' = X blockdiag(A) (so the product yields dW blockdiag(A) directly)
// and are written transposed into xt.
template <int D>
__device__ __forceinline__ void x_block(int bt, int fx4, const uint16_t *__restrict__ X, int64_t n, int64_t N,
                                        const float (&a)[D][D], int KBt, uint16_t *__restrict__ xt,
                                        uint16_t (&tile)[64][64 + 8]) {
  const int tid = threadIdx.x;
  u32x4 v[4][2];
  load_subtiles4(v, X, n, (int64_t)bt * 64, N, 4 * fx4, 4);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int id = tid + 256 * i;
      float x[8], o[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[2 * e] = bf16_lo(v[q][i][e]);
        x[2 * e + 1] = bf16_hi(v[q][i][e]);
      }
#pragma unroll
      for (int g = 0; g < 8 / D; ++g)
#pragma unroll
        for (int k = 0; k < D; ++k) {
          float y = 0.0f;
#pragma unroll
          for (int j = 0; j < D; ++j) y = fmaf(x[g * D + j], a[j][k], y);
          o[g * D + k] = y;
        }
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(o[2 * e], o[2 * e + 1]);
      *reinterpret_cast<u32x4 *>(&tile[id >> 3][(id & 7) * 8]) = w;
    }
    __syncthreads();
    tile_store_t<true>(bt, (int64_t)(4 * fx4 + q) * 64, KBt, xt, tile);
    __syncthreads();  // the tile is rewritten for the next sub-tile
  }
}

// dY part (bt, p): sub-tiles [sf0, sf1) of 64 out-features for tokens
// 64 bt .. 64 bt + 63, written transposed into dyt (when set) and summed per
// row into rsum[0..1] (rows tid / 8 and tid / 8 + 32, totals in threads with
// tid % 8 == 0).  Sub-tiles are loaded four at a time, the next four while the
// current ones are stored, and go through the two LDS tiles in pairs (one
// barrier pair per two sub-tiles).
__device__ __forceinline__ void dy_part(int bt, int sf0, int sf1, const uint16_t *__restrict__ dY, int64_t m,
                                        int64_t N, int KBt, uint16_t *__restrict__ dyt,
                                        uint16_t (*tile)[64][64 + 8], float (&rsum)[2]) {
  const int tid = threadIdx.x;
  auto process = [&](const u32x4 (&v)[4][2], int base) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (base + q >= sf1) break;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int id = tid + 256 * i;
        float sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += bf16_lo(v[q][i][e]) + bf16_hi(v[q][i][e]);
        // over the row's eight 8-feature chunks (lanes id .. id + 7)
        sum += __shfl_xor(sum, 1, 64);
        sum += __shfl_xor(sum, 2, 64);
        sum += __shfl_xor(sum, 4, 64);
        rsum[i] += sum;
        if (dyt != nullptr) *reinterpret_cast<u32x4 *>(&tile[q & 1][id >> 3][(id & 7) * 8]) = v[q][i];
      }
      if (dyt == nullptr || ((q & 1) == 0 && base + q + 1 < sf1)) continue;  // store pairs of sub-tiles
      __syncthreads();
      if (q & 1) tile_store_t<false>(bt, (int64_t)(base + q - 1) * 64, KBt, dyt, tile[0]);
      tile_store_t<false>(bt, (int64_t)(base + q) * 64, KBt, dyt, tile[q & 1]);
      __syncthreads();  // the tiles are rewritten by the next pair
    }
  };
  // two register buffers, statically indexed: trips of eight sub-tiles
  u32x4 va[4][2], vb[4][2];
  load_subtiles4(va, dY, m, (int64_t)bt * 64, N, sf0, sf1 - sf0);
  for (int base = sf0; base < sf1; base += 8) {
    if (base + 4 < sf1) load_subtiles4(vb, dY, m, (int64_t)bt * 64, N, base + 4, sf1 - base - 4);
    process(va, base);
    if (base + 4 >= sf1) break;
    if (base + 8 < sf1) load_subtiles4(va, dY, m, (int64_t)bt * 64, N, base + 8, sf1 - base - 8);
    process(vb, base + 4);
  }
}

// ---- backward prepass, bf16: one launch for all operands --------------------
// Blocks [0, KBt * nrp): dY parts, block (bt, p) = (id % KBt, id / KBt) covers
// out-feature sub-tiles [p * spf, (p + 1) * spf) and writes its partial row
// sums to rsp[p * Nt + t] (Nt = KBt * 64; no atomics); these are the longest
// blocks and go first.  Then nq quantise blocks into the input-gradient operand
// layout (four tiles each, block (q % gq, q / gq), K = rows of Z), then
// KBt * nfx4 X' blocks of 64 tokens x 256 in-features (block (x % KBt, x / KBt)).
template <int D>
__global__ __launch_bounds__(256) void k_bwd_prep(const uint16_t *__restrict__ Z, int64_t m, int64_t n, Quantizer qz,
                                                   uint32_t *__restrict__ frag, int KBq, int gq, int nq,
                                                   const uint16_t *__restrict__ X, const uint16_t *__restrict__ dY,
                                                   const float *__restrict__ A, int64_t N, int KBt, int nfx4,
                                                   int nfy, int spf, int nrp,
                                                   uint16_t *__restrict__ xt, uint16_t *__restrict__ dyt,
                                                   float *__restrict__ rsp, uint64_t *__restrict__ maskbits,
                                                   int64_t nbc, int mask_mode) {
  // one LDS array: four code tiles (quantise blocks) or two 64 x 64 bf16
  // tiles (dY parts, X' blocks)
  __shared__ __attribute__((aligned(16))) uint8_t lds[4 * sizeof(CodeTile)];
  static_assert(4 * sizeof(CodeTile) >= 2 * 64 * (64 + 8) * sizeof(uint16_t), "bf16 tiles fit");
  CodeTile *codes = reinterpret_cast<CodeTile *>(lds);
  uint16_t (*tile)[64][64 + 8] = reinterpret_cast<uint16_t (*)[64][64 + 8]>(lds);
  const int id = blockIdx.x, tid = threadIdx.x;
  const int ndy = KBt * nrp;
  float rsum[2] = {0.0f, 0.0f};
  if (id < ndy) {
    const int bt = id % KBt, p = id / KBt;
    dy_part(bt, p * spf, min((p + 1) * spf, nfy), dY, m, N, KBt, dyt, tile, rsum);
    if ((tid & 7) == 0) {
      const int64_t Nt = (int64_t)KBt * 64, t = (int64_t)bt * 64 + (tid >> 3);
      rsp[(int64_t)p * Nt + t] = rsum[0];
      rsp[(int64_t)p * Nt + t + 32] = rsum[1];
    }
    return;
  }
  const int q = id - ndy;
  if (q < nq) {
    int bq, by;
    quant_tile_of_block(q, gq, nq, bq, by);
    quant_block<kQuantBwd>(bq, by, 4 * gq, Z, m, n, qz, nullptr, 0, nullptr, codes, frag, KBq, maskbits, nbc,
                           mask_mode);
    return;
  }
  const int x = q - nq;
  float a[D][D];
#pragma unroll
  for (int jj = 0; jj < D; ++jj)
#pragma unroll
    for (int k = 0; k < D; ++k) a[jj][k] = A[jj * D + k];
  x_block<D>(x % KBt, x / KBt, X, n, N, a, KBt, xt, tile[0]);
}

// ---- launchers -------------------------------------------------------------

static inline int grid_for(int64_t items, int64_t per_block) {
  int64_t g = ceil_div(items, per_block);
  if (g > 65536) g = 65536;
  return (int)(g < 1 ? 1 : g);
}

hipError_t launch_fwd_prep_bf16(const uint16_t *Z, int64_t m, int64_t n, const Quantizer &qz, uint32_t *frag,
                                uint8_t *packed,
                                const uint16_t *X, int64_t N, int64_t Np, int64_t ldp, int d, const float *A,
                                const float *b, uint16_t *Xp, float *sp, const FwdSave *save, hipStream_t st) {
  const int KB = (int)(ldp / 64);
  // quantise blocks: K = columns (ldp / 64 tiles, four per block), M = rows padded to 256
  const int gq = (KB + 3) / 4, nq = gq * (int)(round_up(m, 256) / 64);
  const int nbt = (int)(Np / 64), nkc = act_chunks(ldp), spc = act_steps_per_chunk(ldp);
  const unsigned grid = (unsigned)(nq + nbt * nkc);
  if (save != nullptr) {
    const int KBq = (int)(round_up(m, 128) / 64), KBx = (int)(round_up(n, 256) / 64);
    const int64_t nbc = mask_col_blocks(n);
    if (d == 8)
      k_fwd_prep<8, true><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, packed, gq, nq, X, N, A, b, Xp, KB, spc, nkc, Np, sp,
                                                save->frag_t, KBq, save->mask_r, save->mask_l, nbc, save->xt, KBx);
    else
      k_fwd_prep<4, true><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, packed, gq, nq, X, N, A, b, Xp, KB, spc, nkc, Np, sp,
                                                save->frag_t, KBq, save->mask_r, save->mask_l, nbc, save->xt, KBx);
  } else {
    if (d == 8)
      k_fwd_prep<8, false><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, packed, gq, nq, X, N, A, b, Xp, KB, spc, nkc, Np, sp,
                                                 nullptr, 0, nullptr, nullptr, 0, nullptr, 0);
    else
      k_fwd_prep<4, false><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, packed, gq, nq, X, N, A, b, Xp, KB, spc, nkc, Np, sp,
                                                 nullptr, 0, nullptr, nullptr, 0, nullptr, 0);
  }
  return hipGetLastError();
}

hipError_t launch_pack2bit(const void *src, int kind, bool bf16, int64_t m, int64_t n, uint8_t *packed,
                           const Quantizer &qz, hipStream_t st) {
  const int64_t total = m * n;
  const int grid = grid_for(total / 16, 256);
  if (kind == 1) k_pack2bit<uint8_t, true><<<grid, 256, 0, st>>>((const uint8_t *)src, total, packed, qz);
  else if (bf16) k_pack2bit<uint16_t, false><<<grid, 256, 0, st>>>((const uint16_t *)src, total, packed, qz);
  else k_pack2bit<float, false><<<grid, 256, 0, st>>>((const float *)src, total, packed, qz);
  return hipGetLastError();
}

template <int D, typename OT, bool kScalar>
static void decode_codes_dispatch(int kind, const void *src, int64_t total, const float *A, const float *b,
                                  float scale, float shift, void *W, hipStream_t st) {
  const int64_t per = kind == 2 ? 4096 : 1024;  // codes per 1 KiB wave chunk
  const int64_t chunks = total / per, groups = total / D;
  int grid = grid_for(chunks, 8);   // four waves per block, two chunks per wave
  // packed codes with a general map build a 16 KiB table per block: at most six
  // blocks per CU (LDS), each wave taking several chunks
  if (kind == 2 && !kScalar && grid > 6 * 256) grid = 6 * 256;
  if (kind == 2)
    k_decode_codes<D, 2, OT, kScalar><<<grid, 256, 0, st>>>((const uint8_t *)src, chunks, groups, A, b, scale, shift,
                                                            (OT *)W);
  else
    k_decode_codes<D, 1, OT, kScalar><<<grid, 256, 0, st>>>((const uint8_t *)src, chunks, groups, A, b, scale, shift,
                                                            (OT *)W);
}

template <int D, typename OT>
static void dequant_dispatch(int kind, bool zbf16, const void *src, int64_t m, int64_t n, const float *A,
                             const float *b, void *W, hipStream_t st) {
  if (kind != 0) {
    decode_codes_dispatch<D, OT, false>(kind, src, m * n, A, b, 1.0f, 0.0f, W, st);
    return;
  }
  const int64_t groups = m * n / D;
  const int grid = grid_for(groups, 256);
  if (zbf16) k_dequant<D, uint16_t, OT><<<grid, 256, 0, st>>>((const uint16_t *)src, groups, A, b, (OT *)W);
  else k_dequant<D, float, OT><<<grid, 256, 0, st>>>((const float *)src, groups, A, b, (OT *)W);
}

hipError_t launch_dequant(const void *src, int kind, bool z_bf16, int64_t m, int64_t n, int d,
                          const float *A, const float *b, void *W, bool out_bf16, hipStream_t st) {
  if (d == 8) {
    if (out_bf16) dequant_dispatch<8, uint16_t>(kind, z_bf16, src, m, n, A, b, W, st);
    else dequant_dispatch<8, float>(kind, z_bf16, src, m, n, A, b, W, st);
  } else {
    if (out_bf16) dequant_dispatch<4, uint16_t>(kind, z_bf16, src, m, n, A, b, W, st);
    else dequant_dispatch<4, float>(kind, z_bf16, src, m, n, A, b, W, st);
  }
  return hipGetLastError();
}

hipError_t launch_decode_scalar(const void *src, int kind, int64_t total, float scale, float shift, void *W,
                                bool out_bf16, hipStream_t st) {
  if (total % 8 == 0) {
    if (out_bf16) decode_codes_dispatch<8, uint16_t, true>(kind, src, total, nullptr, nullptr, scale, shift, W, st);
    else decode_codes_dispatch<8, float, true>(kind, src, total, nullptr, nullptr, scale, shift, W, st);
  } else {
    if (out_bf16) decode_codes_dispatch<4, uint16_t, true>(kind, src, total, nullptr, nullptr, scale, shift, W, st);
    else decode_codes_dispatch<4, float, true>(kind, src, total, nullptr, nullptr, scale, shift, W, st);
  }
  return hipGetLastError();
}

}  // namespace lcvq

namespace lcvq {
hipError_t launch_bwd_prep_bf16(const uint16_t *Z, int64_t m, int64_t n, const Quantizer &qz, uint32_t *frag,
                                const uint16_t *X,
                                const uint16_t *dY, const float *A, int d, int64_t N, uint16_t *xt,
                                uint16_t *dyt, float *rsp, uint64_t *maskbits, int mask_mode, hipStream_t st) {
  const int64_t nbc = mask_col_blocks(n);
  // codes: M = columns of Z padded to 256 (four 64-column tiles per block), K = rows
  // padded to 128 (skipped when frag == nullptr)
  const int gq = (int)(round_up(n, 256) / 256), KBq = (int)(round_up(m, 128) / 64);
  const int nq = frag != nullptr ? gq * KBq : 0;
  // X' blocks (only when xt is wanted) and dY parts (always: they give the row
  // sums; the transposed copy is written only where dyt is set)
  const int KBt = (int)(bwd_tokens(N) / 64);
  const int nfx4 = xt != nullptr ? (int)(round_up(n, 256) / 256) : 0;
  const int nfy = (int)(round_up(m, 256) / 64), spf = rowsum_subtiles_per_part(m), nrp = rowsum_parts(m);
  const unsigned grid = (unsigned)(nq + KBt * (nfx4 + nrp));
  if (d == 8)
    k_bwd_prep<8><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, KBq, gq, nq, X, dY, A, N, KBt, nfx4, nfy, spf, nrp,
                                        xt, dyt, rsp, maskbits, nbc, mask_mode);
  else
    k_bwd_prep<4><<<grid, 256, 0, st>>>(Z, m, n, qz, frag, KBq, gq, nq, X, dY, A, N, KBt, nfx4, nfy, spf, nrp,
                                        xt, dyt, rsp, maskbits, nbc, mask_mode);
  return hipGetLastError();
}
}  // namespace lcvq
