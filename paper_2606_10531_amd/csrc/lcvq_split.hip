// The codes products (forward, input gradient) for shapes whose wide tiles
// (k_gemm_codes, lcvq_gemm.hip) would leave compute units idle: few tokens, few
// out- or in-features, or a last round of tiles that is nearly empty.
//
// Block tile 32 MI weight-side rows x 64 tokens.  The block's four waves split
// K (wave w takes the 64-wide steps w, w + 4, ..., so together they read 256
// consecutive K of every activation row), each with an accumulator of the whole
// tile, and add their sums through LDS in a fixed order at the end.  A block does
// an eighth (MI = 4) or a sixteenth (MI = 2) of a wide tile's work with the same
// matrix-core instructions per converted codes operand, and two blocks share a
// compute unit, so one's epilogue runs under the other's products.  What bounds
// it: with the chip full, operand traffic (the waves share nothing: 64 tokens x 64
// K of activations and MI KiB of codes per step and wave); with one block per
// compute unit, that traffic's 64 bytes per clock into the unit and its latency.
// Operand layouts, the codes conversion and the epilogues are those of
// k_gemm_codes.
#include "lcvq_mfma.hpp"
#include "lcvq_prep.hpp"

namespace lcvq {

constexpr int kW = 4;  // waves of a block, each on its own part of K

// kMode 0: forward (B = X' fragments), 1: input gradient (B = dY, row length ldB)
template <int kMode, int D, int MI>
__global__ __launch_bounds__(256, 2) void k_codes_split(
    const uint32_t *__restrict__ frag, int KB, const uint16_t *__restrict__ Bsrc, int64_t ldB, int tiles_m,
    int tiles_n, const float *__restrict__ vecT, int vparts, int64_t vstride, const float *__restrict__ A,
    const float *__restrict__ bvec, uint16_t *__restrict__ out, int64_t ldo, int64_t Mvalid, int64_t Tvalid,
    const uint16_t *__restrict__ X, float *__restrict__ mapp) {
  constexpr int P = 2 * MI;  // 16-row blocks of the tile
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of_block(tiles_m, tiles_n, tm, tn);
  const int64_t tw = (int64_t)tn * 64;

  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(frag + (size_t)(tm * MI) * KB * 256, (int64_t)MI * KB * 1024);
  const __amdgpu_buffer_rsrc_t rsB =
      kMode == 0 ? make_rsrc(Bsrc + (tw >> 5) * (int64_t)KB * 2048, (int64_t)2 * KB * 4096)
                 : make_rsrc(Bsrc + tw * ldB, (Tvalid - tw < 64 ? Tvalid - tw : 64) * ldB * 2);
  floatx4 acc[P][4];  // [row block 2 mi + rb][16-token block tb]
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  acc_fence(acc);

  // Codes: two register buffers of one step each (steps past KB load nothing and
  // read as zero).  The conversion of the next operand is placed between the
  // MFMAs of the current one, as in k_gemm_codes.
  u32x4 ca[2][MI];
  auto load_a = [&](int buf, int kb) {
    const bool live = kb < KB;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
      ca[buf][mi] = __builtin_amdgcn_raw_buffer_load_b128(rsA, live ? lane * 16 : (int)kOffNone,
                                                          live ? (mi * KB + kb) * 1024 : 0, 0);
  };
  auto conv = [&](int buf, int s2) {  // operand s2 = P kk2 + 2 mi + rb of a step
    const int kk2 = s2 / P, p = s2 % P;
    return nibbles_to_bf16x8_ordered(ca[buf][p >> 1][2 * (p & 1) + kk2]);
  };
  // the MFMAs of half-step kk2: b[tb] the four token blocks' operands
  auto half = [&](int buf, int kk2, bf16x8 &an, const u32x4 (&b)[4]) {
    if (kk2 == 0) an = conv(buf, 0);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int s2 = P * kk2 + p;
      const bf16x8 a = an;
      if (s2 == 0) mfma16_valu_a(acc[p][0], a, __builtin_bit_cast(bf16x8, b[0]));
      else mfma16(acc[p][0], a, __builtin_bit_cast(bf16x8, b[0]));
      mfma16(acc[p][1], a, __builtin_bit_cast(bf16x8, b[1]));
      if (s2 + 1 < 2 * P) an = conv(buf, s2 + 1);
      mfma16(acc[p][2], a, __builtin_bit_cast(bf16x8, b[2]));
      mfma16(acc[p][3], a, __builtin_bit_cast(bf16x8, b[3]));
    }
  };
  __shared__ __attribute__((aligned(1024))) char lds[kW * 16384];  // dY stages (kMode 1), then the waves' sums

  if constexpr (kMode == 0) {
    // X' fragments: whole 1 KiB per load, straight into registers, two steps ahead
    u32x4 cb[2][2][4];  // [buffer][half-step][token block]
    auto load = [&](int buf, int kb) {
      load_a(buf, kb);
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int kk2 = 0; kk2 < 2; ++kk2)
          cb[buf][kk2][tb] = __builtin_amdgcn_raw_buffer_load_b128(
              rsB, kb < KB ? (int)(((((tb >> 1) * KB + kb) * 4) + 2 * (tb & 1) + kk2) * 1024 + lane * 16) : (int)kOffNone,
              0, 0);
    };
    load(0, wave);
    __builtin_amdgcn_sched_barrier(0);
    load(1, wave + kW);
    __builtin_amdgcn_sched_barrier(0);
    for (int kb = wave; kb < KB; kb += 2 * kW) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 an;
        half(u, 0, an, cb[u][0]);
        half(u, 1, an, cb[u][1]);
        __builtin_amdgcn_sched_barrier(0);
        load(u, kb + (2 + u) * kW);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    // dY rows.  Lanes that follow each other must read memory that follows each
    // other: with the operand's own mapping (neighbouring lanes = tokens, a row
    // apart) a 1 KiB load takes the address path 64 cycles instead of 16
    // (measured 8.5 against 23 TB/s from the L2).  So a direct-to-LDS load brings
    // eight whole 128-byte runs, lane L chunk (L % 8) ^ (L / 8) (16 bytes) of row
    // 8 r + L / 8, into the wave's own LDS stage: row t's chunk k sits at
    // 128 t + 16 (k ^ (t % 8)), which keeps the operand reads free of bank
    // conflicts.  Chunks outside dY arrive as zeros.  Only the wave itself uses its
    // two stages, so no barrier is needed.  (Through registers and LDS writes the
    // same product took 17.4 us instead of 15.7 at 256 tokens of 4096 x 4096, 82
    // instead of 79 at 1000 of 11008 x 4096.)
    u32x4 b0[4], b1[4];
    char *stage = lds + wave * 16384;
    const int lrow = lane >> 3, lch = (lane & 7) ^ lrow;
    const uint32_t goff = (uint32_t)((lrow * ldB + 8 * lch) * 2);
    const uint32_t roff = (uint32_t)(c16 * 128 + ((q ^ (c16 & 7)) << 4));
    const int kb_lim = (int)ldB - 8 - 8 * lch;  // the lane's chunk exists at step kb iff 64 kb <= kb_lim
    const uint32_t gstep = (uint32_t)(16 * ldB);  // eight rows
    auto load_g = [&](int st, int kb) {
      const uint32_t off = kb < KB && kb * 64 <= kb_lim ? goff + (uint32_t)kb * 128u : kOffNone;
#pragma unroll
      for (int r = 0; r < 8; ++r)
        buffer_to_lds16(rsB, (lds_void *)(stage + st * 8192 + r * 1024), off == kOffNone ? kOffNone : off + r * gstep);
    };
    auto get = [&](u32x4 (&b)[4], int st, int kk2) {
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
        b[tb] = *reinterpret_cast<const u32x4 *>(stage + st * 8192 + tb * 2048 + (roff ^ (kk2 << 6)));
    };
    // The wait before a stage is read leaves the codes loads that were issued after
    // it in flight.
    load_a(0, wave);
    load_g(0, wave);
    __builtin_amdgcn_sched_barrier(0);
    load_a(1, wave + kW);
    __builtin_amdgcn_sched_barrier(0);
    for (int kb = wave; kb < KB; kb += 2 * kW) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 an;
        const int k = kb + kW * u;
        LCVQ_WAIT_VM(MI);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        get(b0, u, 0);
        get(b1, u, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_g(u ^ 1, k + kW);
        __builtin_amdgcn_sched_barrier(0);
        half(u, 0, an, b0);
        half(u, 1, an, b1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(u, k + 2 * kW);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    LCVQ_WAIT_ALL();  // the last stage's loads have landed before the sums overwrite it
    __syncthreads();  // the stages become the waves' sums
  }
  mfma_drain();

  // ---------------------------------------------------------------- epilogue
  // After the sum, wave w holds 16-token block tb = w of the tile: lane L the 8
  // consecutive weight-side rows c .. c + 7 (c = 32 (tm MI + mi) + 8 (L / 16)) of
  // token t = tw + 16 w + L % 16, for each slab mi.
  const int tl = 16 * wave + c16;
  const int64_t cb0 = (int64_t)tm * MI * 32 + 8 * q;
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + tw * ldo, out == nullptr ? 0 : (Tvalid - tw) * ldo * 2);
  // per-token term: the token's four lanes split its partial rows (as in k_gemm_codes)
  constexpr int kMaxParts = kMaxActChunks;
  static_assert(kMaxParts % 4 == 0, "whole parts per lane");
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vecT + tw, ((int64_t)(vparts - 1) * vstride + Tvalid - tw) * 4);
  float vp[kMaxParts / 4];
#pragma unroll
  for (int i = 0; i < kMaxParts / 4; ++i) {
    const int p = 4 * i + q;
    vp[i] = p < vparts ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rv, (int)((p * vstride + tl) * 4), 0, 0))
                       : 0.0f;
  }
  const bool want_map = kMode == 1 && mapp != nullptr;
  u32x4 xv[kMode == 1 ? MI : 1];  // X[t, c .. c + 7] per slab
  if constexpr (kMode == 1) {
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + tw * Mvalid, want_map ? (Tvalid - tw) * Mvalid * 2 : 0);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int64_t c = cb0 + i * 32;
      xv[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, c < Mvalid ? (uint32_t)(tl * Mvalid + c) * 2u : kOffNone, 0, 0);
    }
  }
  float vt = vp[0];
#pragma unroll
  for (int i = 1; i < kMaxParts / 4; ++i) vt += vp[i];
  vt += __shfl_xor(vt, 16, 64);
  vt += __shfl_xor(vt, 32, 64);

  // constants of the A^T map and the map-gradient sums (see k_gemm_codes)
  bf16x8 amh[2], aml[2];
  float bsel[2][4], gb[D];
  floatx4 dah = floatx4{0.0f, 0.0f, 0.0f, 0.0f}, dal = dah;
  __shared__ __attribute__((aligned(1024))) char pst[kMode == 1 ? kW * 3072 : 16];
  const int tq = c16 & 3, te = c16 >> 2;
  const int toff = 16 * (16 * (2 * (tq >> 1) + (q >> 1)) + 8 * (q & 1) + te) + 8 * (tq & 1);
  auto tr8 = [&](const char *base) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(base + toff));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(base + toff + 64));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  if constexpr (kMode == 1) {
#pragma unroll
    for (int j = 0; j < D; ++j) gb[j] = 0.0f;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const int cp = slab_row(16 * mb + c16);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = 8 * q + i;
        const float v = cp / D == c / D ? A[(cp % D) * D + (c % D)] : 0.0f;
        const __bf16 h = (__bf16)v;
        amh[mb][i] = h;
        aml[mb][i] = (__bf16)(v - (float)h);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) bsel[mb][e] = to_vgpr(bvec[(4 * mb + e) % D]);
    }
  }

  // The four waves' sums through LDS, two slabs (four row blocks) at a time:
  // every wave stores its four token blocks, then reads the four partial sums of
  // its own and adds them in wave order.
  floatx4 (*red)[4][4][64] = reinterpret_cast<floatx4 (*)[4][4][64]>(lds);  // [source wave][tb][row block][lane]
#pragma unroll
  for (int ph = 0; ph < MI / 2; ++ph) {
    if (ph > 0) __syncthreads();
#pragma unroll
    for (int tb = 0; tb < 4; ++tb)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        floatx4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x;
          asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[4 * ph + k][tb][e]));
          r[e] = x;
        }
        red[wave][tb][k][lane] = r;
      }
    __syncthreads();
    float pv[2][8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      floatx4 v = red[0][wave][k][lane];
#pragma unroll
      for (int w = 1; w < kW; ++w) v += red[w][wave][k][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[k >> 1][4 * (k & 1) + e] = v[e];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 xp = xv[kMode == 1 ? 2 * ph + h : 0];
      const int64_t c = cb0 + (2 * ph + h) * 32;
      const uint32_t off = c < Mvalid ? (uint32_t)(tl * ldo + c) * 2u : kOffNone;
      u32x4 w;
      if constexpr (kMode == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(pv[h][2 * e] + vt, pv[h][2 * e + 1] + vt);
      } else {
        u32x4 ph_, pl_;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ph_[e] = pack_bf16x2(pv[h][2 * e], pv[h][2 * e + 1]);
          pl_[e] = pack_bf16x2(pv[h][2 * e] - bf16_lo(ph_[e]), pv[h][2 * e + 1] - bf16_hi(ph_[e]));
        }
        const bf16x8 bh = __builtin_bit_cast(bf16x8, ph_), bl = __builtin_bit_cast(bf16x8, pl_);
        float y[8];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          floatx4 cacc;
#pragma unroll
          for (int e = 0; e < 4; ++e) cacc[e] = vt * bsel[mb][e];
          cacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amh[mb], bh, cacc, 0, 0, 0);
          cacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aml[mb], bh, cacc, 0, 0, 0);
          cacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amh[mb], bl, cacc, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) y[4 * mb + e] = cacc[e];
        }
        if (want_map) {
          char *pp = pst + wave * 3072;  // this wave's X, P high, P low rows of the pair
          *reinterpret_cast<u32x4 *>(pp + lane * 16) = xp;
          *reinterpret_cast<u32x4 *>(pp + 1024 + lane * 16) = ph_;
          *reinterpret_cast<u32x4 *>(pp + 2048 + lane * 16) = pl_;
          const bf16x8 xa = tr8(pp), pbh = tr8(pp + 1024), pbl = tr8(pp + 2048);
          dah = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, pbh, dah, 0, 0, 0);
          dal = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, pbl, dal, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            gb[e % D] = fmaf((e & 1) ? bf16_hi(xp[e >> 1]) : bf16_lo(xp[e >> 1]), vt, gb[e % D]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(y[2 * e], y[2 * e + 1]);
      }
      __builtin_amdgcn_raw_buffer_store_b128(w, ro, off, 0, 0);
    }
  }
  if (want_map) {
    constexpr int kSlots = 16 / D;
    __shared__ float mred[kW][kSlots * D * D + D];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int mrow = 4 * q + e;
      if (mrow / D == c16 / D) mred[wave][(mrow / D) * D * D + (mrow % D) * D + c16 % D] = dah[e] + dal[e];
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) gb[j] += __shfl_xor(gb[j], o, 64);
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < D; ++j) mred[wave][kSlots * D * D + j] = gb[j];
    }
    __syncthreads();
    if (tid < D * D + D) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < kW; ++w) {
        if (tid < D * D) {
#pragma unroll
          for (int sl = 0; sl < kSlots; ++sl) v += mred[w][sl * D * D + tid];
        } else {
          v += mred[w][kSlots * D * D + tid - D * D];
        }
      }
      mapp[(int64_t)tid * gridDim.x + blockIdx.x] = v;
    }
  }
}

// ---- the choice of tiles -----------------------------------------------------
// A product's time by tile: per round of tiles over the 256 compute units a fixed part
// (filling the pipeline, the epilogue) and a part per 64-wide step, plus a part per tile
// and step (the chip filling up: power, operand traffic).  Rows of dY that don't begin on
// 128-byte lines cost the small input-gradient tile, which reads them in 128-byte runs, up
// to a fifth.  X' of more than 250 MB falls out of the last-level cache, and the small
// tiles, which read it more often, count 1.15 times (us, wide / 128 rows / 64 rows: 16000
// tokens of 776 x 16384 319 / 342 / 500, 12000 of 2064 x 20000 748 / 796 / 1134).  Over 213 shapes
// of 64 .. 16384 tokens and 512 .. 28672 features the pick is 0.4 % from the fastest tile on
// average for either product, and slower than the wide tile by more than 0.3 % only once
// (1000 tokens of 1040 x 20000, input gradient, 75.8 against 74.0 us).  Measured: forward,
// 256 tokens of 4096 x 4096 80 / - / 12; 2048 of 4096 x 11008 213 / 128 / -; 4228 of 23936 x
// 1128 196 / 228 / 292; 5262 of 6280 x 10136 596 / 471 / 586.  Input gradient, 1000 of 11008 x
// 4096 217 / 79 / -; 958 of 26032 x 3176 483 / 169 / 219; 2404 of 22736 x 10056 894 / 993 / 1473;
// 4096^3 108 / 129 / -.
int codes_split_slabs(int64_t rows, int64_t tokens, int64_t K, bool dx) {
  struct Cost {  // ns: per round and step, per round, per 256 tiles and step, in all
    int64_t step, round, full, base;
  };
  constexpr Cost kCost[2][3] = {{{1080, 6400, 140, 2000}, {153, 1500, 12, 4900}, {92, 840, 21, 4000}},
                                {{1110, 17000, 175, 400}, {167, 3100, 12, 6000}, {124, 2100, 0, 5300}}};
  const int64_t KB = round_up(K, 128) / 64;
  auto cost = [&](int i, int64_t tiles) {
    const Cost &c = kCost[dx ? 1 : 0][i];
    const int64_t full = c.full + (dx && i > 0 && K % 64 != 0 ? 40 : 0);
    return ceil_div(tiles, 256) * (c.step * KB + c.round) + tiles * full * KB / 256 + c.base;
  };
  const int64_t tt = ceil_div(tokens, 64);
  const int64_t far = !dx && 2 * tokens * K > 250000000 ? 3 : 0;
  const int64_t c0 = cost(0, dx ? ceil_div(rows, 256) * ceil_div(tokens, 256) : ceil_div(rows, 512) * ceil_div(tokens, 128)),
                c4 = cost(1, ceil_div(rows, 128) * tt) * (20 + far) / 20,
                c2 = cost(2, ceil_div(rows, 64) * tt) * (20 + far) / 20;
  if (c0 <= c4 && c0 <= c2) return 0;
  return c2 < c4 ? 2 : 4;
}

// ---- launchers -----------------------------------------------------------------
template <int kMode, int D, int MI>
static hipError_t split_launch(const uint32_t *frag, int KB, const uint16_t *B, int64_t ldB, const float *vec, int parts,
                               int64_t vstride, const float *A, const float *b, uint16_t *out, int64_t rows, int64_t N,
                               const uint16_t *X, float *mapp, hipStream_t st) {
  const int tiles_m = (int)ceil_div(rows, 32 * MI), tiles_n = (int)ceil_div(N, 64);
  k_codes_split<kMode, D, MI><<<tiles_m * tiles_n, 256, 0, st>>>(frag, KB, B, ldB, tiles_m, tiles_n, vec, parts, vstride,
                                                                 A, b, out, rows, rows, N, X, mapp);
  return hipGetLastError();
}

hipError_t launch_fwd_split(int slabs, const uint32_t *frag, const uint16_t *Xp, int64_t ldp, const float *s, uint16_t *Y,
                            int64_t N, int64_t m, hipStream_t st) {
  const int KB = (int)(ldp / kKStep), parts = act_chunks(ldp);
  const int64_t Np = round_up(N, kTile);  // row stride of the partial sums of s
  auto go = slabs == 4 ? split_launch<0, 8, 4> : split_launch<0, 8, 2>;
  return go(frag, KB, Xp, 0, s, parts, Np, nullptr, nullptr, Y, m, N, nullptr, nullptr, st);
}

hipError_t launch_dx_split(int slabs, const uint32_t *frag, const uint16_t *dY, const float *rsp, const float *A,
                           const float *b, int d, uint16_t *dX, const uint16_t *X, float *mapp, int64_t N, int64_t m,
                           int64_t n, hipStream_t st) {
  const int KB = (int)(round_up(m, 128) / kKStep);
  auto go = d == 8 ? (slabs == 4 ? split_launch<1, 8, 4> : split_launch<1, 8, 2>)
                   : (slabs == 4 ? split_launch<1, 4, 4> : split_launch<1, 4, 2>);
  return go(frag, KB, dY, m, rsp, rowsum_parts(m), bwd_tokens(N), A, b, dX, n, N, X, mapp, st);
}

}  // namespace lcvq
