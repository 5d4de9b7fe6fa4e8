// Layer output straight from packed 2-bit codes for up to 16 tokens, for inference
// with the compressed weight (def. forward_x, Sec. 3.2; the paper's inference kernel,
// App. A.2, fuses decode, dot products and reduction in the same spirit):
//
//   Y[t, r] = sum_c code[r, c] X'[t, c] + s[t],  X' = X blockdiag(A) in bf16, s = X b~
//
// on v_mfma_f32_16x16x32_bf16 with 16 weight rows on M and the tokens on N.  The
// packed codes (0.25 byte per weight) are the only large stream and are read once.
// The operand forms (masked words into the fp4 converter, X' in even / odd column
// order, the codes through LDS in whole 64-byte runs) are those of
// lcvq_packed_wide.hip.
//
// Block: 16 MR weight rows; its kW waves split K (256-wide steps w, w + kW, ...) and
// add their tiles in LDS at the end, in wave order.  No split over blocks, so no
// second launch, counters or partial tiles in memory: small matrices get their
// parallelism from short tiles and many waves.  Every wave has the codes of its next
// step in flight while it works on the current one.
//
// Up to four tokens, each wave transforms its own steps' X (its 64 lanes are the 16
// column runs of four tokens, or half runs of two), and the call is one launch; above
// that a prepass writes X' once (k_packed_xprep).
//
// Bound: the codes' bytes plus, after the last of them has arrived, the last step's
// conversions and products (about 370 vector instructions per 64 rows x 256 columns);
// at 16 tokens also the X' fragments from the L2, twice the codes' bytes with 64 rows.
#include "lcvq_mfma.hpp"
#include "lcvq_prep.hpp"

namespace lcvq {

// kD: group size when the block transforms X itself, for up to kTok = 2 or 4 tokens;
// 0 when X' and the parts of s are ready in xq and sp.
template <int MR, int kW, int kD, int kTok>
__global__ __launch_bounds__(64 * kW, kW == 16 || MR > 4 ? 1 : 2) void k_packed(
    const uint8_t *__restrict__ packed, int64_t m, int64_t n, int KT, const uint16_t *__restrict__ xq,
    const float *__restrict__ sp, int parts, const uint16_t *__restrict__ X, const float *__restrict__ A,
    const float *__restrict__ b, int Nc, void *__restrict__ Y, int y_bf16) {
  constexpr bool kFused = kD > 0;
  constexpr int kD1 = kFused ? kD : 8;
  constexpr int kH = 4 / kTok;                  // lanes that share a run of 16 columns
  constexpr int kXB = kFused ? 512 * kTok : 0;  // bytes of X' operands per wave
  constexpr int kStage = 2 * MR * 1024 + kXB;
  static_assert(kStage >= MR * 1024 + 16, "the sums and the parts of s fit");
  __shared__ __attribute__((aligned(1024))) char lds[kW * kStage];
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t r0 = (int64_t)blockIdx.x * 16 * MR, ldb = n / 4;
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(packed + r0 * ldb, (m - r0 < 16 * MR ? m - r0 : 16 * MR) * ldb);
  const __amdgpu_buffer_rsrc_t rsX = kFused ? make_rsrc(X, (int64_t)Nc * n * 2) : make_rsrc(xq, (int64_t)KT * 8192);

  char *stage = lds + wave * kStage, *xst = stage + 2 * MR * 1024;
  const int lrow = lane >> 2, lpiece = (lane & 3) ^ ((lrow >> 1) & 3);
  const uint32_t aoff = (uint32_t)(lrow * ldb + 16 * lpiece), astep = (uint32_t)(16 * ldb);
  const uint32_t roff = (uint32_t)(c16 * 64 + ((q ^ ((c16 >> 1) & 3)) << 4));
  auto load_a = [&](int st, int j) {
#pragma unroll
    for (int k = 0; k < MR; ++k)
      buffer_to_lds16(rsA, (lds_void *)(stage + (st * MR + k) * 1024), j < KT ? aoff + k * astep + 64u * j : kOffNone);
  };
  // X of a step: the operand fragments, or (fused) the 16 / kH columns that lane (run
  // L % 16, q = L / 16) transforms: token q / kH, part q % kH of the run's 16
  constexpr int kXL = kFused ? 2 / kH : 8;
  const int tok = q / kH, h = q % kH;
  u32x4 xr[2][kXL];
  auto load_x = [&](int buf, int j) {
    if constexpr (kFused) {
      const int64_t c = (int64_t)j * 256 + 16 * c16 + 8 * h;
      const uint32_t off = j < KT && tok < Nc && c < n ? (uint32_t)((tok * n + c) * 2) : kOffNone;
#pragma unroll
      for (int i = 0; i < kXL; ++i)
        xr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(rsX, (int)(off == kOffNone ? kOffNone : off + 16u * i), 0, 0);
    } else {
      const bool live = j < KT && c16 < Nc;  // fragments of absent tokens are not read
#pragma unroll
      for (int i = 0; i < kXL; ++i)
        xr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(rsX, live ? (int)((j * 8 + i) * 1024 + lane * 16) : (int)kOffNone,
                                                           0, 0);
    }
  };
  float s = 0.0f;
  const int xtok = kFused ? (c16 < Nc ? c16 : 0) : 0;  // absent tokens read the first one's X'
  floatx4 acc[MR];
#pragma unroll
  for (int rb = 0; rb < MR; ++rb) acc[rb] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  auto compute = [&](int u) {
    if constexpr (kFused) {
      constexpr int kC = 16 / kH;  // columns per lane
      float x[kXL * 8], y[kC];
#pragma unroll
      for (int e = 0; e < 4 * kXL; ++e) {
        const uint32_t w = xr[u][e >> 2][e & 3];
        x[2 * e] = bf16_lo(w);
        x[2 * e + 1] = bf16_hi(w);
      }
#pragma unroll
      for (int g = 0; g < kC / kD1; ++g)
#pragma unroll
        for (int k = 0; k < kD1; ++k) {
          float v = 0.0f;
#pragma unroll
          for (int i = 0; i < kD1; ++i) v = fmaf(x[g * kD1 + i], A[i * kD1 + k], v);
          y[g * kD1 + k] = v;
          s = fmaf(x[g * kD1 + k], b[k], s);
        }
      // chunk (i, lane group, token) of 16 bytes: run c16 is lane group c16 / 4, dword
      // c16 % 4; this lane has its dwords kC / 4 h ..
      if (tok < Nc) {
        uint32_t *p = reinterpret_cast<uint32_t *>(xst + ((((c16 & 3) * 2) * 4 + (c16 >> 2)) * kTok + tok) * 16) + kC / 4 * h;
#pragma unroll
        for (int e = 0; e < kC / 4; ++e) {
          p[e] = pack_bf16x2(y[4 * e], y[4 * e + 2]);
          p[16 * kTok + e] = pack_bf16x2(y[4 * e + 1], y[4 * e + 3]);
        }
      }
    }
    u32x4 a[MR];
#pragma unroll
    for (int rb = 0; rb < MR; ++rb) a[rb] = *reinterpret_cast<const u32x4 *>(stage + (u * MR + rb) * 1024 + roff);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      u32x4 xf;
      if constexpr (kFused) xf = *reinterpret_cast<const u32x4 *>(xst + ((i * 4 + q) * kTok + xtok) * 16);
      else xf = xr[u][i];
#pragma unroll
      for (int rb = 0; rb < MR; ++rb) {
        const uint32_t w = a[rb][i >> 1];
        acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nibbles_to_bf16x8(((i & 1) ? w >> 2 : w) & 0x33333333u),
                                                          __builtin_bit_cast(bf16x8, xf), acc[rb], 0, 0, 0);
      }
    }
  };

  load_a(0, wave);
  load_x(0, wave);
  __builtin_amdgcn_sched_barrier(0);
  for (int j = wave; j < KT; j += 2 * kW) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && j + kW >= KT) break;
      load_a(u ^ 1, j + (u + 1) * kW);
      load_x(u ^ 1, j + (u + 1) * kW);
      __builtin_amdgcn_sched_barrier(0);
      LCVQ_WAIT_VM(MR + kXL);  // all but the loads just issued: this step's codes are in LDS
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      compute(u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ------------------------------------------------------------ epilogue
  if constexpr (kFused) {  // over the runs and parts of a token: every lane of it has the sum
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if constexpr (kH == 2) s += __shfl_xor(s, 16, 64);
  }
  LCVQ_WAIT_ALL();  // the last stage's loads have landed before the sums overwrite it
  __syncthreads();
  floatx4 *red = reinterpret_cast<floatx4 *>(lds);  // [wave][row block][lane]
  float *s_red = reinterpret_cast<float *>(lds + kW * MR * 1024);  // [wave][token]
#pragma unroll
  for (int rb = 0; rb < MR; ++rb) red[(wave * MR + rb) * 64 + lane] = acc[rb];
  if (kFused && c16 == 0 && h == 0) s_red[wave * 4 + tok] = s;
  __syncthreads();
  if (wave >= MR) return;
  // thread (rb = wave, lane): rows 16 rb + 4 q + (0..3), token L % 16
  floatx4 v = red[wave * 64 + lane];
#pragma unroll
  for (int w = 1; w < kW; ++w) v += red[(w * MR + wave) * 64 + lane];
  const int64_t row = r0 + 16 * wave + 4 * q;  // m is a multiple of 8: the four rows are all in or all out
  if (c16 >= Nc || row >= m) return;
  float st = 0.0f;
  if constexpr (kFused) {
#pragma unroll
    for (int w = 0; w < kW; ++w) st += s_red[w * 4 + (c16 & 3)];
  } else {
    for (int p = 0; p < parts; ++p) st += sp[p * 16 + c16];
  }
  const int64_t o = (int64_t)c16 * m + row;
  if (y_bf16) {
    uint2 w;
    w.x = pack_bf16x2(v[0] + st, v[1] + st);
    w.y = pack_bf16x2(v[2] + st, v[3] + st);
    *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(Y) + o) = w;
  } else {
    *reinterpret_cast<floatx4 *>(reinterpret_cast<float *>(Y) + o) = v + st;
  }
}

// ---------------------------------------------------------------- launch ---
bool packed_fused(int Nc) { return Nc <= 4; }

// Rows per block: 16 MR with the fewest rounds of blocks over the 256 compute units and
// those rounds full, MR at most 8, so that every unit gets the same share of the codes
// and reads or makes the X' of a step once per round (28672 x 8192 at one token: MR 4,
// 7 blocks for every 4 units, 20.4 us, MR 7, one for each, 17.6; 11008 x 4096: 7.3 with
// MR 4, 6.7 with 3; 8192 x 28672: 25.2 with 4, 18.7 with 2 and sixteen waves).  Sixteen
// waves where a block's rows are few and K gives each of them about two steps (4096 x
// 11008 7.3 -> 6.9, 4096 x 4096 4.4 against 4.5 without).
// Before (64-row blocks of four waves, K split over blocks, a prepass except for long
// rows): one token through 28672 x 8192 19.5, 8192 x 28672 24.7, 4096 x 11008 13.1,
// 11008 x 4096 15.1, 4096 x 4096 10.8 us, now 17.6, 18.7, 6.9, 6.7 and 4.4; 16 tokens 26.8,
// 33.2, 15.5, 19.9 and 12.5, now 23.4, 30.5, 14.4, 12.1 and 9.6.
template <int kD, int kTok>
static hipError_t launch(const uint8_t *packed, int64_t m, int64_t n, const PackedNarrow &p, const uint16_t *xq,
                         const float *sp, const uint16_t *X, const float *A, const float *b, int Nc, void *Y, bool y_bf16,
                         hipStream_t st) {
  const int64_t rb = ceil_div(m, 16), rounds = ceil_div(rb, 256 * 8);
  const int mr = (int)ceil_div(rb, 256 * rounds);
  const bool w16 = mr <= 2 && p.KT >= 24;
  using K = decltype(&k_packed<1, 8, kD, kTok>);
  static constexpr K k8[8] = {k_packed<1, 8, kD, kTok>, k_packed<2, 8, kD, kTok>, k_packed<3, 8, kD, kTok>,
                              k_packed<4, 8, kD, kTok>, k_packed<5, 8, kD, kTok>, k_packed<6, 8, kD, kTok>,
                              k_packed<7, 8, kD, kTok>, k_packed<8, 8, kD, kTok>};
  const K k = w16 ? (mr == 2 ? k_packed<2, 16, kD, kTok> : k_packed<1, 16, kD, kTok>) : k8[mr - 1];
  k<<<(unsigned)ceil_div(rb, mr), w16 ? 1024 : 512, 0, st>>>(packed, m, n, p.KT, xq, sp, p.parts, X, A, b, Nc, Y,
                                                             y_bf16 ? 1 : 0);
  return hipGetLastError();
}

PackedNarrow packed_narrow(int64_t n) {
  PackedNarrow p{};
  const PackedWidePlan w = packed_wide_plan(1, n, 0);
  p.KT = w.KT;
  p.spp = w.spp;
  p.parts = w.parts;
  p.sp = (int64_t)p.KT * 8192;
  p.bytes = p.sp + (int64_t)p.parts * 16 * 4;
  return p;
}

hipError_t launch_packed(const PackedNarrow &p, const uint8_t *packed, int64_t m, int64_t n, const char *ws, int Nc, void *Y,
                         bool y_bf16, hipStream_t st) {
  return launch<0, 4>(packed, m, n, p, (const uint16_t *)ws, (const float *)(ws + p.sp), nullptr, nullptr, nullptr, Nc, Y,
                      y_bf16, st);
}

hipError_t launch_packed_fused(const PackedNarrow &p, const uint8_t *packed, int64_t m, int64_t n, const uint16_t *X, int Nc,
                               int d, const float *A, const float *b, void *Y, bool y_bf16, hipStream_t st) {
  auto go = d == 8 ? (Nc <= 2 ? launch<8, 2> : launch<8, 4>) : (Nc <= 2 ? launch<4, 2> : launch<4, 4>);
  return go(packed, m, n, p, nullptr, nullptr, X, A, b, Nc, Y, y_bf16, st);
}

}  // namespace lcvq
