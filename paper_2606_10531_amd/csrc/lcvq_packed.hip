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
// add their tiles in LDS at the end, in wave order.  K is not split over blocks, so there
// is no second launch and no partial tile in memory (small matrices get their
// parallelism from short tiles and many waves), except for few rows over more than 32512
// columns (packed_split).  Each wave has two stages: the loads of
// its next step, X first, are issued before the current step is multiplied, and that
// starts with X and takes two row blocks of codes at a time as they arrive, so that
// little is left to do behind the last load.
//
// Up to four tokens, each wave transforms its own steps' X (its 64 lanes are the 16
// column runs of four tokens, or half runs of two), and the call is one launch; above
// that a prepass writes X' once (k_packed_xprep).
//
// Bound: the codes' bytes plus, after the last of them has arrived, two row blocks'
// conversions and products and the waves' sum; at 16 tokens also the X' fragments from
// the L2, twice the codes' bytes with 64 rows.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "lcvq_mfma.hpp"
#include "lcvq_prep.hpp"

namespace lcvq {

// At most N loads in flight; nothing moves across.
template <int N>
__device__ __forceinline__ void wait_vm() {
  LCVQ_WAIT_VM(N);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int... I, class F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for(std::make_integer_sequence<int, N>{}, f);
}

constexpr int kNarrowParts = 32;  // most parts of s of a pass

// kD: group size when the block transforms X itself, for up to kTok = 2 or 4 tokens;
// 0 when X' and the parts of s are ready in xq and sp.  kSplit: block (x, y) takes the
// steps [y span, (y + 1) span) and stores its sums in `part` (span y, token, row), the
// first row tile also its part of s (fused) in `part_s` (span y, 16 tokens), for
// k_packed_sum.
template <int MR, int kW, int kD, int kTok, bool kSplit = false>
__global__ __launch_bounds__(64 * kW, kW == 16 || MR > 4 ? 1 : 2) void k_packed(
    const uint8_t *__restrict__ packed, int64_t m, int64_t n, int KT, const uint16_t *__restrict__ xq,
    const float *__restrict__ sp, int parts, const uint16_t *__restrict__ X, const float *__restrict__ A,
    const float *__restrict__ b, int Nc, void *__restrict__ Y, int y_bf16, int span, float *__restrict__ part,
    float *__restrict__ part_s) {
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
  const int j0 = kSplit ? (int)blockIdx.y * span : 0;
  if constexpr (kSplit) KT = min(KT, j0 + span);  // the block's steps
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(packed + r0 * ldb, (m - r0 < 16 * MR ? m - r0 : 16 * MR) * ldb);
  const __amdgpu_buffer_rsrc_t rsX = kFused ? make_rsrc(X, (int64_t)Nc * n * 2) : make_rsrc(xq, (int64_t)KT * 8192);

  char *stage = lds + wave * kStage, *xst = stage + 2 * MR * 1024;
  const int lrow = lane >> 2, lpiece = (lane & 3) ^ ((lrow >> 1) & 3);
  const uint32_t aoff = (uint32_t)(lrow * ldb + 16 * lpiece), astep = (uint32_t)(16 * ldb);
  const uint32_t roff = (uint32_t)(c16 * 64 + ((q ^ ((c16 >> 1) & 3)) << 4));
  auto load_a = [&](int st, int j) {
    uint32_t base = (uint32_t)(wave * kStage + st * MR * 1024);
    asm volatile("" : "+s"(base));  // the addresses are made here: held over the loop, they would crowd out A
#pragma unroll
    for (int k = 0; k < MR; ++k)
      buffer_to_lds16(rsA, (lds_void *)(lds + base + k * 1024), j < KT ? aoff + k * astep + 64u * j : kOffNone);
  };
  // X of a step: the operand fragments, or (fused) the 16 / kH columns that lane (run
  // L % 16, q = L / 16) transforms: token q / kH, part q % kH of the run's 16
  constexpr int kXL = kFused ? 2 / kH : 8;
  const int tok = q / kH, h = q % kH;
  u32x4 xr[2][kXL];
  auto load_x = [&](int buf, int j) {
    if constexpr (kFused) {
      const int c = j * 256 + 16 * c16 + 8 * h;  // (steps past KT lie past n)
      const uint32_t off = tok < Nc && c < (int)n ? (uint32_t)(tok * (int)n + c) * 2u : kOffNone;
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
  float am[kD1][kD1], bm[kD1];  // (fused) the map, in scalar registers for all steps
  float s = 0.0f;
  const int xtok = kFused ? (c16 < Nc ? c16 : 0) : 0;  // absent tokens read the first one's X'
  floatx4 acc[MR];
#pragma unroll
  for (int rb = 0; rb < MR; ++rb) acc[rb] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  // the step's X' operands: transformed here through the wave's LDS (fused), or as loaded
  auto operands = [&](int u, u32x4 (&xf)[8]) __attribute__((always_inline)) {
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
          for (int i = 0; i < kD1; ++i) v = fmaf(x[g * kD1 + i], am[i][k], v);
          y[g * kD1 + k] = v;
          s = fmaf(x[g * kD1 + k], bm[k], s);
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
#pragma unroll
      for (int i = 0; i < 8; ++i) xf[i] = *reinterpret_cast<const u32x4 *>(xst + ((i * 4 + q) * kTok + xtok) * 16);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) xf[i] = xr[u][i];
    }
  };
  auto rows = [&](int u, int rb0, int nrb, const u32x4 (&xf)[8]) __attribute__((always_inline)) {
    u32x4 a[MR];
#pragma unroll
    for (int rb = rb0; rb < rb0 + nrb; ++rb) a[rb] = *reinterpret_cast<const u32x4 *>(stage + (u * MR + rb) * 1024 + roff);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int rb = rb0; rb < rb0 + nrb; ++rb) {
        const uint32_t w = a[rb][i >> 1];
        acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nibbles_to_bf16x8(((i & 1) ? w >> 2 : w) & 0x33333333u),
                                                          __builtin_bit_cast(bf16x8, xf[i]), acc[rb], 0, 0, 0);
      }
  };
  // One step from stage u, with kLater younger loads in flight: X first, which its codes'
  // loads follow, then two row blocks at a time as they arrive.
  auto step = [&](auto later, int u) __attribute__((always_inline)) {
    constexpr int kLater = decltype(later)::value;
    u32x4 xf[8];
    wait_vm<kLater + MR>();
    operands(u, xf);
    __builtin_amdgcn_sched_barrier(0);
    static_for<(MR + 2 - 1) / 2>([&](auto g) __attribute__((always_inline)) {
      constexpr int rb = 2 * decltype(g)::value, n = MR - rb < 2 ? MR - rb : 2;
      wait_vm<kLater + MR - rb - n>();
      rows(u, rb, n, xf);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto load = [&](int u, int j) __attribute__((always_inline)) {  // kXL + MR loads
    load_x(u, j);
    __builtin_amdgcn_sched_barrier(0);
    load_a(u, j);
    __builtin_amdgcn_sched_barrier(0);
  };
  load(0, j0 + wave);
  if constexpr (kFused) {  // (behind the first loads: nothing waits for it before they are out)
#pragma unroll
    for (int i = 0; i < kD1; ++i) {
      bm[i] = b[i];
#pragma unroll
      for (int k = 0; k < kD1; ++k) am[i][k] = A[i * kD1 + k];
    }
  }
  // Steps in pairs, the last of an odd number behind the loop.  There is no way out
  // between the loads and the step they belong to: with one, the compiler had moved the
  // loads behind it, or waited for all of them at the loop's head.
  int j = j0 + wave;
  for (; j + kW < KT; j += 2 * kW) {
    load(1, j + kW);
    step(std::integral_constant<int, MR + kXL>{}, 0);
    load(0, j + 2 * kW);
    step(std::integral_constant<int, MR + kXL>{}, 1);
  }
  if (j < KT) step(std::integral_constant<int, 0>{}, 0);

  // ------------------------------------------------------------ epilogue
  if constexpr (kFused) {  // over the runs and parts of a token: every lane of it has the sum
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if constexpr (kH == 2) s += __shfl_xor(s, 16, 64);
  }
  float st = 0.0f;
  if constexpr (!kFused && !kSplit) {  // read here, under the waits: behind the sums it costs up to 1 us
    // the four lanes of a token take every fourth part (one lane for all of them was a
    // chain of loads: 14336 x 4096 at 16 tokens 11.1 us a call, now 9.9)
    if (wave < MR) {
#pragma unroll
      for (int i = 0; i < kNarrowParts / 4; ++i)
        if (c16 < Nc && 4 * i + q < parts) st += sp[(4 * i + q) * 16 + c16];
      st += __shfl_xor(st, 16, 64);
      st += __shfl_xor(st, 32, 64);
    }
  }
  LCVQ_WAIT_ALL();  // the last stage's loads have landed before the sums overwrite it
  __syncthreads();
  floatx4 *red = reinterpret_cast<floatx4 *>(lds);  // [wave][row block][lane]
  float *s_red = reinterpret_cast<float *>(lds + kW * MR * 1024);  // [wave][token]
  if (c16 < Nc) {  // (absent tokens' columns are not summed)
#pragma unroll
    for (int rb = 0; rb < MR; ++rb) red[(wave * MR + rb) * 64 + lane] = acc[rb];
  }
  if (kFused && c16 == 0 && h == 0) s_red[wave * 4 + tok] = s;
  __syncthreads();
  if constexpr (kFused) {
#pragma unroll
    for (int w = 0; w < kW; ++w) st += s_red[w * 4 + (c16 & 3)];
    if (kSplit && blockIdx.x == 0 && tid < Nc) part_s[blockIdx.y * 16 + tid] = st;  // (lane t: token t)
  }
  // thread (rb, lane): rows 16 rb + 4 q + (0..3), token L % 16
  for (int rb = wave; rb < MR; rb += kW) {
    const int64_t row = r0 + 16 * rb + 4 * q;  // m is a multiple of 8: the four rows are all in or all out
    if (c16 >= Nc || row >= m) return;
    floatx4 v = red[rb * 64 + lane];
#pragma unroll
    for (int w = 1; w < kW; ++w) v += red[(w * MR + rb) * 64 + lane];
    if constexpr (kSplit) {
      *reinterpret_cast<floatx4 *>(part + ((int64_t)blockIdx.y * Nc + c16) * m + row) = v;
      continue;
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
}

// Four rows of a token per thread: the spans' sums in order, and s.
__global__ __launch_bounds__(256) void k_packed_sum(const float *__restrict__ part, int spans, int64_t m, int Nc,
                                                    const float *__restrict__ sp, int parts, void *__restrict__ Y,
                                                    int y_bf16) {
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const int t = blockIdx.y, lane = threadIdx.x & 63;
  float st = lane < parts ? sp[lane * 16 + t] : 0.0f;  // at most 64 parts, one per lane
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) st += __shfl_xor(st, o, 64);
  if (row >= m) return;
  const float *p = part + t * m + row;
  floatx4 v = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int i = 0; i < spans; ++i) v += *reinterpret_cast<const floatx4 *>(p + (int64_t)i * Nc * m);
  const int64_t o = (int64_t)t * m + row;
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
// and reads or makes the X' of a step once per round (28672 x 8192: MR 7, one block for
// each unit; with MR 4, 7 blocks for every 4 units, 16.6 us against 16.7 at one token, but
// 11008 x 4096 7.3 against 6.7 with 3 and 8192 x 28672 23.1 against 16.4 with 2).
// Waves: sixteen where a block's rows are few and K gives each of them about two steps
// (4096 x 11008 7.3 -> 6.9, 4096 x 4096 4.4 against 4.5 without).  Four where the block
// transforms X itself, has 64 rows or more and K is 16 to 63 steps, so that each wave has
// four or more of them: longer chains of steps hide the waits better than more waves (one
// token, eight -> four waves: 28672 x 8192 16.6 -> 15.2 us, 20480 x 4096 8.6 -> 7.6, 16384 x
// 6144 9.0 -> 8.6; but 28672 x 2048, eight steps in all, 6.5 -> 6.9, 32768 x 16384 34.9 ->
// 35.8, 8192 x 8192 with 32 rows 7.0 -> 7.6).  Eight elsewhere.
// Against 64-row blocks of four waves with K split over blocks and a prepass except for
// long rows (one graph of calls, weights from memory, us): one token through 28672 x 8192
// 15.9 -> 14.6, 8192 x 28672 22.3 -> 15.7, 4096 x 11008 12.8 -> 6.4, 11008 x 4096 14.3 -> 5.8,
// 4096 x 4096 10.9 -> 4.3; 16 tokens 23.6 -> 20.4, 28.9 -> 25.1, 14.6 -> 10.7, 18.7 -> 9.1 and
// 12.7 -> 8.1.
template <int kD, int kTok>
static hipError_t launch(const uint8_t *packed, int64_t m, int64_t n, const PackedNarrow &p, const PackedSplit &split,
                         char *ws, const uint16_t *X, const float *A, const float *b, int Nc, void *Y, bool y_bf16,
                         hipStream_t st) {
  const uint16_t *xq = kD > 0 ? nullptr : (const uint16_t *)ws;
  const float *sp = kD > 0 ? nullptr : (const float *)(ws + p.sp);
  if (split.spans > 0) {
    float *part_s = (float *)(ws + split.sp), *part = (float *)(ws + split.part);
    k_packed<4, 4, kD, kTok, true><<<dim3((unsigned)ceil_div(m, 64), (unsigned)split.spans), 256, 0, st>>>(
        packed, m, n, p.KT, xq, nullptr, 0, X, A, b, Nc, Y, 0, split.span, part, part_s);
    k_packed_sum<<<dim3((unsigned)ceil_div(m, 1024), (unsigned)Nc), 256, 0, st>>>(
        part, split.spans, m, Nc, part_s, kD > 0 ? split.spans : split.parts, Y, y_bf16 ? 1 : 0);
    return hipGetLastError();
  }
  const int64_t rb = ceil_div(m, 16), rounds = ceil_div(rb, 256 * 8);
  const int mr = (int)ceil_div(rb, 256 * rounds);
  using K = decltype(&k_packed<1, 8, kD, kTok>);
  static constexpr K k8[8] = {k_packed<1, 8, kD, kTok>, k_packed<2, 8, kD, kTok>, k_packed<3, 8, kD, kTok>,
                              k_packed<4, 8, kD, kTok>, k_packed<5, 8, kD, kTok>, k_packed<6, 8, kD, kTok>,
                              k_packed<7, 8, kD, kTok>, k_packed<8, 8, kD, kTok>};
  K k = k8[mr - 1];
  int waves = 8;
  if (mr <= 2 && p.KT >= 24) {
    k = mr == 2 ? k_packed<2, 16, kD, kTok> : k_packed<1, 16, kD, kTok>;
    waves = 16;
  }
  if constexpr (kD > 0) {
    static constexpr K k4[5] = {k_packed<4, 4, kD, kTok>, k_packed<5, 4, kD, kTok>, k_packed<6, 4, kD, kTok>,
                                k_packed<7, 4, kD, kTok>, k_packed<8, 4, kD, kTok>};
    if (mr >= 4 && p.KT >= 16 && p.KT < 64) {
      k = k4[mr - 4];
      waves = 4;
    }
  }
  k<<<(unsigned)ceil_div(rb, mr), 64 * waves, 0, st>>>(packed, m, n, p.KT, xq, sp, p.parts, X, A, b, Nc, Y, y_bf16 ? 1 : 0, 0,
                                                        nullptr, nullptr);
  return hipGetLastError();
}

// Parts of s: of up to four steps, which the prepass takes side by side, as long as they
// are at most kNarrowParts (5120 x 28672 at 16 tokens: 16 parts of seven steps 26.6 us a
// call, 28 of four 25.6).
PackedNarrow packed_narrow(int64_t n) {
  PackedNarrow p{};
  p.KT = (int)ceil_div(n, 256);
  p.spp = std::max((int)ceil_div(p.KT, kNarrowParts), std::min((int)ceil_div(p.KT, kMaxActChunks), 4));
  p.parts = p.spp > 0 ? (int)ceil_div(p.KT, p.spp) : 0;
  p.sp = (int64_t)p.KT * 8192;
  p.bytes = p.sp + (int64_t)p.parts * 16 * 4;
  return p;
}

// Blocks of 64 rows that split K where up to 6144 rows meet 128 steps of K or more: one
// block's chain of steps is then longer than the second launch that adds the spans (a
// block for each compute unit, or two above 4096 rows; at most 16 spans).  Us a call,
// split / not, at 1, 4 and 16 tokens: 1024 x 65536 9.7 / 21.3, 10.7 / 30.7 and 17.1 / 41.8; 4096 x
// 40960 14.5 / 15.1, 16.7 / 21.1 and 21.0 / 29.7; 2048 x 131008 20 / 39, 24 / 59 and 33 / 84.  Not
// below: 2048 x 28672 9.9 / 11.1 and 11.7 / 15.4, but 18.4 / 17.9 at 16, 4096 x 28672 12.1 / 11.4;
// nor with more rows: 8192 x 65536 37.8 / 33.9 at one token.  The workspace does not depend
// on m, and what does not fit in the fixed array is not split with a workspace either, so
// that both give the same bits.
constexpr int64_t kMaxSplitRows = 32768;  // spans times rows
int64_t packed_split_bytes(int64_t n) {
  const PackedNarrow w = packed_narrow(n);
  const int64_t bytes = round_up(w.bytes, 256) + 64 * 64 + kMaxSplitRows * 64;
  return w.KT < 128 || bytes > kPackedScratchBytes ? 0 : bytes;
}

PackedSplit packed_split(int64_t m, int64_t n) {
  PackedSplit p{};
  const PackedNarrow w = packed_narrow(n);
  const int64_t tiles = ceil_div(m, 64);
  if (packed_split_bytes(n) == 0 || tiles < 1 || tiles > 96) return p;
  const int64_t most = std::min<int64_t>((tiles > 64 ? 512 : 256) / tiles, 16);
  p.span = (int)ceil_div(w.KT, most);
  p.spans = (int)ceil_div(w.KT, p.span);
  p.spp = std::max(4, (int)ceil_div(w.KT, 64));
  p.parts = (int)ceil_div(w.KT, p.spp);
  p.sp = round_up(w.bytes, 256);
  p.part = p.sp + 64 * 64;  // at most 64 parts of s of 16 tokens
  p.bytes = p.part + p.spans * m * 64;
  return p;
}

hipError_t launch_packed(const PackedNarrow &p, const PackedSplit &split, const uint8_t *packed, int64_t m, int64_t n,
                         char *ws, int Nc, void *Y, bool y_bf16, hipStream_t st) {
  return launch<0, 4>(packed, m, n, p, split, ws, nullptr, nullptr, nullptr, Nc, Y, y_bf16, st);
}

hipError_t launch_packed_fused(const PackedNarrow &p, const PackedSplit &split, const uint8_t *packed, int64_t m,
                               int64_t n, char *ws, const uint16_t *X, int Nc, int d, const float *A, const float *b,
                               void *Y, bool y_bf16, hipStream_t st) {
  auto go = d == 8 ? (Nc <= 2 ? launch<8, 2> : launch<8, 4>) : (Nc <= 2 ? launch<4, 2> : launch<4, 4>);
  return go(packed, m, n, p, split, ws, X, A, b, Nc, Y, y_bf16, st);
}

}  // namespace lcvq
