// Layer output from packed 2-bit codes for more than 16 tokens (prompts, large
// decode batches): Y[t, r] = sum_c code[r, c] X'[t, c] + s[t], X' = X blockdiag(A)
// rounded to bf16, s = X b~ (def. forward_x, Sec. 3.2), with the codes read in
// their packed form and never written out wider.
//
//   prepass : X' in the product's B-operand order, partial sums of s.
//   product : block tile 32 MI rows x 64 tokens; the four waves split K (256-wide
//             steps w, w + 4, ...), each with an accumulator of the whole tile, and
//             add their sums through LDS at the end, as k_codes_split does.
//
// Operands.  A row's 16-byte piece q of a step holds the codes of columns
// 64 q .. 64 q + 63 of the step's 256.  Its dword kk masked with 0x33333333 is eight
// 4-bit codes (columns 16 kk + 0, 2, .. 14 of the piece), shifted by two first the
// odd ones: each feeds the fp4 converter as it is, exact for 0 .. 3.  So sub-step
// (kk, par) of the step multiplies, in lane group q, columns 64 q + 16 kk + 2 e + par,
// e = 0 .. 7, and X' is stored in that order: fragment 2 kk + par of (16 tokens, step)
// is 64 lanes x 16 bytes.
//
// The codes come by direct-to-LDS loads with neighbouring lanes on neighbouring
// memory (four lanes per 64-byte run of a row; with the operand's own mapping,
// neighbouring lanes a row apart, a load takes the address path 64 cycles instead of
// 16), each wave into its own two stages of its next and current step, so no barrier
// is needed.  Piece q of row r sits at slot q ^ ((r / 2) % 4) of the row's 64 bytes,
// which keeps the 16-byte reads free of bank conflicts.
//
// Bound: the matrix core where the tiles fill the chip, else operand latency.  The
// 16-token passes that this replaces read the codes once per 16 tokens and took two
// launches each: 512 tokens through 11008 x 4096 and 4096 x 11008 1033 us, now 86.
#include <algorithm>

#include "lcvq_mfma.hpp"
#include "lcvq_prep.hpp"

namespace lcvq {

constexpr int kWk = 256;  // K columns per step

// Block (tb, p): tokens 16 tb .. + 15, steps [p spp, (p + 1) spp), up to four of them
// at a time (waves 4 i .. 4 i + 3 take the part's steps i, i + blockDim / 256, ..:
// a step costs a latency of loads; 512 tokens of 11008 columns take 8.4 us, 256 took
// 7.7 with one step at a time).
// Wave kk of a step, lane (token L % 16, q = L / 16): columns 64 q + 16 kk .. + 15.
template <int D>
__global__ __launch_bounds__(1024) void k_packed_xprep(const uint16_t *__restrict__ X, int Nc, int64_t n, int KT, int spp,
                                                       const float *__restrict__ A, const float *__restrict__ b,
                                                       uint16_t *__restrict__ xq, float *__restrict__ sp, int Tp) {
  __shared__ float red[16][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kk = wave & 3, q = lane >> 4, c16 = lane & 15;
  const int tb = blockIdx.x, p = blockIdx.y, t = 16 * tb + c16;
  const uint16_t *row = X + (int64_t)(t < Nc ? t : 0) * n;
  u32x4 *dst = reinterpret_cast<u32x4 *>(xq) + (int64_t)tb * KT * 8 * 64 + 2 * kk * 64 + lane;
  float s = 0.0f;
  const int j1 = min(KT, (p + 1) * spp);
  for (int j = p * spp + (wave >> 2); j < j1; j += (int)blockDim.x >> 8) {
    const int64_t c = (int64_t)j * kWk + 64 * q + 16 * kk;
    u32x4 w[2] = {u32x4{0u, 0u, 0u, 0u}, u32x4{0u, 0u, 0u, 0u}};
    if (t < Nc && c < n) {  // n is a multiple of 64: the 16 columns are in or out together
      w[0] = *reinterpret_cast<const u32x4 *>(row + c);
      w[1] = *reinterpret_cast<const u32x4 *>(row + c + 8);
    }
    float x[16], y[16];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      x[2 * e] = bf16_lo(w[e >> 2][e & 3]);
      x[2 * e + 1] = bf16_hi(w[e >> 2][e & 3]);
    }
#pragma unroll
    for (int g = 0; g < 16 / D; ++g)
#pragma unroll
      for (int k = 0; k < D; ++k) {
        float v = 0.0f;
#pragma unroll
        for (int i = 0; i < D; ++i) v = fmaf(x[g * D + i], A[i * D + k], v);
        y[g * D + k] = v;
        s = fmaf(x[g * D + k], b[k], s);
      }
    u32x4 ev, od;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ev[e] = pack_bf16x2(y[4 * e], y[4 * e + 2]);
      od[e] = pack_bf16x2(y[4 * e + 1], y[4 * e + 3]);
    }
    dst[(int64_t)j * 512] = ev;
    dst[(int64_t)j * 512 + 64] = od;
  }
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  if (lane < 16) red[wave][lane] = s;
  __syncthreads();
  if (threadIdx.x < 16) {
    float v = red[0][threadIdx.x];
    for (int w = 1; w < (int)blockDim.x >> 6; ++w) v += red[w][threadIdx.x];
    sp[(int64_t)p * Tp + 16 * tb + threadIdx.x] = v;
  }
}

template <int MI, bool kYBf16>
__global__ __launch_bounds__(256, 2) void k_packed_wide(const uint8_t *__restrict__ packed, int64_t m, int64_t n, int KT,
                                                        const uint16_t *__restrict__ xq, int tiles_m, int tiles_n,
                                                        const float *__restrict__ sp, int parts, int Tp, int Nc,
                                                        void *__restrict__ Y) {
  constexpr int P = 2 * MI;
  __shared__ __attribute__((aligned(1024))) char lds[65536];  // codes stages, then the waves' sums
  static_assert(4 * 2 * P * 1024 <= 65536, "two stages per wave");
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of_block(tiles_m, tiles_n, tm, tn);
  const int64_t r0 = (int64_t)tm * 32 * MI, ldb = n / 4;
  const int t0 = tn * 64;
  // rows past m lie beyond the buffer (their codes meet no stored output)
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(packed + r0 * ldb, (m - r0 < 32 * MI ? m - r0 : 32 * MI) * ldb);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(xq + (int64_t)(t0 >> 4) * KT * 4096, (int64_t)4 * KT * 8192);

  floatx4 acc[P][4];  // [row block 2 mi + rb][16-token block tb]
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  acc_fence(acc);

  // ---- codes: load k of a step brings 16 rows, lane L row 16 k + L / 4, slot L % 4
  char *stage = lds + wave * (2 * P * 1024);
  const int lrow = lane >> 2, lpiece = (lane & 3) ^ ((lrow >> 1) & 3);
  const uint32_t aoff = (uint32_t)(lrow * ldb + 16 * lpiece), astep = (uint32_t)(16 * ldb);
  auto load_a = [&](int st, int j) {
#pragma unroll
    for (int k = 0; k < P; ++k)
      buffer_to_lds16(rsA, (lds_void *)(stage + (st * P + k) * 1024), j < KT ? aoff + k * astep + 64u * j : kOffNone);
  };
  // operand row 16 rb + L % 16 of slab mi is weight row 32 mi + slab_row(16 rb + L % 16)
  uint32_t roff[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const int r = slab_row(16 * rb + c16);
    roff[rb] = (uint32_t)(r * 64 + ((q ^ ((r >> 1) & 3)) << 4));
  }
  u32x4 a[P];  // the lane's pieces of the current step
  auto get_a = [&](int st) {
#pragma unroll
    for (int p = 0; p < P; ++p)
      a[p] = *reinterpret_cast<const u32x4 *>(stage + st * P * 1024 + (p >> 1) * 2048 + roff[p & 1]);
  };
  // ---- X': group (step, kk) of eight fragments, two groups ahead
  u32x4 cb[2][2][4];  // [buffer][par][token block]
  auto load_b = [&](int buf, int j, int kk) {
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
        cb[buf][par][tb] = __builtin_amdgcn_raw_buffer_load_b128(
            rsB, j < KT ? (int)(((tb * KT + j) * 8 + 2 * kk + par) * 1024 + lane * 16) : (int)kOffNone, 0, 0);
  };
  auto conv = [&](int kk, int s2) {  // operand s2 = P par + p of dword kk
    const uint32_t w = a[s2 % P][kk];
    return nibbles_to_bf16x8_ordered((s2 < P ? w : w >> 2) & 0x33333333u);
  };
  auto compute = [&](int kk) {
    const int buf = kk & 1;
    bf16x8 an = conv(kk, 0);
#pragma unroll
    for (int s2 = 0; s2 < 2 * P; ++s2) {
      const int par = s2 / P, p = s2 % P;
      const bf16x8 av = an;
      if (s2 == 0) mfma16_valu_a(acc[p][0], av, __builtin_bit_cast(bf16x8, cb[buf][par][0]));
      else mfma16(acc[p][0], av, __builtin_bit_cast(bf16x8, cb[buf][par][0]));
      mfma16(acc[p][1], av, __builtin_bit_cast(bf16x8, cb[buf][par][1]));
      if (s2 + 1 < 2 * P) an = conv(kk, s2 + 1);
      mfma16(acc[p][2], av, __builtin_bit_cast(bf16x8, cb[buf][par][2]));
      mfma16(acc[p][3], av, __builtin_bit_cast(bf16x8, cb[buf][par][3]));
    }
  };

  // Per step: its codes are read from the stage, the next step's codes go on their
  // way into the other one, and the four groups run with the loads of the group
  // after next issued behind each.  The wait before a stage is read allows the 16
  // loads issued after that stage's (two groups) to be in flight; the first one
  // holds everything back.
  load_a(0, wave);
  __builtin_amdgcn_sched_barrier(0);
  load_b(0, wave, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_b(1, wave, 1);
  __builtin_amdgcn_sched_barrier(0);
  int st = 0;
  for (int j = wave; j < KT; j += 4) {
    LCVQ_WAIT_VM(16);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    get_a(st);
    st ^= 1;
    __builtin_amdgcn_sched_barrier(0);
    load_a(st, j + 4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      compute(kk);
      __builtin_amdgcn_sched_barrier(0);
      load_b(kk & 1, kk < 2 ? j : j + 4, (kk + 2) & 3);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  LCVQ_WAIT_ALL();  // the last stage's loads have landed before the sums overwrite it
  mfma_drain();
  __syncthreads();

  // ---- the waves' sums, two slabs at a time; wave w finishes tokens 16 w .. + 15
  const int tl = 16 * wave + c16, t = t0 + tl;
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * i + q < parts && t < Nc) s += sp[(int64_t)(4 * i + q) * Tp + t];
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
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
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      floatx4 v[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        v[k] = red[0][wave][2 * h + k][lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) v[k] += red[w][wave][2 * h + k][lane];
        v[k] += s;
      }
      const int64_t r = r0 + 32 * (2 * ph + h) + 8 * q;  // m is a multiple of 8
      if (t < Nc && r < m) {
        if constexpr (kYBf16) {
          u32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(v[e >> 1][2 * (e & 1)], v[e >> 1][2 * (e & 1) + 1]);
          *reinterpret_cast<u32x4 *>(reinterpret_cast<uint16_t *>(Y) + (int64_t)t * m + r) = w;
        } else {
          floatx4 *dst = reinterpret_cast<floatx4 *>(reinterpret_cast<float *>(Y) + (int64_t)t * m + r);
          dst[0] = v[0];
          dst[1] = v[1];
        }
      }
    }
  }
}

// Most tokens of a pass: its grid has a thread per 16 outputs (64-row tiles), which for the
// most out-features (2^21) has to stay below 2^32.  (In-features of 1024 or more hit the
// workspace limit first.)
constexpr int64_t kMaxPassTokens = (int64_t)1 << 15;

// Tokens per pass: as many whole 64-token tiles as `bytes` hold, in passes of equal
// size.  A token's result does not depend on the pass or the tile it falls in (the
// waves' shares of K, the order of their sums and the parts of s follow from n alone),
// so every workspace of at least 64 tokens gives the same bits; 16-token passes, which
// packed_passes picks by the sizes alone, sum in another order.
PackedWidePlan packed_wide_plan(int64_t N, int64_t n, int64_t bytes) {
  PackedWidePlan p{};
  p.KT = (int)ceil_div(n, kWk);
  p.spp = (int)ceil_div(p.KT, kMaxActChunks);
  p.parts = p.spp > 0 ? (int)ceil_div(p.KT, p.spp) : 0;
  p.per_token = (int64_t)p.KT * kWk * 2 + p.parts * 4;
  const int64_t most = p.per_token > 0 ? std::min(bytes / p.per_token / 64 * 64, kMaxPassTokens) : 0;
  if (N <= 16 || most < 64) return p;  // T = 0: 16-token passes
  p.T = (int)round_up(ceil_div(N, ceil_div(N, most)), 64);
  p.sp = (int64_t)p.T * p.KT * kWk * 2;
  p.bytes = p.T * p.per_token;
  return p;
}

// The most that any number of tokens up to N takes in a pass of up to kPackedWideBytes,
// i.e. one pass while they fit, else the largest pass.
int64_t packed_wide_bytes(int64_t N, int64_t n) {
  const int64_t per_token = packed_wide_plan(1, n, 0).per_token;
  if (N <= 16 || per_token == 0) return 0;
  return std::min({round_up(N, 64), kPackedWideBytes / per_token / 64 * 64, kMaxPassTokens}) * per_token;
}

hipError_t launch_packed_xprep(const uint16_t *X, int Nc, int64_t n, int KT, int spp, int parts, int d, const float *A,
                               const float *b, uint16_t *xq, float *sp, int Tp, hipStream_t st) {
  const dim3 g((unsigned)ceil_div(Nc, 16), (unsigned)parts);
  const unsigned threads = 256u * (unsigned)(spp < 4 ? spp : 4);
  (d == 8 ? k_packed_xprep<8> : k_packed_xprep<4>)<<<g, threads, 0, st>>>(X, Nc, n, KT, spp, A, b, xq, sp, Tp);
  return hipGetLastError();
}

// ns per 64 K of the tiles of a pass, 128 or 64 rows (one tile with the chip full, times the
// rounds of tiles over the compute units)
static int64_t wide_ns(int64_t N, int64_t m, bool four) {
  return (four ? 187 : 117) * ceil_div(ceil_div(m, four ? 128 : 64) * ceil_div(N, 64), 256);
}

// Whether passes of 16 tokens finish sooner: a wide tile's four waves take KT / 4 steps each
// whatever the tokens, so with few tokens and few rows over a long K they leave the chip
// idle.  ns, fitted to 648 calls of 17 .. 48 tokens, 64 .. 28672 rows and 1024 .. 40960 columns
// (the pick is 0.3 % from the faster one on average, 15 % at most).  Measured, us, wide /
// passes: 17 tokens of 1088 x 24000 46.8 / 24.6, 2048 x 28672 51.8 / 26.7, 4096 x 11008 24.3 /
// 16.5; 32 tokens of 1024 x 28672 52.7 / 32, 8192 x 28672 51.0 / 40.3; but 48 of 8192 x 28672 51.7 /
// 60, 32 of 4096 x 4096 13.2 / 15.3 and 17 of 28672 x 8192 30.6 / 33.3.
bool packed_passes(int64_t N, int64_t m, int64_t n) {
  const int64_t KT = ceil_div(n, kWk), rest = N % 16;
  const int64_t wide = 6500 + KT * std::min(wide_ns(N, m, true), wide_ns(N, m, false)) * 7 / 2;
  const int64_t pass = 5500 + 80 * KT + m * n / 32000;
  // the last pass transforms X itself, if it is of up to four tokens
  return N / 16 * pass + (rest == 0 ? 0 : rest <= 2 ? pass * 7 / 10 : rest <= 4 ? pass * 17 / 20 : pass) < wide;
}

hipError_t launch_packed_wide(const PackedWidePlan &p, const uint8_t *packed, int64_t m, int64_t n, const char *ws, int Nc,
                              void *Y, bool y_bf16, hipStream_t st) {
  const int64_t tt = ceil_div(Nc, 64);
  const bool four = wide_ns(Nc, m, true) <= wide_ns(Nc, m, false);
  const int tiles_m = (int)ceil_div(m, four ? 128 : 64);
  auto k = four ? (y_bf16 ? k_packed_wide<4, true> : k_packed_wide<4, false>)
                : (y_bf16 ? k_packed_wide<2, true> : k_packed_wide<2, false>);
  k<<<(unsigned)(tiles_m * tt), 256, 0, st>>>(packed, m, n, p.KT, (const uint16_t *)ws, tiles_m, (int)tt,
                                              (const float *)(ws + p.sp), p.parts, p.T, Nc, Y);
  return hipGetLastError();
}

}  // namespace lcvq
