// Device helpers of the kernels that issue matrix-core instructions from inline
// assembly (gfx950): the instruction itself, the wait states it needs, the codes
// conversion, explicit waits and the block-to-tile mapping.
#pragma once

#include "lcvq_common.hpp"

namespace lcvq {

constexpr int kTile = 256;   // block tile (M and N)
constexpr int kKStep = 64;   // K per main-loop step

// s_waitcnt with every counter at zero.
#define LCVQ_WAIT_ALL() __builtin_amdgcn_s_waitcnt(0)
// s_waitcnt vmcnt(N) lgkmcnt(0) (gfx9 encoding; expcnt left at its maximum).
#define LCVQ_WAIT_VM_LGKM0(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4))
// s_waitcnt vmcnt(N) only (lgkmcnt and expcnt left at their maximum).
#define LCVQ_WAIT_VM(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | (7 << 4) | (15 << 8))
// s_waitcnt lgkmcnt(0) only.
#define LCVQ_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4))
// Workgroup barrier without the release fence of __syncthreads() (which would
// drain the prefetch loads); the asm statements keep the compiler from moving
// memory operations across it.  LDS visibility is ensured by the waits above.
#define LCVQ_BARRIER()                   \
  do {                                   \
    asm volatile("" ::: "memory");       \
    __builtin_amdgcn_s_barrier();        \
    asm volatile("" ::: "memory");       \
  } while (0)

// Blocks are dispatched round-robin over the eight XCDs.  Give each XCD a
// contiguous run of tile ids, and walk tiles in bands of eight M-tiles, so the
// blocks sharing an XCD's L2 share operand tiles (with 256 tiles: 8 M-tiles x
// 4 token tiles per XCD, the fewest operand bytes per L2 for these products).  Any
// number of tiles is dealt out so, the first XCDs one more each: with runs only
// for whole multiples of eight, an XCD of any other grid held every eighth tile,
// one M-tile against many token tiles (5262 tokens of 6280 x 10136, forward 738 ->
// 486 us; 2404 of 22736 x 10056, input gradient 1516 -> 977).
__device__ __forceinline__ void tile_of_block(int tiles_m, int tiles_n, int &tm, int &tn) {
  const int per = (int)gridDim.x / 8, rem = (int)gridDim.x % 8;  // the first rem XCDs take one tile more
  const int xcd = (int)blockIdx.x % 8;
  const int id = xcd * per + min(xcd, rem) + (int)blockIdx.x / 8;
  constexpr int GM = 8;
  const int band = id / (GM * tiles_n);
  const int first = band * GM;
  const int gm = min(tiles_m - first, GM);
  const int in = id - band * GM * tiles_n;
  tm = first + in % gm;
  tn = in / gm;
}

// acc = A * B + acc, operands loaded (no VALU producer): issued in program order.
__device__ __forceinline__ void mfma16(floatx4 &acc, const bf16x8 &a, const bf16x8 &b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// The same with A produced by VALU instructions: the leading s_nop covers the
// VALU-write to matrix-core-read wait states.
__device__ __forceinline__ void mfma16_valu_a(floatx4 &acc, const bf16x8 &a, const bf16x8 &b) {
  asm volatile("s_nop 2\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Wait states between the zeroing of the accumulators (vector writes) and the
// first matrix-core read of them, R x C accumulators.  Each statement passes
// four accumulators through itself, so every zeroing write precedes the whole
// chain and every MFMA follows it: at least R C / 4 statements and a final
// s_nop 4 lie between a write and a read.
template <int R, int C>
__device__ __forceinline__ void acc_fence(floatx4 (&acc)[R][C]) {
  static_assert(C % 4 == 0, "four accumulators per statement");
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < C; j += 4) {
      if (i + 1 < R || j + 4 < C)
        asm volatile("s_nop 0" : "+a"(acc[i][j]), "+a"(acc[i][j + 1]), "+a"(acc[i][j + 2]), "+a"(acc[i][j + 3]));
      else
        asm volatile("s_nop 4" : "+a"(acc[i][j]), "+a"(acc[i][j + 1]), "+a"(acc[i][j + 2]), "+a"(acc[i][j + 3]));
    }
}
// Wait states between the last matrix-core write of an accumulator and the
// epilogue's vector reads of it.  The statement is a scheduling boundary with
// a memory clobber; the reads are copies the compiler places at their uses,
// which all lie in the epilogue after it.
__device__ __forceinline__ void mfma_drain() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// The codes conversion as ordered inline assembly: it stays where it is written
// (between two MFMAs of the previous operand), so the two MFMAs that follow it
// supply the wait states its consumer needs.
__device__ __forceinline__ bf16x8 nibbles_to_bf16x8_ordered(uint32_t w) {
  uint32_t p0, p1, p2, p3;
  asm volatile("v_cvt_scalef32_pk_bf16_fp4 %0, %1, 2.0" : "=v"(p0) : "v"(w));
  asm volatile("v_cvt_scalef32_pk_bf16_fp4 %0, %1, 2.0 op_sel:[1,0,0]" : "=v"(p1) : "v"(w));
  asm volatile("v_cvt_scalef32_pk_bf16_fp4 %0, %1, 2.0 op_sel:[0,1,0]" : "=v"(p2) : "v"(w));
  asm volatile("v_cvt_scalef32_pk_bf16_fp4 %0, %1, 2.0 op_sel:[1,1,0]" : "=v"(p3) : "v"(w));
  return __builtin_bit_cast(bf16x8, u32x4{p0, p1, p2, p3});
}

__device__ __forceinline__ float as_f(uint32_t u) { return __uint_as_float(u); }
// Copy a (uniform) value into a vector register.
__device__ __forceinline__ float to_vgpr(float x) {
  float v;
  asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
  return v;
}
__device__ __forceinline__ uint32_t as_u(float f) { return __float_as_uint(f); }

}  // namespace lcvq
