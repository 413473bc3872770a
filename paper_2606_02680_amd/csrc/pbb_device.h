// Device-side helpers shared by the HIP kernels of libpbb (decode and prefill).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pbb_index.h"

namespace pbb {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// Cache-policy operand of global_load_lds selecting the non-temporal ("nt") hint.
constexpr int kCachePolicyNT = 2;

constexpr float kNegInf = -__builtin_huge_valf();
// Largest sum of one lane's eight softmax weights of a column that a key step keeps without
// moving its reference: 2^8, so every weight stays <= 2^8, and a key whose score rises more
// than 8 log2 units above the reference (the usual dominant key of a peaked row) becomes the
// new reference and enters with weight exactly 1, unrounded.
constexpr float kWeightCap = 256.0f;

// float -> bf16 with round-to-nearest-even (inputs are finite).
__device__ __forceinline__ uint16_t float_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Rotary embedding of one channel pair at absolute position t: the angle in turns,
// t * turns_per_pos, is reduced to [0, 1) in fp64 (exact enough for any t < 2^31) and the
// hardware sine and cosine (which take turns) give cos and sin.
__device__ __forceinline__ void rope_cos_sin(int t, double turns_per_pos, float& cs, float& sn) {
  const double r = (double)t * turns_per_pos;
  const float f = (float)(r - __builtin_floor(r));
  cs = __builtin_amdgcn_cosf(f);
  sn = __builtin_amdgcn_sinf(f);
}

// (x, y) = channels (c, c + d/2) turned by the angle: (x cos - y sin, y cos + x sin), with the
// same fused operations wherever it is evaluated.
__device__ __forceinline__ void rope_turn(float x, float y, float cs, float sn, float& ox,
                                          float& oy) {
  ox = __builtin_fmaf(x, cs, -(y * sn));
  oy = __builtin_fmaf(y, cs, x * sn);
}

// Workgroup barrier that orders LDS reads and writes made by ordinary instructions, without
// waiting for LDS DMA still in flight (whose completion the caller tracks with vmcnt).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Waits until at most `ahead` groups (wave-uniform, at most N) of OPS vector-memory instructions
// each, the youngest ones, are outstanding.
template <int N, int OPS>
__device__ __forceinline__ void wait_groups(int ahead) {
  static_assert(N * OPS < 64, "vmcnt immediate");
  if constexpr (N == 0) {
    __builtin_amdgcn_s_waitcnt(0x0F70);
  } else {
    if (ahead >= N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N * OPS) & 15) | (((N * OPS) >> 4) << 14));
    else wait_groups<N - 1, OPS>(ahead);
  }
}

// First source a(t) of the support of target t: PBB (mode 0) max(0, h(floor(t/h) - 1)) with
// h = block/2 (Sec. 3 "Flash-PBB"), SWA max(0, t - window + 1) (Prop. 2).  Never decreases in t.
__device__ __forceinline__ int support_start(int mode, int block, int window, int t) {
  int lo;
  if (mode == 0) {
    const int h = block >> 1;
    lo = h * (t / h - 1);
  } else {
    lo = t - window + 1;
  }
  return lo > 0 ? lo : 0;
}

// Last target whose support contains source s (the largest t with support_start(t) <= s):
// PBB h(floor(s/h) + 2) - 1, SWA s + window - 1.
__device__ __forceinline__ int support_last_target(int mode, int block, int window, int s) {
  if (mode == 0) {
    const int h = block >> 1;
    return h * (s / h + 2) - 1;
  }
  return s + window - 1;
}

// Value of lane l ^ 16 and of lane l ^ 32 (gfx950 v_permlane16_swap / v_permlane32_swap with
// both operands x: one result is the lane's own value, the other its partner's), on the VALU
// instead of an LDS permute.
__device__ __forceinline__ float max_xor16_32(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ float sum_xor16_32(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Two floats as a bf16 pair (x in the low half), round to nearest even: one instruction.
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const bf16x2 v = {(__bf16)x, (__bf16)y};
  return __builtin_bit_cast(uint32_t, v);
}

// Two 16-channel output blocks of a 16-column tile (lane (c16, j4) holds channels 4 j4 .. +3 of
// column c16 in each), scaled and packed to bf16: the odd quarters of the first swap with the even
// quarters of the second, after which quarter j4 holds channels 8 (j4 / 2) .. +7 of block j4 mod 2.
__device__ __forceinline__ u32x4 pair_blocks(f32x4 x, f32x4 y, float scale) {
  const uint32_t x0 = pack_bf16(x[0] * scale, x[1] * scale), x1 = pack_bf16(x[2] * scale, x[3] * scale);
  const uint32_t y0 = pack_bf16(y[0] * scale, y[1] * scale), y1 = pack_bf16(y[2] * scale, y[3] * scale);
  const auto s0 = __builtin_amdgcn_permlane16_swap(x0, y0, false, false);
  const auto s1 = __builtin_amdgcn_permlane16_swap(x1, y1, false, false);
  return u32x4{(uint32_t)s0[0], (uint32_t)s1[0], (uint32_t)s0[1], (uint32_t)s1[1]};
}

// LDS tiles of the prefill and backward kernels.  A 32-row tile (rows of D bf16) is stored as
// [row / 8][128-byte line of the row][8 rows x 8 pieces of 16 bytes], one 1 KiB LDS DMA per block,
// which reads whole cache lines; tile_block is the byte offset of row group y and line z.  Piece p
// of a line of row r sits at slot 8 (r mod 8) + (p ^ tile_swz(r)).  Both reads of a tile are then
// free of bank conflicts (64 banks; a 16-byte read serves per cycle the 16 lanes that share lane
// bit 5 and the parity of lane bits 2..4, an 8-byte or transposed read the 32 lanes that share the
// parity of lane bits 3..5), and a read's address is a lane constant for its piece within the line
// (2 for row operands, 4 for transposed reads) plus an immediate.
template <int D>
__device__ __forceinline__ constexpr int tile_block(int y, int z) {
  return (y * (D / 64) + z) * 1024;
}
__device__ __forceinline__ constexpr int tile_swz(int r) { return r & 6; }

// One 16-byte LDS DMA (global_load_lds) from a wave-uniform base plus a 32-bit lane offset, so
// that the address is formed by the instruction (scalar base + vector offset) rather than by
// 64-bit vector arithmetic.
__device__ __forceinline__ void dma16(const unsigned char* base, uint32_t off, unsigned char* lds) {
  __builtin_amdgcn_global_load_lds((const void*)(base + off),
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// Transposed LDS read (gfx950 ds_read_b64_tr_b16) at addr + OFF.  Issued as inline asm: the
// compiler cannot tell these reads apart from the LDS DMA still in flight and would otherwise
// wait for every outstanding load before each of them.  The caller waits with an s_waitcnt
// that takes the results as operands, so that nothing reads them earlier.
template <int OFF>
__device__ __forceinline__ u32x2 tr_read(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS offset immediate");
  u32x2 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
  return r;
}

}  // namespace pbb
