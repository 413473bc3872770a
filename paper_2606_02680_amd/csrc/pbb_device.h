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

// LDS tiles of the prefill and backward kernels.  A 32-row tile (rows of D bf16) is stored in
// 1 KiB blocks, one LDS DMA each, that hold whole rows (so that the DMA reads them contiguously):
// 4 rows as [128-byte line][row][8 pieces of 16 bytes] at d = 128, 8 rows as [row][8 pieces] at
// d = 64.  Piece p of a line of row r sits in slot p ^ tile_swz(r) of its eight.  Both reads of a
// tile are then free of bank conflicts (64 banks; a 16-byte read serves per cycle the 16 lanes
// that share lane bit 5 and the parity of lane bits 2..4, an 8-byte or transposed read the 32
// lanes that share the parity of lane bits 3..5), and a read's address is a lane constant for its
// piece within the line (2 for row operands, 4 for transposed reads) plus an immediate, where a
// row-major tile with its swizzle across the row takes one address addition per read.
template <int D>
__device__ __forceinline__ constexpr int tile_row(int r) {
  return D == 128 ? (r >> 2) * 1024 + (r & 3) * 128 : r * 128;
}
constexpr int kTileLine = 512;   // from a row's first line to its second (d = 128)
__device__ __forceinline__ constexpr int tile_swz(int r) { return r & 6; }

// One 16-byte LDS DMA (global_load_lds) from a wave-uniform base plus a 32-bit lane offset, so
// that the address is formed by the instruction (scalar base + vector offset) rather than by
// 64-bit vector arithmetic.
__device__ __forceinline__ void dma16(const unsigned char* base, uint32_t off, unsigned char* lds) {
  __builtin_amdgcn_global_load_lds((const void*)(base + off),
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// DMA of 16 rows of a tensor into half a tile, 1 KiB per instruction.  dma_offsets: this lane's
// byte offsets from the first row (`stride` bytes between rows).  dma_rows16: the rows from the
// wave-uniform address p, of which `left` more than the first exist (negative: p itself lies past
// the last one); every 16-byte piece of the rows past it reads the last row's last piece, so that an
// infinity elsewhere in that row meets no weight of 0.  Callers step p along, so that a step's loads
// cost no multiplication: the scalar work of an issue stands in every wave's serial step (with a
// multiplication and a limit per block, some 40 more scalar instructions per step, the d = 128
// kernels of the backward were 2 to 3 % slower).
template <int D>
constexpr int kDmaBlocks = D / 64;   // blocks of 8 rows

template <int D>
__device__ __forceinline__ void dma_offsets(int lane, uint32_t stride, uint32_t (&off)[kDmaBlocks<D>]) {
#pragma unroll
  for (int y = 0; y < kDmaBlocks<D>; ++y) {
    const int r = D == 128 ? 4 * y + ((lane >> 3) & 3) : lane >> 3;
    const int line = D == 128 ? lane >> 5 : 0;
    off[y] = (uint32_t)r * stride + (uint32_t)(128 * line + (((lane & 7) ^ tile_swz(r)) << 4));
  }
}

template <int D>
__device__ __forceinline__ void dma_rows16(const unsigned char* p, int left, uint32_t stride,
                                           const uint32_t (&off)[kDmaBlocks<D>],
                                           unsigned char* lds) {
  constexpr int N = kDmaBlocks<D>;
  if (left >= 15) {
#pragma unroll
    for (int y = 0; y < 2 * N; ++y)
      dma16(y < N ? p : p + (size_t)stride * 8, off[y % N], lds + 1024 * y);
  } else {
#pragma unroll
    for (int y = 0; y < 2 * N; ++y) {
      const int r0 = y < N ? 0 : 8;   // first row of the block's eight
      const int last = min(left - r0, 7);   // the last one that exists
      const unsigned char* q = p + (int64_t)(r0 + min(last, 0)) * (int64_t)stride;
      const uint32_t lim = (uint32_t)max(last, 0) * stride + (uint32_t)(2 * D - 16);
      dma16(q, last < 0 ? lim : min(off[y % N], lim), lds + 1024 * y);
    }
  }
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

// This lane's LDS byte addresses in a 32-row tile at `base`, for 16x16 products.  Row operand of
// 32-channel slice kk (row c16, piece 4kk + j4): ra[kk mod 2] + kTileLine (kk / 2); rows 16..
// 32 D bytes further on.  Transposed reads of 16-channel chunk nb (row 4j4 + c16/4, channels
// 16nb + 4(c16 mod 4) .. +3): ta[nb mod 4] + kTileLine (nb / 4); rows 16.. 32 D bytes further on.
template <int D>
__device__ __forceinline__ void tile_addresses(uint32_t base, int c16, int j4, uint32_t (&ra)[2],
                                               uint32_t (&ta)[4]) {
#pragma unroll
  for (int x = 0; x < 2; ++x)
    ra[x] = base + tile_row<D>(c16) + (((4 * x + j4) ^ tile_swz(c16)) << 4);
  const int r = 4 * j4 + (c16 >> 2);
#pragma unroll
  for (int x = 0; x < 4; ++x)
    ta[x] = base + tile_row<D>(r) + (((2 * x + ((c16 & 3) >> 1)) ^ tile_swz(r)) << 4) +
            ((c16 & 1) << 3);
}

// The transposed operands of a 32-row tile at offset OFF: dst[2nb] holds rows 4j4 .. +3 and
// dst[2nb + 1] rows 16 + 4j4 .. +3 of channel 16nb + c16 (the row order of a 16x16 result pair's
// registers).  wait_chunks waits for every LDS read issued so far; its operands make uses follow.
template <int D, int OFF>
__device__ __forceinline__ void read_chunks(u32x2 (&dst)[D / 8], const uint32_t (&ta)[4], uint32_t sb) {
  constexpr int H = 32 * D;
  dst[0] = tr_read<OFF>(ta[0] + sb);
  dst[1] = tr_read<OFF + H>(ta[0] + sb);
  dst[2] = tr_read<OFF>(ta[1] + sb);
  dst[3] = tr_read<OFF + H>(ta[1] + sb);
  dst[4] = tr_read<OFF>(ta[2] + sb);
  dst[5] = tr_read<OFF + H>(ta[2] + sb);
  dst[6] = tr_read<OFF>(ta[3] + sb);
  dst[7] = tr_read<OFF + H>(ta[3] + sb);
  if constexpr (D == 128) {
    dst[8] = tr_read<OFF + kTileLine>(ta[0] + sb);
    dst[9] = tr_read<OFF + H + kTileLine>(ta[0] + sb);
    dst[10] = tr_read<OFF + kTileLine>(ta[1] + sb);
    dst[11] = tr_read<OFF + H + kTileLine>(ta[1] + sb);
    dst[12] = tr_read<OFF + kTileLine>(ta[2] + sb);
    dst[13] = tr_read<OFF + H + kTileLine>(ta[2] + sb);
    dst[14] = tr_read<OFF + kTileLine>(ta[3] + sb);
    dst[15] = tr_read<OFF + H + kTileLine>(ta[3] + sb);
  }
}

__device__ __forceinline__ bf16x8 join_chunks(u32x2 x, u32x2 y) {
  const u32x4 w = {x[0], x[1], y[0], y[1]};
  return __builtin_bit_cast(bf16x8, w);
}

template <int D>
__device__ __forceinline__ void wait_chunks(u32x2 (&v)[D / 8]) {
  if constexpr (D == 128)
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                   "+v"(v[6]), "+v"(v[7]), "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]),
                   "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15]));
  else
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                   "+v"(v[6]), "+v"(v[7]));
}

}  // namespace pbb
