// HIP backward of the PBB (and SWA) prefill attention on gfx950: gradients of q, k, v for
// training (the paper's fused kernel includes backward propagation, Sec. 3; its grouped backward
// sums the gradients of the query heads that share a KV head, Appendix F.4).
//
// For target t with support A(t), p_s = exp(z_s - lse_t), z_s = scale q_t.k_s (Eq.(attention);
// lse_t the forward's log-partition, Appendix A.4 Eq.(lse)) and upstream gradient g_t:
//   dv_s += p_s g_t
//   ds_s  = p_s (g_t.v_s - delta_t),   delta_t = g_t.o_t
//   dq_t  = scale sum_s ds_s k_s,      dk_s += scale ds_s q_t
// summed over the query heads of each KV head for dk and dv.  Two launches:
//   dq:    the prefill kernel's structure (128 query columns per workgroup, two 16-column
//          groups per wave, walk their key interval in 32-key steps through LDS), no running
//          maximum (lse is known); each column also computes its delta and lse * log2(e) and
//          writes lse * log2(e) and -delta to the workspace for the second launch (both
//          launches start the dout.v accumulators at -delta, so the MFMA yields dp - delta);
//   dk/dv: transposed roles: each workgroup holds 64 keys of one KV head in registers and
//          walks, for every query head of the group, the interval of targets whose supports
//          contain those keys (PBB: up to h(floor(s/h) + 2) - 1; SWA: s + W - 1).
// A wave computes only the steps that its own columns or keys need.
// Every gradient element is written once, by the one workgroup that owns it (no atomics,
// deterministic).  Matrix-core products use v_mfma_f32_16x16x32_bf16 with the score layout of
// the forward (16 B-operand columns, 32 rows in two halves), P and dS rounded to bf16 as
// operands, fp32 accumulation, bf16 (RNE) outputs.
//
// Bound.  Paper's shape (12/2 heads, d 64, B 128, n 65536): dq moves 446 MB in 94 us (4.7 TB/s,
// near a copy's rate), dk/dv 275 MB in 66 us; FastDiv index arithmetic, 16-byte stores, steps
// skipped per wave and scalar-stepped tile addresses took them from 105 and 72 us.  c3's heads
// (n 16384, batch 4): 2.07 and 3.32 ms (1150 and 950 TFLOP/s of the 6 d and 8 d operations per pair
// that each computes), bound by each wave's serial step at two waves per SIMD (matrix cores busy
// 0.57 and 0.48) while the card's power limit holds the clock near 2.0 GHz: dropping the transposed
// reads or the exponentials from a copy of the kernel changed its time by 1 to 3 %.
// 32x32x16 products measured 5 % slower for dq there, and for dk/dv (32 keys per wave) 96 against
// 72 us at d = 64 and twice as slow at d = 128 (one wave per SIMD, accumulators copied between
// register files every step).

#include <type_traits>

#include "pbb_device.h"
#include "pbb_internal.h"

namespace pbb {
namespace {

// Waves per workgroup of the dq and dk/dv launches (16 kDqColGroups query columns or 16 keys per
// wave).
constexpr int kDqWaves = 4;
constexpr int kDqColGroups = 2;   // 16-column groups per dq wave
constexpr int kDkdvWaves = 4;
constexpr int kDkdvWavesPerEU = 2; // occupancy the dk/dv register budget is set for

// ------------------------------------------------------------------------------------------
// dq: 128 query columns (TQ positions x G heads, position-major) per workgroup, 32 per wave in two
// groups of 16, which share every K and V read of a step.
template <int D>
__global__ __launch_bounds__(kDqWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
void bwd_dq_kernel(BackwardArgs a, TilePlan pl) {
  constexpr int NW = kDqWaves, QC = kDqColGroups;
  constexpr int KK = D / 32, NB = D / 16, ROWB = D * 2;
  constexpr int HALF = 16 * ROWB;
  constexpr int TILE = 2 * HALF;
  constexpr int BUF = 2 * TILE;          // K tile, V tile
  constexpr int STAGES = 3;
  constexpr int OPS = D / 32;            // DMA instructions of a wave per step
  static_assert(NW == 4, "one (tensor, 16-row half) of a step per wave");
  __shared__ __align__(1024) unsigned char smem[STAGES * BUF];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, j4 = lane >> 4;
  const int G = a.group, n = a.n;
  auto support_lo = [&](int t) -> int { return pl.support_lo(t, a.block, a.window); };
  int bg, tile;
  pl.locate((int)blockIdx.x, (int)gridDim.x, bg, tile);
  if (tile < 0) return;
  const int b = pl.by_hkv.div(bg);
  const int g = bg - b * a.hkv;
  const int t0 = tile * pl.tq;
  const int t_last = min(n - 1, t0 + pl.tq - 1);
  const int s_first = support_lo(t0) >> 5;
  const int nsteps = (t_last >> 5) - s_first + 1;

  const uint32_t rowstride = (uint32_t)a.hkv * ROWB;
  const unsigned char* kbase = (const unsigned char*)a.k + ((size_t)b * n * a.hkv + g) * ROWB;
  const unsigned char* vbase = (const unsigned char*)a.v + ((size_t)b * n * a.hkv + g) * ROWB;

  // This lane's query columns: column col -> position t0 + col / G, head g*G + col % G.  Columns
  // past the tile's positions repeat its last position and are never stored.
  const size_t row0 = ((size_t)b * n + t0) * a.hq + (size_t)g * G;   // row of (t0, head g*G)
  struct Column {
    int cp, head;   // position within the tile (the last one for columns past it), query head
    bool valid;
  };
  auto column = [&](int qc, int c) -> Column {
    const int col = (wave * QC + qc) * 16 + c;
    const int cp = pl.by_group.div(col);
    const int cu = min(cp, t_last - t0);
    return Column{cu, col - cp * G, cp == cu};
  };
  auto row_offset = [&](const Column& x) { return (uint32_t)(x.cp * a.hq + x.head) * (uint32_t)ROWB; };
  int tcol[QC], lo_c[QC];
  float lse2[QC], ndl[QC];  // lse * log2(e) and -delta of each column
  bf16x8 qB[QC][KK], gB[QC][KK];

  // DMA of a step: wave w loads 16 rows (half w & 1) of K (w < 2) or V; rows past t_last read row
  // t_last instead (masked, and inside the tensor).
  const int wrow = s_first * 32 + 16 * (wave & 1);
  const unsigned char* src = (wave >= 2 ? vbase : kbase) + (size_t)wrow * rowstride;
  int left = t_last - wrow;
  uint32_t doff[kDmaBlocks<D>];
  dma_offsets<D>(lane, rowstride, doff);
  auto issue = [&](int stage) {   // the next step
    dma_rows16<D>(src, left, rowstride, doff, smem + stage * BUF + wave * HALF);
    src += (size_t)rowstride * 32;
    left -= 32;
  };

  // delta = dout . out of each column (the four quarters j hold channel slices 8j.. of every
  // 32-channel block), and lse * log2(e): -delta and lse * log2(e) are kept in registers for dq
  // and written to the workspace for the dk/dv launch.
  {
    bf16x8 oB[QC][KK];
    float l[QC];
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      const Column x = column(qc, c16);
      tcol[qc] = t0 + x.cp;
      lo_c[qc] = support_lo(tcol[qc]);
      const uint32_t off = row_offset(x) + 16 * j4;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        gB[qc][kk] = *(const bf16x8*)((const unsigned char*)a.dout + row0 * ROWB + (off + 64u * kk));
        oB[qc][kk] = *(const bf16x8*)((const unsigned char*)a.out + row0 * ROWB + (off + 64u * kk));
      }
      l[qc] = a.lse[((size_t)b * a.hq + (size_t)(g * G + x.head)) * n + tcol[qc]];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        qB[qc][kk] = *(const bf16x8*)((const unsigned char*)a.q + row0 * ROWB + (off + 64u * kk));
    }
    issue(0);
    if (nsteps > 1) issue(1);
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      const Column x = column(qc, c16);
      float part = 0.0f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          part = __builtin_fmaf((float)gB[qc][kk][e], (float)oB[qc][kk][e], part);
      lse2[qc] = l[qc] * 1.4426950408889634f;
      ndl[qc] = -sum_xor16_32(part);
      if (x.valid && j4 == 0) {
        float* w = a.ws + ((size_t)b * a.hq + (size_t)(g * G + x.head)) * 2 * n + tcol[qc];
        w[0] = lse2[qc];
        w[n] = ndl[qc];
      }
    }
    // the queries have landed
#pragma unroll
    for (int qc = 0; qc < QC; ++qc)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qB[qc][kk]));
  }

  // LDS byte addresses in stage 0 (tile_addresses), the V tile TILE further on.
  uint32_t ra[2], ka[4];
  {
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    tile_addresses<D>(base, c16, j4, ra, ka);
  }
  const __attribute__((address_space(3))) unsigned char* lds0 = nullptr;

  // The wave's own range of steps [wlo, whi], and the run [ua, ub) of them that needs no mask.
  const int tw_lo = t0 + pl.by_group.div(wave * 16 * QC);
  const int tw_hi = min(t0 + pl.by_group.div(wave * 16 * QC + 16 * QC - 1), t_last);
  const int wlo = tw_lo <= t_last ? (support_lo(tw_lo) >> 5) - s_first : nsteps;
  const int whi = (tw_hi >> 5) - s_first;
  const int ua = ((support_lo(tw_hi) + 31) >> 5) - s_first;
  const int ub = ((tw_lo + 1) >> 5) - s_first;

  f32x4 acc[QC][NB];
#pragma unroll
  for (int qc = 0; qc < QC; ++qc)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[qc][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const float c = a.scale_log2;
  int rstage = 0;

  auto begin_step = [&](int st) -> uint32_t {
    wait_groups<STAGES - 2, OPS>(nsteps - 1 - st);
    lds_barrier();
    if (st + STAGES - 1 < nsteps) issue(rstage == 0 ? STAGES - 1 : rstage - 1);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t sb = (uint32_t)(rstage * BUF);
    rstage = rstage == STAGES - 1 ? 0 : rstage + 1;
    return sb;
  };

  // One step, masked or not: each its own loop below.
  auto step = [&](int st, uint32_t sb, auto masked) {
    f32x4 s0[QC], s1[QC], d0[QC], d1[QC];
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      s0[qc] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      s1[qc] = s0[qc];
      d0[qc] = f32x4{ndl[qc], ndl[qc], ndl[qc], ndl[qc]};  // the products land on -delta
      d1[qc] = d0[qc];
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const auto* p = lds0 + ra[kk & 1] + sb + kTileLine * (kk >> 1);
      const bf16x8 k0 = *(const __attribute__((address_space(3))) bf16x8*)(p);
      const bf16x8 k1 = *(const __attribute__((address_space(3))) bf16x8*)(p + HALF);
      const bf16x8 v0 = *(const __attribute__((address_space(3))) bf16x8*)(p + TILE);
      const bf16x8 v1 = *(const __attribute__((address_space(3))) bf16x8*)(p + TILE + HALF);
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) {
        s0[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qB[qc][kk], s0[qc], 0, 0, 0);
        s1[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qB[qc][kk], s1[qc], 0, 0, 0);
        d0[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v0, gB[qc][kk], d0[qc], 0, 0, 0);
        d1[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v1, gB[qc][kk], d1[qc], 0, 0, 0);
      }
    }
    // The K^T reads for dq go out now, under the softmax arithmetic.
    u32x2 kr[2 * NB];
    read_chunks<D, 0>(kr, ka, sb);
    // ds = p (dp - delta) (the accumulators started at -delta), p = exp2(s c - lse2).  Masked keys
    // get p = 0 whatever the target's log-partition is (their exponent is replaced).  Element e of
    // s0 is key k0 + 4 j4 + e, of s1 key k0 + 16 + 4 j4 + e.
    const int k0 = (s_first + st) * 32 + 4 * j4;
    bf16x8 dsB[QC];
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      const int lo = lo_c[qc] - k0, up = tcol[qc] - k0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dp = e < 4 ? d0[qc][e] : d1[qc][e - 4];
        float x = __builtin_fmaf(e < 4 ? s0[qc][e] : s1[qc][e - 4], c, -lse2[qc]);
        if constexpr (decltype(masked)::value) {
          const int t = e < 4 ? e : 12 + e;
          x = t >= lo && t <= up ? x : kNegInf;
        }
        dsB[qc][e] = (__bf16)(fast_exp2(x) * dp);
      }
    }
    // dq^T += K^T ds^T.
    wait_chunks<D>(kr);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const bf16x8 kt = join_chunks(kr[2 * nb], kr[2 * nb + 1]);
#pragma unroll
      for (int qc = 0; qc < QC; ++qc)
        acc[qc][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt, dsB[qc], acc[qc][nb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const int m1 = min(max(ua, wlo), whi + 1);   // [m1, m2): no masks
  const int m2 = min(max(ub, m1), whi + 1);
  int st = 0;
  for (; st < wlo; ++st) begin_step(st);
  for (; st < m1; ++st) {
    const uint32_t sb = begin_step(st);
    step(st, sb, std::true_type{});
  }
  for (; st < m2; ++st) {
    const uint32_t sb = begin_step(st);
    step(st, sb, std::false_type{});
  }
  for (; st <= whi; ++st) {
    const uint32_t sb = begin_step(st);
    step(st, sb, std::true_type{});
  }
  for (; st < nsteps; ++st) begin_step(st);

  // (The columns are worked out again: kept across the key loop, they would cost registers.)
  int ce = c16;
  asm("" : "+v"(ce));
#pragma unroll
  for (int qc = 0; qc < QC; ++qc) {
    u32x4 w[NB / 2];
#pragma unroll
    for (int q = 0; q < NB / 2; ++q) w[q] = pair_blocks(acc[qc][2 * q], acc[qc][2 * q + 1], a.scale);
    const Column x = column(qc, ce);
    if (x.valid) {
      unsigned char* drow = (unsigned char*)a.dq + row0 * ROWB + row_offset(x);
#pragma unroll
      for (int q = 0; q < NB / 2; ++q)
        *(u32x4*)(drow + 64 * q + 32 * (j4 & 1) + 16 * (j4 >> 1)) = w[q];
    }
  }
}

// ------------------------------------------------------------------------------------------
// dk, dv: 64 keys of one KV head per workgroup, 16 per wave, held as matrix-core B operands; the
// workgroup walks, for each query head of the group in turn, the 32-target steps of the targets
// whose supports contain its keys, through LDS: Q and dout rows and the steps' lse * log2(e) and
// -delta values.
template <int D>
__global__ __launch_bounds__(kDkdvWaves * 64)
__attribute__((amdgpu_waves_per_eu(kDkdvWavesPerEU)))
void bwd_dkdv_kernel(BackwardArgs a, DkdvPlan pl) {
  constexpr int NW = kDkdvWaves;
  constexpr int KK = D / 32, NB = D / 16, ROWB = D * 2;
  constexpr int HALF = 16 * ROWB;
  constexpr int TILE = 2 * HALF;
  constexpr int BUF = 2 * TILE + 256;   // Q tile, dout tile, lse2[32] and -delta[32]
  constexpr int STAGES = 4;             // two stages of two target steps each
  constexpr int KT = 16 * NW;           // keys per workgroup
  static_assert(NW == 4, "one (tensor, 16-row half) of a step per wave");
  __shared__ __align__(1024) unsigned char smem[STAGES * BUF];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, j4 = lane >> 4;
  const int G = a.group, n = a.n;
  auto last_target = [&](int s) -> int { return pl.last_target(s, a.block, a.window); };
  int bg, tile;
  pl.locate((int)blockIdx.x, (int)gridDim.x, bg, tile);
  const int b = pl.by_hkv.div(bg), g = bg - b * a.hkv;
  const int s0k = tile * KT;                       // first key of the workgroup
  const int s1k = min(n - 1, s0k + KT - 1);        // last key
  const int q_end = min(n - 1, last_target(s1k));  // targets before s0k see none of these keys
  const int qsteps = ((q_end - s0k) >> 5) + 1;
  const int nsteps = G * qsteps;                   // (head, target step) pairs

  // This wave's keys (keys past the prompt repeat its last one and are never stored).  Of each
  // head's target steps it computes [jlo, jhi], those with a target that sees one of its keys;
  // [ja, jb) of them need no mask: every target comes at or after the wave's last key and at or
  // before the last target of its first (the supports are intervals ending at the target).
  const int kw = min(s0k + 16 * wave, n - 1);
  const int key = min(s0k + 16 * wave + c16, n - 1);
  const bool valid = s0k + 16 * wave + c16 < n;
  const int t_hi = min(q_end, last_target(key));
  const int jlo = (kw - s0k) >> 5;
  const int jhi = s0k + 16 * wave < n
                      ? (min(q_end, last_target(min(kw + 15, n - 1))) - s0k) >> 5 : -1;
  const int ja = (kw + 15 - s0k + 31) >> 5;
  const int jb = (min(q_end, last_target(kw)) - s0k + 1) >> 5;
  const size_t krow = (((size_t)b * n + kw) * a.hkv + g) * ROWB;   // row of the wave's first key
  const uint32_t koff = (uint32_t)(key - kw) * (uint32_t)(a.hkv * ROWB);
  bf16x8 kB[KK], vB[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const uint32_t o = koff + (uint32_t)(64 * kk + 16 * j4);
    kB[kk] = *(const bf16x8*)((const unsigned char*)a.k + krow + o);
    vB[kk] = *(const bf16x8*)((const unsigned char*)a.v + krow + o);
  }

  // DMA of a (head, target step): wave w loads 16 rows (half w & 1) of Q (w < 2) or dout; rows
  // past q_end read row q_end instead (masked).  Wave 0 also loads lse2 (lanes 0..31) and -delta
  // (lanes 32..63) of the same targets.
  const uint32_t qrowstride = (uint32_t)a.hq * ROWB;
  const int wrow = s0k + 16 * (wave & 1);
  const unsigned char* head0 = (const unsigned char*)(wave >= 2 ? a.dout : a.q) +
                               (((size_t)b * n + wrow) * a.hq + (size_t)g * G) * ROWB;
  const int jl = lane & 31;
  const float* whead0 = a.ws + ((size_t)b * a.hq + (size_t)g * G) * 2 * n + s0k;
  uint32_t doff[kDmaBlocks<D>];
  dma_offsets<D>(lane, qrowstride, doff);
  const unsigned char* src = head0;   // rows of the next (head, step) to load
  const float* wsrc = whead0;
  int left = q_end - wrow, ij = 0;
  auto issue_next = [&](int stage) {
    unsigned char* tp = smem + stage * BUF;
    dma_rows16<D>(src, left, qrowstride, doff, tp + wave * HALF);
    if (wave == 0)   // left: targets after the step's first (its row 0 is this wave's)
      __builtin_amdgcn_global_load_lds((const void*)(wsrc + min(jl, left) + (size_t)(lane >> 5) * n),
                                       (__attribute__((address_space(3))) void*)(tp + 2 * TILE),
                                       4, 0, 0);
    src += (size_t)qrowstride * 32;
    wsrc += 32;
    left -= 32;
    if (++ij == qsteps) {   // the next head
      ij = 0;
      head0 += ROWB;
      whead0 += 2 * (size_t)n;
      src = head0;
      wsrc = whead0;
      left = q_end - wrow;
    }
  };
  issue_next(0);
  if (nsteps > 1) issue_next(1);

  // LDS byte addresses in stage 0 (tile_addresses), the dout tile TILE further on; lse2 and -delta
  // of rows 4j4 .. +3 at la and la + 128, of rows 16 + 4j4 .. +3 64 further on.
  uint32_t ra[2], ta[4];
  const uint32_t lds_base =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  tile_addresses<D>(lds_base, c16, j4, ra, ta);
  const uint32_t la = lds_base + 2 * TILE + 16 * j4;
  const __attribute__((address_space(3))) unsigned char* lds0 = nullptr;
  typedef const __attribute__((address_space(3))) bf16x8* lds_row;
  typedef const __attribute__((address_space(3))) f32x4* lds_f4;

  f32x4 acck[NB], accv[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    acck[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    accv[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  const float c = a.scale_log2;
  // the keys and values have landed
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(kB[kk]), "+v"(vB[kk]));

  // One target step, masked or not: each its own loop below (a branch around the mask inside one
  // loop cost 5 % at d = 128, two copies joined in one loop 25 % in register copies).
  auto step = [&](int jc, uint32_t sb, auto masked) {
    // Scores with targets on the rows (two halves of 16) and this wave's keys on the columns;
    // the dout.v products land on -delta of their target row.
    f32x4 s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = {0.0f, 0.0f, 0.0f, 0.0f};
    // The Q rows first; the dout rows travel under the score products, whose exponentials then run
    // beside the dout.v products.  The order is pinned: few waves per SIMD do not hide the waits that
    // the scheduler spreads between the products (3469 against 3585 us at c3's heads; the dout^T
    // reads pinned before the dout.v products as well 3814 us; the whole backward at d = 64, 12/2
    // heads, B 2048, n 2048 217.7 / 229.3, 16/1 heads, n 2000 503.9 / 531.3; with four waves per SIMD
    // no difference: the paper's shape 158.0 / 157.4).
    bf16x8 qa[KK], qb[KK], ga[KK], gb[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const auto* p = lds0 + ra[kk & 1] + sb + kTileLine * (kk >> 1);
      qa[kk] = *(lds_row)(p);
      qb[kk] = *(lds_row)(p + HALF);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    f32x4 d0 = *(lds_f4)(lds0 + la + sb + 128), d1 = *(lds_f4)(lds0 + la + sb + 192);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const auto* p = lds0 + ra[kk & 1] + sb + kTileLine * (kk >> 1) + TILE;
      ga[kk] = *(lds_row)(p);
      gb[kk] = *(lds_row)(p + HALF);
    }
    const f32x4 l0 = *(lds_f4)(lds0 + la + sb), l1 = *(lds_f4)(lds0 + la + sb + 64);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kk], kB[kk], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qb[kk], kB[kk], s1, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga[kk], vB[kk], d0, 0, 0, 0);
      d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gb[kk], vB[kk], d1, 0, 0, 0);
    }
    // The dout^T reads for dv go out now, under the softmax arithmetic.
    u32x2 gr[2 * NB];
    read_chunks<D, TILE>(gr, ta, sb);
    bf16x8 pB, dsB;
    // Pairs outside the support get p = 0 whatever their target's log-partition is: it is their
    // exponent that is replaced (a score of -inf would give NaN where the log-partition is NaN or
    // -inf).  Element e of s0 is target q0 + 4 j4 + e, of s1 target q0 + 16 + 4 j4 + e.
    const int q0 = s0k + 32 * jc + 4 * j4;
    const int lo = key - q0, up = t_hi - q0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = __builtin_fmaf(e < 4 ? s0[e] : s1[e - 4], c, -(e < 4 ? l0[e] : l1[e - 4]));
      if constexpr (decltype(masked)::value) {
        const int t = e < 4 ? e : 12 + e;
        x = t >= lo && t <= up ? x : kNegInf;
      }
      const float pe = fast_exp2(x);
      pB[e] = (__bf16)pe;
      dsB[e] = (__bf16)(pe * (e < 4 ? d0[e] : d1[e - 4]));
    }
    // dv^T += dout^T p, dk^T += Q^T ds: dout^T and Q^T by transposed reads.  The Q^T reads go out
    // before the dv products so that they overlap them.
    wait_chunks<D>(gr);
    u32x2 qr[2 * NB];
    read_chunks<D, 0>(qr, ta, sb);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      accv[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(join_chunks(gr[2 * nb], gr[2 * nb + 1]), pB,
                                                         accv[nb], 0, 0, 0);
    wait_chunks<D>(qr);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      acck[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(join_chunks(qr[2 * nb], qr[2 * nb + 1]), dsB,
                                                         acck[nb], 0, 0, 0);
  };

  // Target steps go in pairs (buffers 0-1 and 2-3): at the start of a pair this wave's loads of
  // both steps have landed; one barrier makes every wave's share visible and frees the other
  // pair's buffers (every wave has finished the previous pair), and the next pair is issued into
  // them -- one barrier per two steps (measured 2-4 % faster than one per step).
  int gs = 0;
  uint32_t sb = 0;   // stage offset of step gs
  auto begin_step = [&]() {
    if ((gs & 1) == 0) {
      __builtin_amdgcn_s_waitcnt(0x0F70);
      lds_barrier();
      const int ob = ((gs >> 1) & 1) ? 0 : 2;
      if (gs + 2 < nsteps) issue_next(ob);
      if (gs + 3 < nsteps) issue_next(ob + 1);
    }
    sb = (uint32_t)((((gs >> 1) & 1) * 2 + (gs & 1)) * BUF);
    ++gs;
    __builtin_amdgcn_sched_barrier(0);
  };
  const int j1 = min(max(ja, jlo), jhi + 1);
  const int j2 = min(max(jb, j1), jhi + 1);
  for (int hi = 0; hi < G; ++hi) {
    int j = 0;
    for (; j < jlo && j < qsteps; ++j) begin_step();
    for (; j < j1; ++j) {
      begin_step();
      step(j, sb, std::true_type{});
    }
    for (; j < j2; ++j) {
      begin_step();
      step(j, sb, std::false_type{});
    }
    for (; j <= jhi; ++j) {
      begin_step();
      step(j, sb, std::true_type{});
    }
    for (; j < qsteps; ++j) begin_step();
  }

  const uint32_t ooff = koff + (uint32_t)(32 * (j4 & 1) + 16 * (j4 >> 1));
#pragma unroll
  for (int q = 0; q < NB / 2; ++q) {
    const u32x4 wk = pair_blocks(acck[2 * q], acck[2 * q + 1], a.scale);
    const u32x4 wv = pair_blocks(accv[2 * q], accv[2 * q + 1], 1.0f);
    if (valid) {
      *(u32x4*)((unsigned char*)a.dk + krow + (ooff + 64u * q)) = wk;
      *(u32x4*)((unsigned char*)a.dv + krow + (ooff + 64u * q)) = wv;
    }
  }
}

// Where the dq launch takes the heaviest tiles first (the whole backward, by weight against in
// order, us): 32/8 heads, d 128, B 2048, n 4000 (1000 workgroups, 3 half-blocks after the first)
// 352 / 370, n 12000 (3000, 11) 1047 / 1028; B 512, n 8000 (2000, 31) 250 / 230.  16/1 heads, d 64,
// B 128, n 4000 (500, 62) 47.8 / 46.9; 12/2 heads, B 2708, n 7980 (760, 5) 341 / 360.
template <int D>
constexpr OrderLimits kDqByWeight = {D == 128 ? 2048 : 4096, D == 128 ? 24 : 32};

template <int D>
hipError_t launch_backward_d(const BackwardArgs& a, hipStream_t stream) {
  const TilePlan pl = TilePlan::make(a.batch, a.hkv, a.group, a.n, a.mode == kSupportPBB, a.block,
                                     a.window, 16 * kDqColGroups * kDqWaves / a.group,
                                     kDqByWeight<D>);
  hipLaunchKernelGGL((bwd_dq_kernel<D>), dim3((unsigned)((size_t)a.batch * a.hkv * pl.ranks())),
                     dim3(kDqWaves * 64), 0, stream, a, pl);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const DkdvPlan kp = DkdvPlan::make(a.hkv, a.n, a.mode == kSupportPBB, a.block, 16 * kDkdvWaves);
  hipLaunchKernelGGL((bwd_dkdv_kernel<D>), dim3((unsigned)((size_t)a.batch * a.hkv * kp.tiles)),
                     dim3(kDkdvWaves * 64), 0, stream, a, kp);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_backward_bf16(const BackwardArgs& a, int32_t head_dim, hipStream_t stream) {
  return head_dim == 128 ? launch_backward_d<128>(a, stream) : launch_backward_d<64>(a, stream);
}

}  // namespace pbb
