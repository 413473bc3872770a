// HIP prefill kernel for Post-Boundary Bridge (PBB) attention on gfx950 (MI355X, CDNA4).
//
// Every position t = 0..n-1 of a prompt attends with one softmax over its own support
// (Sec. 3, Eq.(pbb) and Eq.(attention)).  With h = B/2 that support is the interval
// [a(t), t], a(t) = max(0, h*(floor(t/h) - 1)) (Sec. 3 "Flash-PBB"; Appendix A.3): the causal
// block prefix plus, for the first h phases of a block, the preceding half-block, i.e. causal
// block tiles plus h x h bridge rectangles (Appendix F.4), never a dense n x n mask.  The
// sliding-window variant uses [max(0, t-W+1), t] (Prop. 2).  a(t) never decreases, so the
// keys any run of consecutive positions needs form one interval.
//
// Work unit: TQ = floor(128 / G) consecutive positions of one (sequence, KV head) with all G
// query heads of that KV head, i.e. up to 128 query columns ordered position-major, head-minor
// (native grouped-query attention: the K/V tile is read once for the group), 32 columns per wave
// in two groups of 16.  Keys of the unit's interval stream through LDS in 32-key steps, each tile
// loaded once per workgroup by LDS DMA and shared by the 4 waves.  Per step a wave computes
// S^T = K Q^T and O^T += V^T P^T on v_mfma_f32_16x16x32_bf16 exactly as the decode kernel does,
// the 16 B-operand columns being 16 queries; per-column bounds mask the tile, and a wave computes
// only the steps that its own columns need.  The online softmax keeps fp32 running references and
// sums (the log-sum-exp rescaling of Appendix A.4, Eq.(lse)).  Outputs are rounded to bf16 (RNE);
// the log-partition is written in natural-log units.  Finally every workgroup copies those of its
// positions that fall in the last `slots` positions of the prompt into the ring (slot s mod slots,
// Appendix F.1), the state decode continues from.
//
// LDS tiles: tile_row() and tile_swz() in pbb_device.h.
//
// Bound: instruction issue (matrix and vector work of a SIMD overlap only in part; at c3's heads
// the matrix cores draw the card's power limit as well).  What a tile costs beside its key steps
// counts at d = 64 and small blocks, where it walks 3 to 5 of them: index arithmetic by FastDiv
// instead of divisions, packed conversions and 16-byte stores in the epilogue, steps skipped per
// wave, scalar-stepped tile addresses and LDS addresses that are two or four lane constants plus
// immediates took the paper's shape (12/2 heads, d 64, B 128, n 65536; 238 MB) from 74.1 to 61.4
// us (3.9 TB/s) and c3's heads (n 16384, batch 4) from 1529 to 1485 us (1065 TFLOP/s), loops of
// their own for masked and unmasked steps (long walks only) another 1 to 2 % there.  32x32x16 matrix instructions
// (32 columns at once, a fifth fewer vector instructions) measured 1574 against 1485 us and 62.0
// against 61.4.

#include <type_traits>

#include "pbb_device.h"
#include "pbb_internal.h"

namespace pbb {
namespace {

// Waves per workgroup and 16-column groups per wave.  Measured with the present kernel: one group
// per wave 1.4x slower at c3's heads, n 8192 (twice the LDS bytes per product); 8 waves of two
// groups 11 % slower there and 2 % at the paper's shape (every barrier holds twice the waves).
constexpr int kPrefillWaves = 4;
constexpr int kPrefillGroups = 2;
constexpr int kPrefillCols = 16 * kPrefillGroups * kPrefillWaves;
// LDS stages and the occupancy the register budget is set for (waves per SIMD = workgroups per
// CU): three at d = 128 (168 VGPRs and, with loops apart, 12 bytes of scratch that the last masked
// steps use, 48 KiB of LDS), four at d = 64 (128 VGPRs, 32 KiB).  Five stages at d = 64 (three workgroups per CU) take 9.2
// against 7.8 us at 12/2 heads, B 128, n 2048, 56.5 / 55.4 at n 65536, and the same at large blocks.
constexpr int kPrefillStages128 = 3, kPrefillOcc128 = 3;
constexpr int kPrefillStages64 = 4, kPrefillOcc64 = 4;
// Starting reference of the running maximum (log2 units): finite and below any score.
constexpr float kNoScore = -1.0e30f;

// LOOPS: masked and unmasked steps in loops of their own (kPrefillLoopKeys).
template <int D, int ST, int OCC, bool LOOPS>
__global__ __launch_bounds__(kPrefillWaves * 64) __attribute__((amdgpu_waves_per_eu(OCC)))
void prefill_bf16_kernel(PrefillArgs a, TilePlan pl) {
  constexpr int NW = kPrefillWaves;
  constexpr int QC = kPrefillGroups;
  constexpr int KK = D / 32;            // 32-channel slices of the score contraction
  constexpr int NB = D / 16;            // 16-channel blocks of the output
  constexpr int ROWB = D * 2;           // bytes of one K or V row
  constexpr int PPR = D / 8;            // 16-byte pieces per row
  constexpr int HALF = 16 * ROWB;       // 16 rows of a tile
  constexpr int TILE = 2 * HALF;
  constexpr int BUF = 2 * TILE;         // K tile, then V tile
  constexpr int STAGES = ST;
  static_assert(STAGES >= 3, "stages");
  static_assert(NW == 4, "one (tensor, 16-row half) of a step per wave");
  __shared__ __align__(1024) unsigned char smem[STAGES * BUF];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15;
  const int j4 = lane >> 4;
  const int G = a.group;
  const int n = a.n;

  // First source of the support of target t.
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

  const uint32_t rowstride = (uint32_t)a.hkv * ROWB;  // bytes between consecutive positions
  const unsigned char* kbase = (const unsigned char*)a.k + ((size_t)b * n * a.hkv + g) * ROWB;
  const unsigned char* vbase = (const unsigned char*)a.v + ((size_t)b * n * a.hkv + g) * ROWB;

  // This lane's query columns: column col -> position t0 + col / G, head g*G + col % G.  Columns
  // past the tile's positions get zero queries and see no key of a masked step (tcol -1); they
  // load the last position's row, and nothing of them is stored.
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
  bf16x8 qB[QC][KK];
#pragma unroll
  for (int qc = 0; qc < QC; ++qc) {
    const Column x = column(qc, c16);
    tcol[qc] = x.valid ? t0 + x.cp : -1;
    lo_c[qc] = support_lo(t0 + x.cp);
    const uint32_t off = row_offset(x) + 16 * j4;
    const unsigned char* qbase = (const unsigned char*)a.q + row0 * ROWB;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qB[qc][kk] = *(const bf16x8*)(qbase + (off + 64u * kk));
  }

  // DMA of a step: wave w loads 16 rows (half w & 1) of K (w < 2) or V.  In the last step, rows
  // past t_last read row t_last instead (inside the tensor; masked for every column).
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

  // Steps 0 .. STAGES-2 go out first; step st then issues step st + STAGES - 1.
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nsteps) issue(s);

  // LDS byte addresses of this lane's reads in stage 0 (tile_addresses; the V tile is TILE on).
  uint32_t ra[2], va[4];
  {
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    tile_addresses<D>(base, c16, j4, ra, va);
  }
  const __attribute__((address_space(3))) unsigned char* lds0 = nullptr;

  // The wave's own range of steps [wlo, whi] (its columns' positions tw_lo .. tw_hi), and the
  // run [ua, ub) of them whose keys all lie in every column's support (a(t) never decreases).
  // `cut`: the wave holds columns past the tile's positions.
  const int tw_lo = t0 + pl.by_group.div(wave * 16 * QC);
  const int tw_end = t0 + pl.by_group.div(wave * 16 * QC + 16 * QC - 1);
  const bool cut = tw_end > t_last;
  const int tw_hi = min(tw_end, t_last);
  const int a_hi = support_lo(tw_hi);
  const int wlo = tw_lo <= t_last ? (support_lo(tw_lo) >> 5) - s_first : nsteps;
  const int whi = (tw_hi >> 5) - s_first;
  const int ua = ((a_hi + 31) >> 5) - s_first;
  const int ub = ((tw_lo + 1) >> 5) - s_first;

  // m starts at a finite floor below any score, so that a column whose keys are all masked so
  // far gets exp2(-inf - m) = 0 without a separate test; its first real maximum always moves m.
  float m[QC], lsum[QC];
  f32x4 acc[QC][NB];
#pragma unroll
  for (int qc = 0; qc < QC; ++qc) {
    m[qc] = kNoScore;
    lsum[qc] = 0.0f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[qc][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  const float sc = a.scale_log2;
  // the queries have landed (the key steps issued after them may still be in flight)
#pragma unroll
  for (int qc = 0; qc < QC; ++qc)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qB[qc][kk]));
  // Columns past the tile's positions score 0 and, in masked steps, -inf: with the reference at its
  // floor they vote for one move of the wave's references, in the tile's first step that no
  // position masks, and with reference 0 (tiles without such a step) for none.  So what they do to
  // the rounding of the wave's other columns depends on no query.
  if (cut) {
    const float m0 = ua < ((t0 + 1) >> 5) - s_first ? kNoScore : 0.0f;
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      m[qc] = tcol[qc] >= 0 ? kNoScore : m0;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        qB[qc][kk] = __builtin_bit_cast(
            bf16x8, tcol[qc] >= 0 ? __builtin_bit_cast(u32x4, qB[qc][kk]) : u32x4{0u, 0u, 0u, 0u});
    }
  }

  int rstage = 0;
  constexpr int OPS = D / 32;           // DMA instructions of a wave per step

  // Begins step st: its tiles have landed; returns the stage offset.
  auto begin_step = [&](int st) -> uint32_t {
    // This wave's loads of step st have landed once at most the loads of the steps issued
    // after it (up to STAGES - 2) are outstanding; the barrier then covers every wave's loads,
    // and every wave is done with step st-1, whose stage the loads of step st+STAGES-1 reuse.
    wait_groups<STAGES - 2, OPS>(min(STAGES - 2, nsteps - 1 - st));
    lds_barrier();
    if (st + STAGES - 1 < nsteps)
      issue(rstage == 0 ? STAGES - 1 : rstage - 1);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t sb = (uint32_t)(rstage * BUF);
    rstage = rstage == STAGES - 1 ? 0 : rstage + 1;
    return sb;
  };

  // One step, masked or not: with LOOPS by the loop that it stands in, else by a branch.
  auto step = [&](int st, uint32_t sb, auto masked) {
    f32x4 s0[QC], s1[QC];
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) {
      s0[qc] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      s1[qc] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const auto* kp = lds0 + ra[kk & 1] + sb + kTileLine * (kk >> 1);
      const bf16x8 ka = *(const __attribute__((address_space(3))) bf16x8*)(kp);
      const bf16x8 kb = *(const __attribute__((address_space(3))) bf16x8*)(kp + HALF);
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) {
        s0[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qB[qc][kk], s0[qc], 0, 0, 0);
        s1[qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb, qB[qc][kk], s1[qc], 0, 0, 0);
      }
    }
    // Element e of s0 is key k0 + 4 j4 + e of the lane's column, of s1 key k0 + 16 + 4 j4 + e.
    if (LOOPS ? decltype(masked)::value : st < ua || st >= ub) {
      const int k0 = (s_first + st) * 32 + 4 * j4;
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) {
        const int lo = lo_c[qc] - k0, up = tcol[qc] - k0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s0[qc][e] = e >= lo && e <= up ? s0[qc][e] : kNegInf;
          s1[qc][e] = 16 + e >= lo && 16 + e <= up ? s1[qc][e] : kNegInf;
        }
      }
    }
    // Online softmax in log2 units with a lazily moved reference m (the log-sum-exp rescaling
    // of Eq.(lse)): the weights are taken against the current m, and m moves to the column
    // maxima (the accumulators rescaled, the weights taken again) only in a step where the
    // eight weights of some lane and column sum above 2^8 or to infinity: a column's first
    // step with a real score (m starts at a finite floor), any step in which a score rises
    // more than 8 log2 units above m, and steps where several rise more than 5.  No other step
    // computes a maximum.  The result is the same softmax (numerator and denominator share
    // every reference change), and the weights that enter the sums and products stay <= 2^8.
    bf16x8 pB[QC];
    float ps[QC];
    auto weights = [&]() {
      bool over = false;
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) {
        float sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float pe =
              fast_exp2(__builtin_fmaf(e < 4 ? s0[qc][e] : s1[qc][e - 4], sc, -m[qc]));
          sum += pe;
          pB[qc][e] = (__bf16)pe;
        }
        ps[qc] = sum;
        over |= !(sum <= kWeightCap);
      }
      return over;
    };
    auto column_max = [&](int qc) {
      float mx = kNegInf;
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, e < 4 ? s0[qc][e] : s1[qc][e - 4]);
      return max_xor16_32(mx) * sc;
    };
    // The wave's first step sets the reference before its weights (it would always move it);
    // its sums and accumulators are still zero.
    if (st == wlo) {
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) m[qc] = fmaxf(m[qc], column_max(qc));
    }
    // V^T operand of O^T += V^T P^T: lane (c16, j4) needs channel 16nb + c16 of keys
    // 4j4..4j4+3 and 16+4j4..16+4j4+3 (the key order of P^T in the score layout).  One
    // transposed read per half: within each 16-lane group, lane i names 4 channels
    // 16nb + 4(i mod 4) .. +3 of key row 4j4 + i/4, and lane c16 receives channel 16nb + c16 of
    // those four rows.  At d = 64 the reads travel under the weights, which hides them where few
    // waves share a SIMD (12/2 heads, B 2048, n 2048, 98 workgroups per unit: 40.6 -> 37.3 us; at
    // the paper's shape 53.7 -> 53.2); at d = 128 their 32 registers would be spilled.
    u32x2 vr[2 * NB];
    if constexpr (D == 64) {
      read_chunks<D, TILE>(vr, va, sb);
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool over = weights();
    if constexpr (D == 64) wait_chunks<D>(vr);
    if (__builtin_amdgcn_ballot_w64(over) != 0) {
#pragma unroll
      for (int qc = 0; qc < QC; ++qc) {
        const float cand = column_max(qc);
        const bool grow = cand > m[qc];
        const float alpha = grow ? fast_exp2(m[qc] - cand) : 1.0f;
        m[qc] = grow ? cand : m[qc];
        lsum[qc] *= alpha;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[qc][nb] *= alpha;
      }
      weights();
    }
#pragma unroll
    for (int qc = 0; qc < QC; ++qc) lsum[qc] += ps[qc];
    if constexpr (D == 128) {
      read_chunks<D, TILE>(vr, va, sb);
      wait_chunks<D>(vr);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const bf16x8 vt = join_chunks(vr[2 * nb], vr[2 * nb + 1]);
#pragma unroll
      for (int qc = 0; qc < QC; ++qc)
        acc[qc][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pB[qc], acc[qc][nb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const int m1 = min(max(ua, wlo), whi + 1);   // [m1, m2): no masks
  const int m2 = min(max(ub, m1), whi + 1);
  int st = 0;
  for (; st < wlo; ++st) begin_step(st);
  if constexpr (LOOPS) {
    for (; st < m1; ++st) {
      const uint32_t sb = begin_step(st);
      step(st, sb, std::true_type{});
    }
    for (; st < m2; ++st) {
      const uint32_t sb = begin_step(st);
      step(st, sb, std::false_type{});
    }
  }
  for (; st <= whi; ++st) {
    const uint32_t sb = begin_step(st);
    step(st, sb, std::true_type{});
  }
  for (; st < nsteps; ++st) begin_step(st);

  // Outputs: o = acc / l (bf16 RNE), lse = (m + log2 l) * ln 2.  Lane (c16, j4) holds channels
  // 16nb + 4j4 .. +3 of its column; a swap of neighbouring quarters gives each lane 8 consecutive
  // channels of every second block, so that a store writes 16 bytes per lane.  (The columns are
  // worked out again: kept across the key loop, they would cost registers that it needs.)
  int ce = c16;
  asm("" : "+v"(ce));
#pragma unroll
  for (int qc = 0; qc < QC; ++qc) {
    const float l = sum_xor16_32(lsum[qc]);
    const float inv = 1.0f / l;
    u32x4 w[NB / 2];
#pragma unroll
    for (int q = 0; q < NB / 2; ++q) w[q] = pair_blocks(acc[qc][2 * q], acc[qc][2 * q + 1], inv);
    const Column x = column(qc, ce);
    if (x.valid) {
      unsigned char* orow = (unsigned char*)a.out + row0 * ROWB + row_offset(x);
#pragma unroll
      for (int q = 0; q < NB / 2; ++q)
        *(u32x4*)(orow + 64 * q + 32 * (j4 & 1) + 16 * (j4 >> 1)) = w[q];
      if (a.lse != nullptr && j4 == 0)
        a.lse[((size_t)b * a.hq + (size_t)(g * G + x.head)) * n + t0 + x.cp] =
            (m[qc] + __builtin_log2f(l)) * 0.69314718055994531f;
    }
  }

  // Ring state after the prompt: positions max(0, n - slots) .. n-1 at slot s mod slots.
  if (a.k_ring != nullptr) {
    const int first = max(t0, n - a.slots);
    const int count = t_last - first + 1;
    for (int idx = tid; idx < 2 * count * PPR; idx += NW * 64) {
      const int which = idx / (count * PPR);
      const int rest = idx - which * count * PPR;
      const int t = first + rest / PPR;
      const int pc = rest % PPR;
      const unsigned char* src = (which ? vbase : kbase) + (size_t)t * rowstride + pc * 16;
      unsigned char* dst = (unsigned char*)(which ? a.v_ring : a.k_ring) +
                           ((size_t)bg * a.slots + (t % a.slots)) * ROWB + pc * 16;
      *(u32x4*)dst = *(const u32x4*)src;
    }
  }
}

// Where the heaviest tiles go first.  By weight against in order, us: 32/8 heads, d 128, B 2048,
// n 16000 (4000 workgroups, 15 half-blocks after the first) 370 / 378; B 512, n 4000 (1000, 15)
// 36.3 / 39.2, n 8000 (2000, 31) 68.1 / 65.6; batch 4, B 2048, n 8192 (8192, 7) 839 / 721.  16/4
// heads, d 64, B 512, n 16000 (2000, 62) 40.2 / 43.0, n 32000 (4000, 124) 81.3 / 76.4.
template <int D>
constexpr OrderLimits kPrefillByWeight = {4096, D == 128 ? 24 : 96};

// Keys of a half-block (or window) from which masked and unmasked steps stand in loops of their own
// at d = 128 (always at d = 64).  A branch around the mask inside one loop lengthens every step, loops
// apart take 12 bytes of scratch and more instructions to fetch, which counts in short walks.  Apart
// against together, us: 8/8 heads, B 4096, n 16384 181.4 / 190.7; 32/8 heads, B 2048, batch 4, n 16384
// 1450 / 1467; 24/8 heads, W 2578, batch 4, n 2829 180 / 185; 8/8 heads, W 903, n 58082 262.5 / 262.0;
// 32/8 heads, B 1024, batch 2, n 8192 237.7 / 234.6; 24/8 heads, B 78, batch 7, n 14977 376 / 360.
constexpr int kPrefillLoopKeys = 1024;

template <int D, int ST, int OCC, bool LOOPS>
hipError_t launch_prefill_loops(const PrefillArgs& a, hipStream_t stream) {
  const TilePlan pl = TilePlan::make(a.batch, a.hkv, a.group, a.n, a.mode == kSupportPBB, a.block,
                                     a.window, kPrefillCols / a.group, kPrefillByWeight<D>);
  const size_t blocks = (size_t)a.batch * a.hkv * pl.ranks();
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL((prefill_bf16_kernel<D, ST, OCC, LOOPS>), dim3((unsigned)blocks),
                     dim3(kPrefillWaves * 64), 0, stream, a, pl);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_bf16(const PrefillArgs& a, int32_t head_dim, hipStream_t stream) {
  if (head_dim == 64)
    return launch_prefill_loops<64, kPrefillStages64, kPrefillOcc64, true>(a, stream);
  const int keys = a.mode == kSupportPBB ? a.block / 2 : a.window;
  return (keys < a.n ? keys : a.n) >= kPrefillLoopKeys
             ? launch_prefill_loops<128, kPrefillStages128, kPrefillOcc128, true>(a, stream)
             : launch_prefill_loops<128, kPrefillStages128, kPrefillOcc128, false>(a, stream);
}

}  // namespace pbb
