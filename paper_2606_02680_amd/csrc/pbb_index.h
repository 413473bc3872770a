// Index arithmetic of the prefill and backward launches, usable on the host and in kernels (and by
// a plain C++ compiler: nothing here needs HIP).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define PBB_HD __host__ __device__ __forceinline__
#else
#define PBB_HD inline
#endif

namespace pbb {

// x / d for 0 <= x < 2^31 and a launch constant d, without a division (the kernels divide by the
// half-block, the group size and grid extents, and a 32-bit division costs ~25 instructions):
// mul = ceil(2^(31+s) / d) with 2^(s-1) < d <= 2^s, and x / d = (2 x mul >> 32) >> s.  Exact: the
// excess of mul d over 2^(31+s) is below d <= 2^s, so the error of x mul / 2^(31+s) stays below
// x 2^-31 / d < 1 / d.
struct FastDiv {
  uint32_t mul, shift, d;
  static FastDiv make(uint32_t d) {
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    return FastDiv{(uint32_t)(((1ull << (31 + s)) + d - 1) / d), s, d};
  }
  PBB_HD int div(int x) const {
    return (int)((uint32_t)(((uint64_t)(2u * (uint32_t)x) * mul) >> 32) >> shift);
  }
};

// Tiles of a unit from the heaviest to the lightest.  A tile's weight is the length of its key
// interval: with tph tiles per half-block, the tile of phase r has r + tph tile lengths of keys in
// the half-blocks after the first, r in the first (SWA: all its tiles are one run with rising
// weight).  So the order is: phases of half-blocks 1..J from the last phase down, then the first
// half-block's.  The last half-block may be cut short: its `rem` phases are the lower ones.
// (Where h is not a multiple of TQ the phases drift: still a permutation, a little off in weight.)
struct TileOrder {
  int first;       // tiles of the first half-block
  int others;      // tiles after it
  int tph, rem;    // tiles per half-block, of the last half-block
  int cut;         // ranks of the phases that the last half-block does not have
  FastDiv by_units, by_j, by_j1;   // units; half-blocks after the first, and all of them but one
  static TileOrder make(int tiles, int tph, int units) {
    TileOrder o;
    o.tph = tph;
    o.first = tiles < tph ? tiles : tph;
    o.others = tiles - o.first;
    const int j = (o.others + tph - 1) / tph;
    o.rem = o.others - (j > 0 ? j - 1 : 0) * tph;
    o.cut = (tph - o.rem) * (j > 0 ? j - 1 : 0);
    o.by_units = FastDiv::make((uint32_t)units);
    o.by_j = FastDiv::make((uint32_t)(j > 0 ? j : 1));
    o.by_j1 = FastDiv::make((uint32_t)(j > 1 ? j - 1 : 1));
    return o;
  }
  PBB_HD int tile(int rank) const {
    if (rank >= others) return first - 1 - (rank - others);
    if (rank < cut) {
      const int q = by_j1.div(rank);
      return (1 + rank - q * (int)by_j1.d) * tph + tph - 1 - q;
    }
    const int q = by_j.div(rank - cut);
    return (1 + rank - cut - q * (int)by_j.d) * tph + rem - 1 - q;
  }
};

// Order of a launch's workgroups over its (unit, tile) pairs.
//
// Launches of at most kByWeightMaxBlocks workgroups (16 per CU), with at least kByWeightMinPhases
// tiles per half-block (SWA: per prompt), deal out their tiles heaviest first instead of in order.
// In order, a CU's few workgroups often have the same phase (with 32 tiles per unit, the 32 CUs of
// an XCD each take one tile index of every unit) and the launch waits for the CUs with the longest
// intervals; with many workgroups per CU that evens out, and tiles in order share their keys in
// an XCD's L2.  Measured, by weight against in order, 32/8 heads, d 128, B 2048: batch 3, n 1021
// (768 workgroups) 36.1 against 49.1 us; batch 1, n 2000 54.8 / 58.7; batch 4, n 2048 146 / 165;
// batch 4, n 4096 (4096) 341 / 347; batch 4, n 8192 (8192) 839 / 721.  16/4 heads, d 64, B 512 (8
// tiles per half-block): batch 8, n 500 15.1 / 17.5, batch 4, n 8192 (4096) 81.9 / 81.5.  12/2
// heads, d 64, B 128 (3 tiles per half-block, which mix anyway): n 16384 20.8 / 18.7.
constexpr int kByWeightMaxBlocks = 4096;
constexpr int kByWeightMinPhases = 8;

// The query tiles of a prefill or dq launch: `tq` consecutive positions per tile, `tiles` per unit
// (sequence, KV head).
struct TilePlan {
  int tq, tiles;
  int pbb;                 // 1: PBB supports, 0: sliding window
  int by_weight;           // 1: tiles are dealt out heaviest first, 0: in order
  FastDiv by_tiles, by_hkv, by_group, by_half;
  TileOrder order;
  static TilePlan make(int batch, int hkv, int group, int n, bool pbb, int block, int tq) {
    TilePlan p;
    p.tq = tq;
    p.tiles = (n + tq - 1) / tq;
    p.pbb = pbb;
    p.by_tiles = FastDiv::make((uint32_t)p.tiles);
    p.by_hkv = FastDiv::make((uint32_t)hkv);
    p.by_group = FastDiv::make((uint32_t)group);
    p.by_half = FastDiv::make((uint32_t)(pbb ? block / 2 : 1));
    const int tph = pbb ? block / 2 / tq : p.tiles;
    p.by_weight = (uint64_t)batch * hkv * p.tiles <= (uint64_t)kByWeightMaxBlocks &&
                  tph >= kByWeightMinPhases;
    p.order = TileOrder::make(p.tiles, tph > 0 ? tph : 1, batch * hkv);
    return p;
  }
  // Unit and tile of workgroup k of `blocks`.  Workgroup k runs on XCD k mod 8: in order, each XCD
  // takes a contiguous run of tiles, so that tiles sharing keys (neighbours of one unit) share
  // that XCD's L2.
  PBB_HD void locate(int k, int blocks, int& unit, int& tile) const {
    if (by_weight) {
      const int rank = order.by_units.div(k);
      unit = k - rank * (int)order.by_units.d;
      tile = order.tile(rank);
    } else {
      const int per = blocks >> 3, rem = blocks & 7;
      const int xcd = k & 7, local = k >> 3;
      const int id = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + local;
      unit = by_tiles.div(id);
      tile = id - unit * tiles;
    }
  }
  // First source a(t) of the support of target t: PBB max(0, h(floor(t/h) - 1)) with h = block/2
  // (Sec. 3 "Flash-PBB"), SWA max(0, t - window + 1) (Prop. 2).  Never decreases in t.
  PBB_HD int support_lo(int t, int block, int window) const {
    const int lo = pbb ? (block >> 1) * (by_half.div(t) - 1) : t - window + 1;
    return lo > 0 ? lo : 0;
  }
};

// The key tiles of a dk/dv launch: `keys` consecutive keys per tile, `tiles` per unit, in order
// (each XCD a contiguous run).
struct DkdvPlan {
  int tiles;
  int pbb;
  FastDiv by_tiles, by_hkv, by_half;
  static DkdvPlan make(int hkv, int n, bool pbb, int block, int keys) {
    DkdvPlan p;
    p.tiles = (n + keys - 1) / keys;
    p.pbb = pbb;
    p.by_tiles = FastDiv::make((uint32_t)p.tiles);
    p.by_hkv = FastDiv::make((uint32_t)hkv);
    p.by_half = FastDiv::make((uint32_t)(pbb ? block / 2 : 1));
    return p;
  }
  PBB_HD void locate(int k, int blocks, int& unit, int& tile) const {
    const int per = blocks >> 3, rem = blocks & 7;
    const int xcd = k & 7, local = k >> 3;
    const int id = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + local;
    unit = by_tiles.div(id);
    tile = id - unit * tiles;
  }
  // Last target whose support contains source s (the largest t with support_lo(t) <= s): PBB
  // h(floor(s/h) + 2) - 1, SWA s + window - 1.
  PBB_HD int last_target(int s, int block, int window) const {
    return pbb ? (block >> 1) * (by_half.div(s) + 2) - 1 : s + window - 1;
  }
};

}  // namespace pbb
