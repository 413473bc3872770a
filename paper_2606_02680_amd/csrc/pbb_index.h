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
// interval.  PBB: the tile that begins r tq .. (r+1) tq - 1 positions into its half-block (phase r)
// has some r + tph tile lengths of keys in the half-blocks after the first, r in the first.  So
// the order is: phases of half-blocks 1..J from the last phase down, then the first half-block's
// tiles from the last down.  The last half-block may be cut short: its `rem` phases are the lower
// ones.  Where tq does not divide the half-block, only some half-blocks have a tile of the last
// phase; the ranks of the others are holes (tile -1).  SWA: one run with rising weight, up to the
// first whole window, taken as a prompt within the first half-block.
struct TileOrder {
  int ranks;       // tiles and holes
  int first;       // tiles of the first half-block
  int others;      // ranks of the half-blocks after it
  int rem;         // phases of the last half-block
  int cut;         // ranks of the phases that the last half-block does not have
  int h, tq, tiles;
  FastDiv by_tq, by_j, by_j1;   // tq; half-blocks after the first, and all of them but one
  static TileOrder make(int n, int h, int tq) {
    TileOrder o;
    o.h = h;
    o.tq = tq;
    o.tiles = (n + tq - 1) / tq;
    const int tph = (h + tq - 1) / tq;
    const int j = (n - 1) / h;
    o.first = o.tiles < tph ? o.tiles : tph;
    o.rem = j > 0 ? (n - j * h + tq - 1) / tq : 0;
    o.others = j > 0 ? (j - 1) * tph + o.rem : 0;
    o.cut = j > 0 ? (tph - o.rem) * (j - 1) : 0;
    o.ranks = o.first + o.others;
    o.by_tq = FastDiv::make((uint32_t)tq);
    o.by_j = FastDiv::make((uint32_t)(j > 0 ? j : 1));
    o.by_j1 = FastDiv::make((uint32_t)(j > 1 ? j - 1 : 1));
    return o;
  }
  PBB_HD int tile(int rank) const {
    if (rank >= others) return first - 1 - (rank - others);
    int j, r;
    if (rank < cut) {
      const int q = by_j1.div(rank);
      j = 1 + rank - q * (int)by_j1.d;
      r = first - 1 - q;   // (with two half-blocks after it, the first one is whole)
    } else {
      const int q = by_j.div(rank - cut);
      j = 1 + rank - cut - q * (int)by_j.d;
      r = rem - 1 - q;
    }
    const int t = by_tq.div(j * h + tq - 1) + r;   // the first tile of the half-block, and r more
    return t < tiles && t * tq < (j + 1) * h ? t : -1;
  }
};

// Order of a launch's workgroups over its (unit, tile) pairs: in order, or heaviest first.
//
// In order, a CU's few workgroups often have the same phase (with 32 tiles per unit, the 32 CUs of
// an XCD each take one tile index of every unit) and the launch waits for the CUs with the longest
// intervals; with many workgroups per CU that evens out.  Heaviest first, tiles that share keys run
// on different XCDs and further apart in time, the more so the more half-blocks a phase's tiles
// come from.  So heaviest first is for launches whose tiles differ in weight (at least
// kByWeightMinPhases tiles per half-block or window) with few workgroups and few half-blocks per
// prompt.  The limits are each kernel's own (OrderLimits).  Prefill, by weight against in order, us:
// 16/2 heads, d 128, B 2048, n 8000 (7 half-blocks after the first, 1000 workgroups) 100.3 / 123.0;
// B 512, n 4000 (15, 500) 21.6 / 23.0, n 16000 (62, 2000) 72.2 / 64.6; 12/2 heads, d 64, B 2708,
// n 7980 (5, 760) 65.7 / 87.7; B 338, n 42000 (248, 4000) 63.8 / 62.4.
//
// Sliding windows: all tiles after the first window weigh the same.  Heaviest first (that is, from
// the last tile down) pays where the first window holds a good part of the tiles, or where it
// spans so many tiles that walks are long: 16/4 heads, d 64, W 2048 (64 tiles), n 16000 (500 tiles
// per unit) 145.5 / 153.1; 16/2 heads, d 128, W 512 (32 tiles), n 8000 (500) 45.1 / 44.6; 12/2
// heads, d 64, W 128 (6 tiles), n 16384 24.2 / 22.4.  With one to two workgroups per CU it pays where
// the second ones are all of the first window: 12/2 heads, d 64, 300 workgroups: W 672 (64 of them
// light) 15 % faster, W 336 (32) 2 %; 500 workgroups: W 1344 (128) 0.5 % slower.
struct OrderLimits {   // (PBB)
  int blocks;   // workgroups, at most
  int halves;   // half-blocks per prompt, at most
};
constexpr int kByWeightMinPhases = 8;
constexpr int kByWeightMinWindow = 4;    // SWA (batch 8, 16/4 heads, d 64, W 240, n 708: 13.4 / 14.8)
constexpr int kByWeightMaxWindow = 4096; // SWA: workgroups, at most
constexpr int kCUs = 256;
constexpr int kByWeightRising = 5;       // SWA: the first window holds at least a fifth of the tiles
constexpr int kByWeightLongWindow = 64;  // or this many

// The query tiles of a prefill or dq launch: `tq` consecutive positions per tile, `tiles` per unit
// (sequence, KV head).
struct TilePlan {
  int tq, tiles;
  int pbb;                 // 1: PBB supports, 0: sliding window
  int by_weight;           // 1: tiles are dealt out heaviest first, 0: in order
  FastDiv by_tiles, by_units, by_hkv, by_group, by_half;
  TileOrder order;
  static TilePlan make(int batch, int hkv, int group, int n, bool pbb, int block, int window, int tq,
                       OrderLimits lim) {
    TilePlan p;
    p.tq = tq;
    p.tiles = (n + tq - 1) / tq;
    p.pbb = pbb;
    p.by_tiles = FastDiv::make((uint32_t)p.tiles);
    p.by_units = FastDiv::make((uint32_t)(batch * hkv));
    p.by_hkv = FastDiv::make((uint32_t)hkv);
    p.by_group = FastDiv::make((uint32_t)group);
    p.by_half = FastDiv::make((uint32_t)(pbb ? block / 2 : 1));
    p.order = TileOrder::make(n, pbb ? block / 2 : n, tq);
    const int phases = (pbb ? block / 2 : window < n ? window : n) / tq;
    const int64_t units = (int64_t)batch * hkv, blocks = units * p.tiles;
    bool pays;
    if (pbb)
      pays = phases >= kByWeightMinPhases && (n - 1) / (block / 2) < lim.halves;
    else if (blocks <= 2 * kCUs)
      pays = phases >= kByWeightMinWindow && units * phases >= blocks - kCUs;
    else
      pays = phases >= kByWeightLongWindow ||
             (phases >= kByWeightMinWindow && p.tiles <= kByWeightRising * phases);
    p.by_weight = pays && blocks <= (pbb ? lim.blocks : kByWeightMaxWindow);
    return p;
  }
  // Workgroups per unit.
  int ranks() const { return by_weight ? order.ranks : tiles; }
  // Unit and tile of workgroup k of `blocks` (tile -1: none).  Workgroup k runs on XCD k mod 8: in
  // order, each XCD takes a contiguous run of tiles, so that tiles sharing keys (neighbours of one
  // unit) share that XCD's L2.
  PBB_HD void locate(int k, int blocks, int& unit, int& tile) const {
    if (by_weight) {
      const int rank = by_units.div(k);
      unit = k - rank * (int)by_units.d;
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
