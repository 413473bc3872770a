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

}  // namespace pbb
