"""Tile order, step ranges and index arithmetic of the prefill and backward launches.

On the CPU: ``csrc/pbb_index.h`` compiled with g++ -- FastDiv against the division over edge and
random dividends, TilePlan's two orders each a permutation of the tiles over all group sizes, the
one by weight with falling weights.  On the GPU: prompts whose launches take the by-weight order
(and neighbours that do not), against the oracle (the backward's dq launch shares them):
half-blocks that the tile length does not divide (whose ranks have holes), cut last half-blocks,
prompts within the first half-block, numbers of units that are no multiple of the 8 XCDs, and tiles
some of whose waves skip steps or hold no position at all.
"""
from __future__ import annotations

import os
import subprocess

import pytest

from tests.test_backward import _check_all, _run
from tests.test_prefill import _cfg, _check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "pbb_index.h"
int main() {
  std::mt19937 rng(5);
  auto check = [](uint32_t d, int x) { return pbb::FastDiv::make(d).div(x) == (int)((uint32_t)x / d); };
  for (int i = 0; i < 200000; ++i) {
    const uint32_t d = i < 3000 ? i + 1 : 1 + (rng() >> (1 + rng() % 31)) % 0x7fffffffu;
    const int m = 0x7fffffff, q = (int)(m / d) * d, r = (int)(rng() >> 1);
    for (int x : {0, 1, (int)(d - 1), (int)(d < 0x7fffffffu ? d : 0), m, q, q > 0 ? q - 1 : 0, r})
      if (!check(d, x)) return std::printf("div %u %d\n", d, x), 1;
  }
  // A launch's workgroups: every (unit, tile) pair once, in both orders; by weight, no tile a tile
  // length or more heavier than one dealt before it (keys from its first position's support to its
  // last position, the last tile taken whole), and at most one hole per half-block.
  int weighed = 0;
  for (int i = 0; i < 6000; ++i) {
    const int group = 1 + rng() % 16, tq = 128 / group, batch = 1 + rng() % 3, hkv = 1 + rng() % 9;
    const int n = 1 + rng() % (i % 2 ? 40000 : 3000);
    const int block = 2 * (1 + rng() % (i % 3 ? 2500 : 200)), window = 1 + rng() % 5000;
    const bool pbb = i % 4 != 0;
    const pbb::OrderLimits lim = {i % 5 ? 1 << 30 : 0, 1 << 30};   // (PBB: both orders)
    const auto p = pbb::TilePlan::make(batch, hkv, group, n, pbb, block, window, tq, lim);
    const int units = batch * hkv, blocks = units * p.ranks();
    std::vector<char> seen((size_t)units * p.tiles, 0);
    std::vector<int> least(units, 1 << 30);
    int holes = 0, pairs = 0;
    for (int k = 0; k < blocks; ++k) {
      int unit, t;
      p.locate(k, blocks, unit, t);
      if (unit < 0 || unit >= units) return std::printf("unit %d %d\n", i, k), 1;
      if (t == -1) { ++holes; continue; }
      if (t < 0 || t >= p.tiles || seen[(size_t)unit * p.tiles + t])
        return std::printf("tile %d %d %d\n", i, k, t), 1;
      seen[(size_t)unit * p.tiles + t] = 1;
      ++pairs;
      const int w = t * tq + tq - p.support_lo(t * tq, block, window);
      if (p.by_weight && w >= least[unit] + tq) return std::printf("weight %d %d %d\n", i, k, w), 1;
      if (w < least[unit]) least[unit] = w;
    }
    const int halves = pbb ? (n - 1) / (block / 2) : 0;
    if (pairs != units * p.tiles || holes > units * halves || (holes && !p.by_weight))
      return std::printf("pairs %d %d %d\n", i, pairs, holes), 1;
    weighed += p.by_weight;
  }
  if (weighed < 1000) return std::printf("weighed %d\n", weighed), 1;
  return 0;
}
"""


def test_index_arithmetic(tmp_path):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    inc = os.path.join(ROOT, "paper_2606_02680_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", inc, str(src), "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("mode,batch,n,hq,hkv,d,block,window,slots", [
    ("pbb", 3, 1021, 8, 2, 128, 2048, 0, 0),     # within the first half-block
    ("pbb", 1, 1337, 6, 1, 64, 500, 0, 0),       # tiles of 21, half-blocks of 250: 11 phases
    ("pbb", 5, 700, 5, 1, 128, 514, 0, 0),       # tiles of 25, half-blocks of 257
    ("pbb", 2, 1500, 7, 1, 64, 342, 0, 0),       # tiles of 18, half-blocks of 171: holes
    ("pbb", 2, 913, 16, 4, 64, 512, 0, 0),       # 8 phases exactly, a cut last half-block
    ("pbb", 2, 913, 16, 4, 64, 510, 0, 0),       # 7 phases: in order
    ("swa", 3, 450, 4, 1, 128, 0, 200, 200),
    ("swa", 1, 130, 16, 1, 64, 0, 64, 70),       # tiles of 8 positions
    ("pbb", 1, 33, 4, 4, 64, 64, 0, 0),          # G = 1: two of a tile's waves hold nothing
])
def test_prefill_orders(cuda, mode, batch, n, hq, hkv, d, block, window, slots):
    _check(_cfg(mode, batch, n, hq, hkv, d, block, window, slots), n, cuda)


@pytest.mark.gpu
@pytest.mark.parametrize("mode,batch,n,hq,hkv,d,block,window", [
    ("pbb", 3, 421, 8, 2, 128, 512, 0),       # dealt out by weight, cut last half-block
    ("pbb", 1, 1100, 6, 1, 64, 400, 0),       # tiles of 21, half-blocks of 200: holes
    ("pbb", 1, 173, 10, 2, 64, 96, 0),        # h 48: key tiles across half-blocks
    ("pbb", 2, 65, 4, 4, 128, 2, 0),          # one key past a tile; every step masked
    ("pbb", 1, 17, 16, 1, 64, 64, 0),         # waves without keys or targets
    ("swa", 1, 300, 6, 1, 128, 0, 45),        # windows that end inside a wave's keys
    ("swa", 2, 129, 4, 2, 64, 0, 4096),
])
def test_backward_orders(cuda, mode, batch, n, hq, hkv, d, block, window):
    got, ref, inputs = _run(mode, batch, n, hq, hkv, d, block, window, cuda)
    _check_all(f"{mode} n={n} hq={hq} hkv={hkv} d={d}", mode, inputs, got, ref, block, window)
