"""fp32 decode with one query head per KV head (the vector-ALU kernel): supports around the 64
keys that a workgroup's streams take at a time, and rings on both sides of the size from which
loads are non-temporal, against the fp64 oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2606_02680_amd as P
import workloads as W
from harness import Run, compare, to_np

pytestmark = pytest.mark.gpu

CASES = [  # mode, batch, hkv, d, block or window, slots
    ("pbb", 5, 2, 64, 2, 2), ("pbb", 9, 1, 128, 130, 130), ("swa", 7, 3, 64, 64, 67),
    ("swa", 6, 2, 128, 65, 65), ("pbb", 3, 4, 64, 512, 512),
    ("pbb", 130, 8, 64, 512, 512),      # 260 MiB of rings: non-temporal loads
    ("swa", 65, 8, 128, 500, 513),
]


@pytest.mark.parametrize("mode,batch,hkv,d,span,slots", CASES)
def test_f32_single_head(cuda, mode, batch, hkv, d, span, slots):
    cfg = W.Config("f32-g1", mode, batch=batch, hq=hkv, hkv=hkv, d=d,
                   block=span if mode == "pbb" else 0, slots=slots,
                   window=span if mode == "swa" else 0, dtype="f32", seed=29, value_scale=1.0,
                   pos_hi=0, steps=3, prefill=True)
    # supports of 1, 63..66 keys and around a block's or window's ends, then random positions
    edge = [0, 62, 63, 64, 65, span - 1, span, span + span // 2]
    g = torch.Generator().manual_seed(7)
    t0 = torch.randint(0, 1 << 16, (batch,), generator=g, dtype=torch.int64)
    t0[:len(edge)] = torch.tensor(edge[:batch])
    run = Run(cfg, t0, cfg.steps, cuda)
    rows = np.unique(np.r_[:min(batch, 10), batch - 1])
    for i in range(cfg.steps):
        q, out = run.step()
        ref = run.oracle_out(rows, i, q)
        compare(cfg, to_np(out)[rows], ref, f"step {i}")
    hist = run.history(rows, cfg.steps - 1)
    for which in ("k", "v"):
        assert np.array_equal(run.ring_rows(rows, which),
                              run.expected_ring(rows, cfg.steps - 1, which, hist))


@pytest.mark.parametrize("mode,d,span", [("pbb", 64, 130), ("pbb", 128, 130), ("swa", 128, 65)])
def test_f32_infinite_value(cuda, mode, d, span):
    """An infinite channel of the current token's value arrives as an infinity: keys past the
    support's end, which the streams read as further copies of that token, add nothing."""
    batch, hkv, ch = 8, 2, 9
    g = torch.Generator().manual_seed(3)
    kw = {"block": span} if mode == "pbb" else {"window": span}
    desc = P.make_desc(batch, hkv, hkv, d, dtype=torch.float32, **kw)
    fn = P.pbb_decode_step if mode == "pbb" else P.swa_decode_step
    kr, vr = (torch.randn(batch, hkv, span, d, generator=g).to(cuda) for _ in range(2))
    q, k, v = (torch.randn(batch, hkv, d, generator=g).to(cuda) for _ in range(3))
    pos = torch.tensor([0, 1, 15, 16, 40, 63, 64, 777], dtype=torch.int32, device=cuda)
    ref, out = torch.empty_like(q), torch.empty_like(q)
    print(f"[f32 single head] infinite value {mode} {d} {span}", flush=True)
    fn(desc, pos, q, k, v, kr, vr, ref)
    v[..., ch] = float("inf")
    fn(desc, pos, q, k, v, kr, vr, out)
    assert torch.isposinf(out[..., ch]).all()
    other = [c for c in range(d) if c != ch]
    assert torch.equal(out[..., other], ref[..., other])
