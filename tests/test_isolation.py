"""Data of one position must not reach the results of positions, heads or keys that do not attend
to it (GPU, through the C ABI): the same call with other data there gives the same bits."""
from __future__ import annotations

import pytest
import torch

import paper_2606_02680_amd as P
from tests.harness import bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,block,window,n", [
    (64, 6, 256, 0, 132),       # tiles of 21 positions: the last one holds 6, their 36 columns
    (128, 6, 256, 0, 132),      # cut a wave's 32 after head 1 of the last position
    (64, 6, 0, 200, 132),
    (64, 5, 200, 0, 82),        # tiles of 25, 7 positions in the last: cut after head 1
])
def test_prefill_cut_tile_heads(cuda, d, hq, block, window, n):
    """A wave with columns past the prompt's end: heads 0 and 1 of the last position sit in the
    wave before, and a query of theirs whose scores rise by ~40 log2 units in the middle of the
    walk (which moves its own wave's softmax references) leaves the other heads' bits alone."""
    batch = 16
    g = torch.Generator().manual_seed(5)
    q, k, v = (torch.randn(batch, n, h, d, generator=g).to(cuda, torch.bfloat16) for h in (hq, 1, 1))
    k[:, 70, 0, 0] = 16.0
    q[..., 0] = 0.0                      # nobody but the changed query sees the key's boost
    if window:
        desc, fn = P.make_desc(batch, hq, 1, d, window=window), P.swa_prefill
    else:
        desc, fn = P.make_desc(batch, hq, 1, d, block=block), P.pbb_prefill
    outs = []
    for boost in (0.0, 16.0):
        q2 = q.clone()
        q2[:, n - 1, :2, 0] = boost
        out = torch.empty_like(q)
        lse = torch.empty((batch, hq, n), dtype=torch.float32, device=cuda)
        print(f"[isolation] prefill {d} {hq} {block} {window} {n} boost {boost}", flush=True)
        fn(desc, q2, k, v, out, lse=lse)
        torch.cuda.synchronize()
        outs.append((out, lse))
    (o0, l0), (o1, l1) = outs
    assert not torch.equal(o0[:, n - 1, :2], o1[:, n - 1, :2])
    assert (bits(o0[:, n - 1, 2:]) == bits(o1[:, n - 1, 2:])).all()
    assert torch.equal(l0[:, 2:, n - 1], l1[:, 2:, n - 1])


@pytest.mark.parametrize("value", [float("nan"), float("-inf")])
@pytest.mark.parametrize("d,hq,block,window,n,t", [
    (128, 4, 256, 0, 300, 140),      # keys after the target and before its support share its steps
    (64, 6, 64, 0, 200, 75),
    (64, 4, 0, 45, 200, 110),
])
def test_backward_bad_log_partition(cuda, d, hq, block, window, n, t, value):
    """A target whose log-partition is NaN or -inf: dk and dv of the keys outside its support keep
    their bits (pairs outside the support weigh exactly 0)."""
    g = torch.Generator().manual_seed(6)
    q, do = (torch.randn(2, n, hq, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(2, n, 2, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    if window:
        desc = P.make_desc(2, hq, 2, d, window=window)
        fwd, bwd, lo = P.swa_prefill, P.swa_backward, max(0, t - window + 1)
    else:
        desc, h = P.make_desc(2, hq, 2, d, block=block), block // 2
        fwd, bwd, lo = P.pbb_prefill, P.pbb_backward, max(0, h * (t // h - 1))
    out = torch.empty_like(q)
    lse = torch.empty((2, hq, n), dtype=torch.float32, device=cuda)
    fwd(desc, q, k, v, out, lse=lse)
    grads = []
    for bad in (False, True):
        if bad:
            lse[:, :, t] = value
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        print(f"[isolation] backward {d} {hq} {block} {window} {n} {value if bad else ''}", flush=True)
        bwd(desc, q, k, v, out, do, lse, dq, dk, dv)
        torch.cuda.synchronize()
        grads.append((dk, dv))
    for a, b in zip(*grads):
        assert not torch.isfinite(b[:, t]).all()
        for keys in (slice(0, lo), slice(t + 1, n)):
            assert torch.equal(a[:, keys], b[:, keys])


@pytest.mark.parametrize("d", [64, 128])
def test_backward_infinite_weight(cuda, d):
    """The first position sees only itself: with a log-partition of -inf its weight is infinite, and
    so is its dq (keys outside the support weigh exactly 0, not exp(-inf + inf))."""
    n, hq = 40, 4
    g = torch.Generator().manual_seed(7)
    q, do = (torch.randn(2, n, hq, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(2, n, 2, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    desc = P.make_desc(2, hq, 2, d, block=64)
    out = torch.zeros_like(q)
    lse = torch.zeros((2, hq, n), dtype=torch.float32, device=cuda)
    lse[:, :, 0] = float("-inf")
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    print(f"[isolation] infinite weight {d}", flush=True)
    P.pbb_backward(desc, q, k, v, out, do, lse, dq, dk, dv)
    assert torch.isinf(dq[:, 0]).all()
    assert torch.isfinite(dq[:, 1:]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_infinity_in_the_last_row(cuda, d):
    """Tile rows past the prompt's end weigh 0 and must hold nothing of the last position but its
    last 8 channels: an infinity in another channel of its value (or of its upstream gradient)
    arrives as an infinity in its output (in dv of its support's keys), not as 0 * inf."""
    n, hq, ch = 132, 8, 5
    g = torch.Generator().manual_seed(8)
    q, do = (torch.randn(2, n, hq, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(2, n, 2, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    desc = P.make_desc(2, hq, 2, d, block=128)
    out = torch.empty_like(q)
    lse = torch.empty((2, hq, n), dtype=torch.float32, device=cuda)
    v2, do2 = v.clone(), do.clone()
    v2[:, n - 1, :, ch] = float("inf")
    do2[:, n - 1, :, ch] = float("inf")
    print(f"[isolation] infinity {d}", flush=True)
    P.pbb_prefill(desc, q, k, v2, out, lse=lse)
    assert torch.isposinf(out[:, n - 1, :, ch]).all()
    P.pbb_prefill(desc, q, k, v, out, lse=lse)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    P.pbb_backward(desc, q, k, v, out, do2, lse, dq, dk, dv)
    assert torch.isposinf(dv[:, 64:, :, ch]).all()       # the support of n - 1 is 64 .. n - 1
    other = [c for c in range(d) if c != ch]
    assert torch.isfinite(dv[..., other]).all()


@pytest.mark.parametrize("batch,hkv,block", [(5, 8, 2048), (2, 4, 512)])
def test_split_decode_infinite_value(cuda, batch, hkv, block):
    """Split launches of 6 and of 2 workgroups per unit: an infinite value of the current token
    arrives as an infinity (the merge takes every state once, none with weight 0)."""
    hq, d, ch = 4 * hkv, 128, 7
    g = torch.Generator().manual_seed(9)
    desc = P.make_desc(batch, hq, hkv, d, block=block)
    assert P.workspace_bytes(desc) > 0
    rings = [torch.randn(batch, hkv, block, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2)]
    q = torch.randn(batch, hq, d, generator=g).to(cuda, torch.bfloat16)
    k, v = (torch.randn(batch, hkv, d, generator=g).to(cuda, torch.bfloat16) for _ in range(2))
    pos = torch.arange(batch, dtype=torch.int32, device=cuda) * 37 + 3 * block + block - 200
    ref, out = torch.empty_like(q), torch.empty_like(q)
    print(f"[isolation] split {batch} {hkv} {block}", flush=True)
    P.pbb_decode_step(desc, pos, q, k, v, *rings, ref)
    v[..., ch] = float("inf")
    P.pbb_decode_step(desc, pos, q, k, v, *rings, out)
    assert torch.isposinf(out[..., ch]).all()
    other = [c for c in range(d) if c != ch]
    assert torch.equal(out[..., other], ref[..., other])
