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
