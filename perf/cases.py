"""The measured work of this framework: decode steps, prompt prefills and training passes.

Every case goes through the package's public entry points with preallocated buffers, as a serving
or training loop holds them.  Head shapes, block sizes, windows and prompt lengths are those of
``workloads/configs.py`` and ``bench.py`` (the paper's model shape: 10-14 query heads on 2 KV
heads, d 64, B 128; the throughput shape: 32/8 heads, d 128, B 2048; the ragged shape: 16/2
heads, d 128, B 1024), with odd and ragged sizes between them.

Kinds of a case:

* ``step``: one eager decode step of the whole batch (append + attention) at random positions;
* ``graph``: ``steps`` consecutive decode steps captured once as a graph and replayed, the
  positions advancing on the device (what a latency-bound decode loop runs);
* ``prefill``: every position of ``batch`` prompts of ``n`` tokens, with the ring state that
  decoding continues from and the log-partitions;
* ``train``: the prefill attention and its backward for one upstream gradient.
"""
from __future__ import annotations

import math

import torch

import paper_2606_02680_amd as P

DEV = "cuda"


def _case(kind, batch, hq, hkv, d, *, block=0, window=0, slots=0, dtype="bf16", n=0, steps=1,
          pos_hi=524288, rope=0.0, spike=0.0):
    """A case as plain values; ``window`` > 0 selects the sliding-window entry points."""
    return {"kind": kind, "batch": batch, "hq": hq, "hkv": hkv, "d": d, "block": block,
            "window": window, "slots": slots or window or block, "dtype": dtype, "n": n,
            "steps": steps, "pos_hi": pos_hi, "rope": rope, "spike": spike}


def listed():
    cases = {
        # One token of one conversation, rotary positions applied in the launch: the smallest call.
        "step_single": _case("step", 1, 12, 2, 64, block=128, rope=1.0e6),
        # The paper's latency workload: batch 1, consecutive steps replayed as a graph.
        "graph_single": _case("graph", 1, 12, 2, 64, block=128, steps=64),
        # A few conversations of a larger model, replayed as a graph (split workgroups).
        "graph_few": _case("graph", 4, 32, 8, 128, block=2048, steps=16),
        # Batched serving at mixed positions: the headline decode workload.
        "step_throughput": _case("step", 256, 32, 8, 128, block=2048),
        # Many short-context sequences, 8 query heads per KV head, a few dominant keys.
        "step_ragged": _case("step", 1024, 16, 2, 128, block=1024, pos_hi=65536, spike=0.01),
        # The sliding-window baseline with a wrapping ring larger than its window, odd batch.
        "step_window": _case("step", 93, 32, 8, 128, window=4096, slots=4225, rope=1.0e6),
        # Full-precision decoding.
        "step_fp32": _case("step", 512, 16, 2, 128, block=1024, dtype="f32", pos_hi=65536),
        # Long prompts of the larger model, into the rings.
        "prefill_long": _case("prefill", 4, 32, 8, 128, block=2048, n=16384),
        # Short prompts of odd length arriving in a small batch.
        "prefill_short": _case("prefill", 3, 32, 8, 128, block=2048, n=1021),
        # A long prompt of the paper's model shape: small blocks, little work per position.
        "prefill_paper": _case("prefill", 1, 12, 2, 64, block=128, n=65536),
        # Training passes at the same two head shapes.
        "train_long": _case("train", 4, 32, 8, 128, block=2048, n=16384),
        "train_paper": _case("train", 1, 12, 2, 64, block=128, n=65536),
    }
    return [{"name": k, **v} for k, v in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above; no larger than the largest listed one of its kind."""
    kind = rng.choice(("step", "step", "graph", "prefill", "train"))
    hq, hkv, d = rng.choice(((10, 2, 64), (12, 2, 64), (14, 2, 64), (16, 4, 64), (32, 8, 128),
                             (16, 2, 128), (24, 8, 128), (8, 8, 128), (16, 1, 64)))
    window = slots = block = 0
    if rng.random() < 0.35:
        window = _log_int(rng, 64, 4096)
        slots = window + rng.choice((0, 1, 37, window))
    else:
        block = 2 * _log_int(rng, 32, 1024)
    span = window or block
    dtype = "f32" if kind == "step" and rng.random() < 0.3 else "bf16"
    rope = 1.0e6 if kind in ("step", "graph") and dtype == "bf16" and rng.random() < 0.4 else 0.0
    common = dict(block=block, window=window, slots=slots, dtype=dtype, rope=rope)
    if kind in ("step", "graph"):
        row = 2 * hkv * (slots or block) * d * (4 if dtype == "f32" else 2)
        most = max(1, min(1024 if kind == "step" else 16, (1 << 31) // row))
        return _case(kind, _log_int(rng, 1, most), hq, hkv, d, **common,
                     steps=1 if kind == "step" else 2 * rng.randint(4, 24),
                     pos_hi=rng.choice((2 * span, 65536, 524288)))
    n = _log_int(rng, 33, 65536)
    # positions x mean support x heads: at most the listed long prompts'
    pairs = 4 * 16384 * 32 * 128 * 1536 // 2
    most = max(1, int(min(8, 131072 // n, pairs // max(1, n * hq * d * min(n, span)))))
    return _case(kind, rng.randint(1, most), hq, hkv, d, **common, n=n)


# ------------------------------------------------------------------------------------------

def _desc(c):
    return P.make_desc(c["batch"], c["hq"], c["hkv"], c["d"], block=c["block"], window=c["window"],
                       slots=c["slots"], dtype=_dtype(c), rope_base=c["rope"])


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _inputs(c, seed):
    """The case's inputs, from the seed alone: N(0, 1) projections, a share ``spike`` of the
    tokens with keys and values scaled by 4, positions uniform below ``pos_hi``."""
    g = torch.Generator(device=DEV).manual_seed(seed * 7919 + 11)
    dt = _dtype(c)

    def randn(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=dt)

    b, hq, hkv, d, n = c["batch"], c["hq"], c["hkv"], c["d"], c["n"]
    s = {}
    if c["kind"] in ("step", "graph"):
        m = c["steps"]
        s["q"] = randn(m, b, hq, d)
        s["k_new"], s["v_new"] = randn(m, b, hkv, d), randn(m, b, hkv, d)
        s["k_ring"], s["v_ring"] = randn(b, hkv, c["slots"], d), randn(b, hkv, c["slots"], d)
        if c["spike"] > 0.0:
            mask = torch.rand((b, 1, c["slots"], 1), generator=g, device=DEV) < c["spike"]
            for name in ("k_ring", "v_ring"):
                s[name].mul_(torch.where(mask, 4.0, 1.0).to(dt))
        s["pos"] = torch.randint(0, c["pos_hi"], (b,), generator=g, device=DEV).to(torch.int32)
    else:
        s["q"] = randn(b, n, hq, d)
        s["k"], s["v"] = randn(b, n, hkv, d), randn(b, n, hkv, d)
        if c["kind"] == "train":
            s["dout"] = randn(b, n, hq, d)
    return s


def prepare(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    desc = s["desc"] = _desc(c)
    s["kind"], s["swa"] = c["kind"], c["window"] > 0
    if c["kind"] in ("step", "graph"):
        s["out"] = torch.empty_like(s["q"])
        s["workspace"] = P.alloc_workspace(desc, DEV)
    if c["kind"] == "step":
        for name in ("q", "k_new", "v_new", "out"):
            s[name] = s[name][0]
    elif c["kind"] == "graph":
        s["graph"] = _capture(c, s)
    else:
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((c["batch"], c["hq"], c["n"]), dtype=torch.float32, device=DEV)
        if c["kind"] == "prefill":
            s["k_ring"], s["v_ring"] = P.alloc_rings(desc, DEV)
            P.ring_init(desc, s["k_ring"], s["v_ring"])
        else:
            for name, like in (("dq", "q"), ("dk", "k"), ("dv", "v")):
                s[name] = torch.empty_like(s[like])
            s["workspace"] = torch.empty(max(1, P.backward_workspace_bytes(desc, c["n"])),
                                         dtype=torch.uint8, device=DEV)
    return s


def _capture(c, s):
    """Graph of an even number of decode steps: the positions alternate between two buffers, and
    the last launch leaves them in ``pos`` again."""
    fn = P.swa_decode_step_advance if s["swa"] else P.pbb_decode_step_advance
    a, b = s["pos"], torch.empty_like(s["pos"])
    s["pos2"] = b

    def body():
        cur, nxt = a, b
        for i in range(c["steps"]):
            fn(s["desc"], cur, nxt, s["q"][i], s["k_new"][i], s["v_new"][i], s["k_ring"],
               s["v_ring"], s["out"][i], workspace=s["workspace"])
            cur, nxt = nxt, cur

    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        body()
    return graph


def run(s):
    desc = s["desc"]
    if s["kind"] == "step":
        fn = P.swa_decode_step if s["swa"] else P.pbb_decode_step
        fn(desc, s["pos"], s["q"], s["k_new"], s["v_new"], s["k_ring"], s["v_ring"], s["out"],
           workspace=s["workspace"])
        return {"out": s["out"], "k_ring": s["k_ring"], "v_ring": s["v_ring"]}
    if s["kind"] == "graph":
        s["graph"].replay()
        return {"out": s["out"], "k_ring": s["k_ring"], "v_ring": s["v_ring"], "pos": s["pos"]}
    prefill = P.swa_prefill if s["swa"] else P.pbb_prefill
    if s["kind"] == "prefill":
        prefill(desc, s["q"], s["k"], s["v"], s["out"], lse=s["lse"], k_ring=s["k_ring"],
                v_ring=s["v_ring"])
        return {"out": s["out"], "lse": s["lse"], "k_ring": s["k_ring"], "v_ring": s["v_ring"]}
    backward = P.swa_backward if s["swa"] else P.pbb_backward
    prefill(desc, s["q"], s["k"], s["v"], s["out"], lse=s["lse"])
    backward(desc, s["q"], s["k"], s["v"], s["out"], s["dout"], s["lse"], s["dq"], s["dk"],
             s["dv"], workspace=s["workspace"])
    return {"out": s["out"], "lse": s["lse"], "dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}


# ------------------------------------------------------------------------------------------

def _mean_support(c):
    """Mean number of keys of a target at a random position (decode)."""
    if c["window"]:
        w, hi = c["window"], c["pos_hi"]
        return w if hi >= 16 * w else sum(min(t + 1, w) for t in range(hi)) / hi
    return 0.75 * c["block"] + 0.5


def _prompt_pairs(c):
    """(target, key) pairs of one prompt."""
    n = c["n"]
    if c["window"]:
        m = min(n, c["window"])
        return m * (m + 1) // 2 + (n - m) * c["window"]
    h = c["block"] // 2
    full, rest = divmod(n, h)
    # half-block j: r + 1 keys for j = 0, h + r + 1 keys after it (r = phase in the half-block)
    pairs = full * (h * (h + 1) // 2) + max(0, full - 1) * h * h
    return pairs + rest * (rest + 1) // 2 + (rest * h if full > 0 else 0)


def work(case):
    c = dict(case)
    b, hq, hkv, d, n = c["batch"], c["hq"], c["hkv"], c["d"], c["n"]
    u = 4 if c["dtype"] == "f32" else 2
    if c["kind"] in ("step", "graph"):
        sup = _mean_support(c)
        # ring rows of the support but the token's own; q, out; new K/V read and appended; pos
        byte = b * ((sup - 1) * 2 * hkv * d * u + 2 * hq * d * u + 4 * hkv * d * u + 4)
        return {"bytes": c["steps"] * byte, "flops": c["steps"] * b * 4 * d * hq * sup}
    pairs = b * hq * _prompt_pairs(c)
    qb, kb, lse = b * n * hq * d * u, b * n * hkv * d * u, 4 * b * hq * n
    rows = 2 * b * hkv * min(n, c["slots"]) * d * u
    if c["kind"] == "prefill":
        return {"bytes": 2 * qb + 2 * kb + lse + rows, "flops": 4 * d * pairs}
    # forward: q, k, v in, out and lse out; backward: those and dout in, dq, dk, dv out
    return {"bytes": (2 * qb + 2 * kb + lse) + (4 * qb + 4 * kb + lse), "flops": 14 * d * pairs}


def tolerance(case):
    # fp32: 1.8e-7 from the exact result (sums of up to a few thousand products).  bf16: 2e-3 to
    # 3e-3 from it (outputs, and the probabilities that enter the value products, are rounded to
    # 8 bits).
    if case["dtype"] == "f32":
        return {"rel": 1e-6}
    return {"rel": 1e-2}


# ------------------------------------------------------------------------------------------

def _start(c, t):
    """First key of the support of targets ``t``."""
    if c["window"]:
        return (t - c["window"] + 1).clamp(min=0)
    h = c["block"] // 2
    return (h * (torch.div(t, h, rounding_mode="floor") - 1)).clamp(min=0)


def _turn(x, t, base):
    """Rotary embedding of ``x`` [b][heads][d] (float64) at positions ``t`` [b]."""
    d = x.shape[-1]
    c = torch.arange(d // 2, device=x.device, dtype=torch.float64)
    ang = t.double().view(-1, 1, 1) * base ** (-2.0 * c / d)
    lo, hi = x[..., :d // 2], x[..., d // 2:]
    cos, sin = torch.cos(ang), torch.sin(ang)
    return torch.cat((lo * cos - hi * sin, hi * cos + lo * sin), dim=-1)


def _exact_decode(c, s):
    b, hq, hkv, d, slots = c["batch"], c["hq"], c["hkv"], c["d"], c["slots"]
    g = hq // hkv
    kr, vr = s["k_ring"].double(), s["v_ring"].double()
    pos = s["pos"].long()
    outs = torch.empty((c["steps"], b, hq, d), dtype=torch.float64, device=DEV)
    rows = torch.arange(b, device=DEV)
    slot = torch.arange(slots, device=DEV).view(1, -1)
    per = max(1, (1 << 27) // (hkv * slots * d))
    for i in range(c["steps"]):
        q, kn = s["q"][i].double(), s["k_new"][i].double()
        if c["rope"]:
            q, kn = _turn(q, pos, c["rope"]), _turn(kn, pos, c["rope"])
        at = pos % slots
        kr[rows, :, at] = kn
        vr[rows, :, at] = s["v_new"][i].double()
        for b0 in range(0, b, per):
            e = slice(b0, min(b, b0 + per))
            t = pos[e].view(-1, 1)
            held = t - (t - slot) % slots                   # position that each slot holds
            seen = held >= _start(c, t)
            m = e.stop - e.start
            kk = kr[e].reshape(m * hkv, slots, d)
            qq = q[e].reshape(m * hkv, g, d)
            z = torch.bmm(kk, qq.transpose(1, 2).contiguous()).transpose(1, 2) / math.sqrt(d)
            z = z.reshape(m, hkv, g, slots).masked_fill(~seen.view(m, 1, 1, slots), -math.inf)
            p = torch.softmax(z, dim=-1).reshape(m * hkv, g, slots)
            outs[i, e] = torch.bmm(p, vr[e].reshape(m * hkv, slots, d)).reshape(m, hq, d)
        pos = pos + 1
    if c["kind"] == "step":
        return {"out": outs[0], "k_ring": kr, "v_ring": vr}
    return {"out": outs, "k_ring": kr, "v_ring": vr, "pos": None}


def _exact_prompt(c, s):
    """Attention over chunks of targets and the window of keys that they can see, one sequence
    and KV head at a time; for training passes with the gradients."""
    b, hq, hkv, d, n = c["batch"], c["hq"], c["hkv"], c["d"], c["n"]
    g, sc = hq // hkv, 1.0 / math.sqrt(d)
    if c["window"]:
        size, back = min(1024, max(64, c["window"])), c["window"] - 1
    else:
        h = c["block"] // 2
        size, back = h * max(1, -(-64 // h)), h
    size, back = min(size, n), min(back, n)
    nc = -(-n // size)
    dev = s["q"].device
    f64 = dict(dtype=torch.float64, device=dev)
    out = torch.zeros((b, n, hq, d), **f64)
    lse = torch.zeros((b, hq, n), **f64)
    train = c["kind"] == "train"
    if train:
        dq, dk, dv = (torch.zeros(x.shape, **f64) for x in (s["q"], s["k"], s["v"]))
    # chunks of targets at a time, so that scores stay below about a GiB
    per = max(1, (1 << 27) // (size * g * (size + back)))
    for i in range(b):
        for j in range(hkv):
            heads = slice(j * g, (j + 1) * g)
            for c0 in range(0, nc, per):
                m = min(per, nc - c0)
                t = torch.arange(c0 * size, (c0 + m) * size, device=dev).view(m, size)
                key = (torch.arange(size + back, device=dev) - back).view(1, -1) + t[:, :1]
                live, inside = t < n, (key >= 0) & (key < n)
                tc, kc = t.clamp(max=n - 1), key.clamp(0, n - 1)
                k, v = s["k"][i, kc, j].double(), s["v"][i, kc, j].double()
                q = s["q"][i, tc][:, :, heads].double().reshape(m, size * g, d)
                seen = (key.unsqueeze(1) >= _start(c, t).unsqueeze(2)) & \
                    (key.unsqueeze(1) <= t.unsqueeze(2)) & inside.unsqueeze(1)
                seen = (seen | ~live.unsqueeze(2)).repeat_interleave(g, dim=1)
                kt = k.transpose(1, 2).contiguous()
                z = (torch.bmm(q, kt) * sc).masked_fill_(~seen, -math.inf)
                l = torch.logsumexp(z, dim=-1, keepdim=True)
                p = z.sub_(l).exp_()
                o = torch.bmm(p, v)
                ok = live.reshape(-1)
                at = t.reshape(-1)[ok]
                out[i, at, heads] = o.reshape(m * size, g, d)[ok]
                lse[i, heads, at] = l.reshape(m * size, g)[ok].t()
                if not train:
                    continue
                do = s["dout"][i, tc][:, :, heads].double()
                do = (do * live.view(m, size, 1, 1)).reshape(m, size * g, d)
                pt = p.transpose(1, 2).contiguous()
                dvc = torch.bmm(pt, do)
                ds = torch.bmm(do, v.transpose(1, 2).contiguous())
                ds = ds.sub_((do * o).sum(-1, keepdim=True)).mul_(p).mul_(sc)
                dq[i, at, heads] = torch.bmm(ds, k).reshape(m * size, g, d)[ok]
                dkc = torch.bmm(ds.transpose(1, 2).contiguous(), q)
                flat = kc.reshape(-1)
                use = inside.reshape(-1, 1)
                dk[i, :, j].index_add_(0, flat, dkc.reshape(-1, d) * use)
                dv[i, :, j].index_add_(0, flat, dvc.reshape(-1, d) * use)
    if train:
        return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    rings = []
    for name in ("k", "v"):
        ring = torch.zeros((b, hkv, c["slots"], d), **f64)
        at = torch.arange(max(0, n - c["slots"]), n, device=dev)
        ring[:, :, at % c["slots"]] = s[name][:, at].double().transpose(1, 2)
        rings.append(ring)
    return {"out": out, "lse": lse, "k_ring": rings[0], "v_ring": rings[1]}


def exact(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    return _exact_decode(c, s) if c["kind"] in ("step", "graph") else _exact_prompt(c, s)
