"""Timed cases of the stitched-prefill path, through the C ABI's Python binding.

Every case is one call, or the run of calls, that a serving program makes:

* ``request``           a whole prefill: fused stitch + deviation (when anything
                        is cached), selection, one patch of every layer, then
                        one attention call per layer;
* ``attend_layer``      one layer's attention over the patched cache (what a
                        repair forward repeats);
* ``attend``            patch + attention of a ragged batch in one call;
* ``stitch``            the stitch alone (the probe is off);
* ``stitch_deviation``  the stitch fused with the per-layer deviation;
* ``deviation_topk``    deviation of K and V over all layers, then selection;
* ``select``            selection on given deviations, one set per layer;
* ``store``             new chunks into the pool: RoPE, KIVI quantisation,
                        importance (the encode direction of the stitch).

Inputs are drawn on the GPU from the seed with the shapes and distributions of
``kvb_workload`` (normal values times a log-uniform scale per channel, planted
deviation on 20 % of the cached rows, chunks cached at random positions).
Chunks and fresh tensors are built here in 64-bit torch, so inputs do not
depend on the library.  bfloat16 tensors are passed by address.
"""
import math

import numpy as np
import torch

from paper_2608_21362_amd import kvb

C = 128           # tokens per chunk
MAX_SRC = 32768   # chunks were cached at positions below this
THETA = 1e6
DTYPES = {"bf16": (kvb.KVB_BF16, torch.bfloat16), "f32": (kvb.KVB_F32, torch.float32)}

# Attention shape and cache format of the 36-layer model the benchmark uses
# (16 query heads, 2 kv heads, head size 128, int4 codes in groups of 32).
QWEN = dict(q_heads=16, kv_heads=2, dim=128, bits=4, k_group=32, v_group=32)
# Prompt structure: `prompts` prompts of `chunks` chunks (`ragged` shortens the
# later ones), `sinks` rows before and `tail` rows after the chunks, the leading
# `cached` percent of the chunks found in the pool, `seam` rows recomputed on
# both sides of every chunk boundary, `rho` percent of the cached rows selected.
ONE = dict(prompts=1, ragged=0, sinks=0, tail=0, seam=16, rho=15)


def listed():
    return [
        # the shortest bucket of the request trace: 256 tokens, one of two chunks cached
        dict(QWEN, **{**ONE, "name": "request_256", "op": "request", "layers": 36, "chunks": 2, "cached": 50}),
        # a 1K-2K+ request of the trace: 2432 tokens, 7 of 19 chunks cached
        dict(QWEN, **{**ONE, "name": "request_2432", "op": "request", "layers": 36, "chunks": 19, "cached": 37}),
        # the benchmark's step: 8192 tokens, every chunk cached, 15 % recomputed per layer
        dict(QWEN, **{**ONE, "name": "request_8k", "op": "request", "layers": 36, "chunks": 64, "cached": 100,
                      "seam": 0}),
        # one layer of that step as a repair forward calls it
        dict(QWEN, **{**ONE, "name": "attend_8k", "op": "attend_layer", "out": "bf16", "chunks": 64, "cached": 100,
                      "seam": 0}),
        # the longest prompt: 32K tokens after 4 sink rows, with seam windows
        dict(QWEN, **{**ONE, "name": "attend_32k", "op": "attend_layer", "out": "bf16", "chunks": 256,
                      "cached": 100, "sinks": 4}),
        # a batch of uneven prompts of up to 2K tokens, half of the chunks cached, patch included
        dict(QWEN, **{**ONE, "name": "attend_batch", "op": "attend", "out": "bf16", "layers": 1, "prompts": 16,
                      "ragged": 60, "chunks": 16, "cached": 50, "tail": 23}),
        # a small model (head size 64, 4 query heads) with fp32 output, three short prompts at odd rows
        dict(QWEN, **{**ONE, "name": "attend_d64", "op": "attend", "out": "f32", "layers": 4, "prompts": 3,
                      "ragged": 40, "chunks": 5, "cached": 100, "sinks": 1, "q_heads": 4, "dim": 64}),
        # int8 chunks with whole-chunk statistics, probe off: dequantise and rotate only
        dict(QWEN, **{**ONE, "name": "stitch_int8", "op": "stitch", "out": "bf16", "layers": 36, "chunks": 32,
                      "cached": 100, "bits": 8, "k_group": 128, "v_group": 128}),
        # the fused stitch of a long prompt
        dict(QWEN, **{**ONE, "name": "stitch_deviation_32k", "op": "stitch_deviation", "layers": 36, "chunks": 256,
                      "cached": 100, "sinks": 4}),
        # one selection for all layers from K and V (the two-step form), a ragged batch
        dict(QWEN, **{**ONE, "name": "deviation_topk_batch", "op": "deviation_topk", "layers": 12, "prompts": 8,
                      "ragged": 50, "chunks": 16, "cached": 75, "tail": 5}),
        # per-layer selection of a long prompt
        dict(QWEN, **{**ONE, "name": "select_32k", "op": "select", "layers": 36, "chunks": 256, "cached": 100,
                      "sinks": 4}),
        # the 12 chunks a 2K+ request did not find, stored for the next request, every layer
        dict(QWEN, **{**ONE, "name": "store_chunks", "op": "store", "layers": 36, "chunks": 12, "cached": 100}),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["request", "request", "attend_layer", "attend_layer", "attend", "stitch", "stitch_deviation",
                     "deviation_topk", "select", "store"])
    c = dict(QWEN, **ONE)
    c.update(op=op, seam=rng.choice([0, 16]), sinks=rng.choice([0, 0, 1, 4]), tail=rng.choice([0, 0, 1, 37, 100]),
             cached=rng.randint(30, 100), rho=rng.choice([15, 15, 25]))
    if rng.random() < 0.3:
        g = rng.choice([32, 64])
        c.update(bits=rng.choice([4, 8]), k_group=128 if g == 64 else 32, v_group=g)
    if op == "request":
        # whole requests keep the benchmark model's shape; cold ones recompute every row
        c.update(layers=rng.choice([12, 24, 36]), chunks=_log(rng, 1, 48))
        if rng.random() < 0.25:
            c.update(cached=0)
        if c["cached"] < 70:
            c["chunks"] = min(c["chunks"], 24)
    elif op == "attend_layer":
        c.update(out="bf16", chunks=_log(rng, 1, 160))
        if rng.random() < 0.3:
            c.update(cached=0, chunks=_log(rng, 1, 26))
        elif c["cached"] < 80:
            c["chunks"] = min(c["chunks"], 60)
    elif op == "attend":
        c.update(out=rng.choice(["bf16", "f32"]), layers=rng.choice([1, 2, 4]), prompts=rng.randint(1, 16),
                 ragged=rng.randint(0, 80), chunks=_log(rng, 1, 16))
        c.update(rng.choice([dict(), dict(), dict(q_heads=4, dim=64), dict(q_heads=32, kv_heads=8),
                             dict(q_heads=8, kv_heads=8, dim=64), dict(q_heads=32, kv_heads=1)]))
    elif op in ("stitch", "stitch_deviation"):
        c.update(layers=rng.choice([1, 12, 36]), chunks=_log(rng, 1, 160))
        c.update(rng.choice([dict(), dict(), dict(kv_heads=4, q_heads=32), dict(dim=64)]))
        if c["kv_heads"] == 4:
            c["chunks"] = min(c["chunks"], 80)
        if op == "stitch":
            c["out"] = rng.choice(["bf16", "bf16", "f32"])
    elif op == "deviation_topk":
        c.update(layers=rng.choice([1, 4, 12]), prompts=rng.randint(1, 16), ragged=rng.randint(0, 80),
                 chunks=_log(rng, 1, 24))
        c.update(rng.choice([dict(), dict(kv_heads=8, q_heads=32), dict(dim=64)]))
    elif op == "select":
        c.update(layers=rng.choice([1, 12, 36]), prompts=rng.choice([1, 1, 2, 16]), ragged=rng.randint(0, 80),
                 chunks=_log(rng, 2, 400))
        if c["prompts"] > 2:
            c["chunks"] = min(c["chunks"], 32)
    else:
        c.update(layers=rng.choice([1, 12, 36]), chunks=_log(rng, 1, 40))
        c.update(rng.choice([dict(), dict(), dict(dim=64)]))
    c["v_group"] = min(c["v_group"], c["dim"])
    if c["chunks"] < 4 and op in ("stitch", "stitch_deviation", "store"):
        c["cached"] = 100  # these need a chunk
    while work(c)["flops"] > 1.45e12 or work(c)["bytes"] > 2.2e9:
        c["chunks"] = c["chunks"] * 7 // 8
    return c


# ---- prompt structure -----------------------------------------------------------

def _layout(c):
    """cu_seqlens, first rows and positions of the cached chunks, row flags
    (1 = cached row, 2 = recomputed whatever its deviation), rows to select."""
    cu, dst_row, dst_pos = [0], [], []
    flags, ks = [], []
    for b in range(c["prompts"]):
        n = max(1, round(c["chunks"] * (1 - c["ragged"] / 100 * b / max(1, c["prompts"]))))
        t = c["sinks"] + C * n + c["tail"]
        hits = round(n * c["cached"] / 100)
        f = np.zeros(t, np.uint8)
        for i in range(hits):
            p = c["sinks"] + C * i
            dst_row.append(cu[-1] + p)
            dst_pos.append(p)
            f[p:p + C] = 1
        cand = f == 1
        f[~cand] = 2
        if c["seam"]:
            for p in range(c["sinks"], c["sinks"] + C * n + 1, C):
                if 0 < p < t:
                    f[max(0, p - c["seam"]):min(t, p + c["seam"])] |= 2
        flags.append(f)
        ks.append(c["rho"] * int(cand.sum()) // 100)
        cu.append(cu[-1] + t)
    return (np.array(cu, np.int32), np.array(dst_row, np.int32), np.array(dst_pos, np.int32), np.concatenate(flags),
            np.array(ks, np.int32))


def _bounds(c):
    cu, _, _, flags, ks = _layout(c)
    rows = min(int(ks.sum()) + int((flags & 2).astype(bool).sum()), int(cu[-1]))
    return cu, rows, int(np.diff(cu).max())


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _table(d, pos):
    w = THETA ** (-2.0 * np.arange(d // 2) / d)
    a = np.asarray(pos, np.float64)[:, None] * w
    return np.cos(a).astype(np.float32), np.sin(a).astype(np.float32)


def _rotate(x, cos, sin):
    """Rotate-half RoPE of x [..., n, d] in its own dtype, tables [n, d/2]."""
    h = x.shape[-1] // 2
    lo, hi = x[..., :h], x[..., h:]
    cos, sin = cos.to(x.dtype), sin.to(x.dtype)
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


def _quantise(x, bits, dim, group):
    """KIVI codes (int64), scale and zero (f32) of x f64, groups along `dim`."""
    n = x.shape[dim] // group
    g = x.unflatten(dim, (n, group))
    mn, mx = g.amin(dim + 1, keepdim=True), g.amax(dim + 1, keepdim=True)
    top, r = float((1 << bits) - 1), mx - mn
    code = torch.where(r != 0, torch.round((g - mn) / r * top).clamp(0, top), torch.zeros_like(g))
    return (code.flatten(dim, dim + 1).long(), (r / top).squeeze(dim + 1).float(), mn.squeeze(dim + 1).float())


def _pack(code, bits):
    if bits == 8:
        return code.to(torch.uint8)
    return (code[..., 0::2] | (code[..., 1::2] << 4)).to(torch.uint8)


def _unpack(code, bits):
    if bits == 8:
        return code.double()
    return torch.stack([code & 15, code >> 4], -1).flatten(-2).double()


def _inputs(c, seed):
    """The tensors a program holds before the call, as a dict."""
    g = torch.Generator("cuda").manual_seed(int(seed) & 0x7FFFFFFF)
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 1])
    cu, dst_row, dst_pos, flags, ks = _layout(c)
    H, Hq, d, T, P = c["kv_heads"], c["q_heads"], c["dim"], int(cu[-1]), len(dst_row)
    op, L = c["op"], c.get("layers", 1)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    scale = lambda *s: torch.exp((torch.rand(s, generator=g, device="cuda") * 2 - 1) * math.log(10.0))  # noqa: E731
    i = dict(L=L, H=H, Hq=Hq, d=d, T=T, P=P, cu=_dev(cu), cu_host=cu, flags=_dev(flags), flags_host=flags,
             ks=_dev(np.tile(ks, (L, 1))), ks_host=ks)
    if op == "select":
        # most rows deviate a little, the planted ones a hundred times more
        x = normal(L, T).abs() * 1e-4
        i["delta"] = x * torch.where(torch.rand((L, T), generator=g, device="cuda") < 0.2, 100.0, 1.0)
        return i
    src = rng.integers(0, MAX_SRC, P).astype(np.int32)
    if op == "store":
        i["k_raw"] = normal(P, L, H, C, d) * scale(1, L, H, 1, d)
        # the program holds the values in the type it has the keys rotated into
        i["v_raw"] = (normal(P, L, H, C, d) * scale(1, L, H, 1, d)).double()
        cos, sin = _table(d, np.arange(MAX_SRC + C))
        i.update(cos=_dev(cos), sin=_dev(sin), u=_dev(np.arange(C, dtype=np.int32)),
                 src=_dev(np.repeat(src, L * H).astype(np.int32)))
        return i
    pos = np.concatenate([np.arange(n) for n in np.diff(cu)])
    pc, ps = (_dev(t) for t in _table(d, pos))
    need_pool = op in ("request", "stitch", "stitch_deviation") and P
    zk, zv = normal(L, H, T, d), normal(L, H, T, d)
    sk, sv = scale(L, H, 1, d), scale(L, H, 1, d)
    if need_pool:
        take = _dev((dst_row[:, None] + np.arange(C)).astype(np.int64)).flatten()
        uc, us = (_dev(t).unflatten(0, (P, 1, 1, C)) for t in _table(d, (src[:, None] + np.arange(C)).flatten()))
        chunk = lambda z, s: (z * s)[:, :, take].double().unflatten(2, (P, C)).permute(2, 0, 1, 3, 4)  # noqa: E731
        code, i["ks_scale"], i["ks_zero"] = _quantise(_rotate(chunk(zk, sk), uc, us), c["bits"], 3, c["k_group"])
        i["k_codes"] = _pack(code, c["bits"])
        code, i["vs_scale"], i["vs_zero"] = _quantise(chunk(zv, sv), c["bits"], 4, c["v_group"])
        i["v_codes"] = _pack(code, c["bits"])
        del code
        for k in ("k_codes", "v_codes", "ks_scale", "ks_zero", "vs_scale", "vs_zero"):
            i[k] = i[k].contiguous()
        rc, rs = _table(d, dst_pos.astype(np.int64) - src)
        i.update(rope_cos=_dev(rc), rope_sin=_dev(rs),
                 chunks=_dev(np.stack([np.arange(P), src, dst_row, dst_pos], 1).astype(np.int32)))
    cand = _dev((flags & 1).astype(bool))
    noisy = (torch.rand((L, 1, T, 1), generator=g, device="cuda") < 0.2) & cand[:, None]
    i["k_fresh"] = _rotate((zk + 0.1 * noisy * normal(L, H, T, d)) * sk, pc, ps).bfloat16()
    i["v_fresh"] = ((zv + 0.1 * noisy * normal(L, H, T, d)) * sv).bfloat16()
    if op in ("attend_layer", "attend", "deviation_topk"):
        # a cache the stitch has filled: the values without the planted part, with a quantisation-sized error
        err = lambda z: z + 0.05 * cand[:, None] * normal(L, H, T, d)  # noqa: E731
        i["k_cache"] = torch.where(cand[:, None], _rotate(err(zk) * sk, pc, ps).bfloat16(), i["k_fresh"])
        i["v_cache"] = torch.where(cand[:, None], (err(zv) * sv).bfloat16(), i["v_fresh"])
    elif op == "request":
        hole = lambda x: torch.where(cand[:, None], torch.zeros_like(x), x)  # noqa: E731
        i["k_cache"], i["v_cache"] = hole(i["k_fresh"]), hole(i["v_fresh"])
    del zk, zv
    if op in ("request", "attend_layer", "attend"):
        i["q"] = torch.empty((L, T, Hq, d), dtype=torch.bfloat16, device="cuda")
        for l in range(L):
            q = normal(Hq, T, d) * scale(Hq, 1, d)
            i["q"][l] = _rotate(q, pc, ps).bfloat16().transpose(0, 1)
    if op in ("attend_layer", "attend"):
        # rows as the selection leaves them: the forced ones and a random rest
        rows, cr = np.full((L, T), -1, np.int32), np.zeros((L, len(cu)), np.int32)
        for l in range(L):
            n = 0
            for b in range(len(cu) - 1):
                f = flags[cu[b]:cu[b + 1]]
                on = (f & 2) != 0
                can = np.nonzero(f & 1)[0]
                on[rng.choice(can, ks[b], replace=False) if ks[b] else []] = True
                r = np.nonzero(on)[0] + cu[b]
                rows[l, n:n + len(r)] = r
                n += len(r)
                cr[l, b + 1] = n
        i.update(rows=_dev(rows), cu_rows=_dev(cr))
    return i


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    L, H, Hq, d, T, P = (s[k] for k in ("L", "H", "Hq", "d", "T", "P"))
    B = c["prompts"]
    new = lambda *shape, dtype=torch.bfloat16: torch.zeros(shape, dtype=dtype, device="cuda")  # noqa: E731
    s["case"], s["B"] = c, B
    _, s["max_rows"], s["max_seq"] = _bounds(c)
    s["pool"] = kvb.pool_layout(L, H, d, c["bits"], c["k_group"], c["v_group"])
    s["out_dtype"], torch_out = DTYPES[c.get("out", "bf16")]
    op = c["op"]
    if op in ("request", "select", "deviation_topk"):
        n = 1 if op == "deviation_topk" else L
        s["rows"] = torch.full((n, T), -1, dtype=torch.int32, device="cuda")
        s["cu_rows"] = new(n, B + 1, dtype=torch.int32)
        s["ws_bytes"] = kvb.kvb_select_workspace_bytes(n, T, B)
        s["ws"] = new(max(16, s["ws_bytes"]), dtype=torch.uint8)
    if op in ("request", "stitch_deviation", "deviation_topk"):
        s["delta"] = new(1 if op == "deviation_topk" else L, T, dtype=torch.float32)
    if op in ("stitch", "stitch_deviation"):
        s["k_cache"], s["v_cache"] = new(L, H, T, d, dtype=torch_out), new(L, H, T, d, dtype=torch_out)
    if op in ("request", "attend_layer"):
        size = (Hq, H, d, T, B, s["max_seq"], s["max_rows"])
        s["v16"] = new(L, H, T, d, dtype=torch.float16)
        s["plans_bytes"] = kvb.kvb_attn_plans_bytes(L, *size)
        s["plans"] = new(max(16, s["plans_bytes"]), dtype=torch.uint8)
        s["attn_bytes"] = kvb.kvb_sparse_attn_workspace_bytes(1, *size, 1)
    if op == "attend":
        s["attn_bytes"] = kvb.kvb_sparse_attn_workspace_bytes(L, Hq, H, d, T, B, s["max_seq"], s["max_rows"], 0)
    if "attn_bytes" in s:
        s["attn_ws"] = new(s["attn_bytes"], dtype=torch.uint8)
        s["status"] = new(4, dtype=torch.int32)
        s["res"] = new(L, T, Hq, d, dtype=torch_out)
    if op == "attend_layer":
        _patch(s)
    if op == "store":
        s["k_rot"] = new(P, L, H, C, d, dtype=torch.float64)
        s["codes"] = [new(P, L, H, C, d * c["bits"] // 8, dtype=torch.uint8) for _ in range(2)]
        s["stats"] = ([new(P, L, H, C // c["k_group"], d, dtype=torch.float32) for _ in range(2)]
                      + [new(P, L, H, C, d // c["v_group"], dtype=torch.float32) for _ in range(2)])
        s["importance"] = new(P, dtype=torch.float64)
    return s


def _patch(s):
    kvb.kvb_patch(s["L"], s["Hq"], s["H"], s["d"], s["T"], s["cu"], s["B"], s["max_seq"], s["rows"], s["cu_rows"], 1,
                  s["max_rows"], s["k_fresh"], s["v_fresh"], s["k_cache"], s["v_cache"], s["v16"], s["plans"],
                  s["plans_bytes"], v_status=s["status"])


def _attend_layer(s, l):
    kvb.kvb_sparse_attn_layer(l, s["L"], s["Hq"], s["H"], s["d"], s["T"], s["cu"], s["B"], s["max_seq"], s["rows"],
                              s["cu_rows"], 1, s["max_rows"], s["q"], s["k_cache"], s["v16"], s["plans"],
                              s["plans_bytes"], s["d"] ** -0.5, s["out_dtype"], s["res"], s["attn_ws"],
                              s["attn_bytes"])


def _stitch_deviation(s):
    kvb.kvb_stitch_deviation(s["pool"], s["P"], s["k_codes"], s["ks_scale"], s["ks_zero"], s["v_codes"],
                             s["vs_scale"], s["vs_zero"], s["chunks"], s["P"], s["rope_cos"], s["rope_sin"], s["T"],
                             s["k_cache"], s["v_cache"], s["k_fresh"], s["delta"])


def _select(s):
    kvb.kvb_select(s["L"], s["T"], s["cu"], s["B"], s["delta"], s["flags"], s["ks"], s["rows"], s["cu_rows"],
                   s["ws"], s["ws_bytes"])


def run(s):
    op = s["case"]["op"]
    if op == "request":
        if s["P"]:
            _stitch_deviation(s)
        _select(s)
        _patch(s)
        for l in range(s["L"]):
            _attend_layer(s, l)
        return {"k": s["k_cache"], "v": s["v_cache"], "v16": s["v16"], "delta": s["delta"], "rows": s["rows"],
                "cu_rows": s["cu_rows"], "out": s["res"]}
    if op == "attend_layer":
        _attend_layer(s, 0)
        return {"out": s["res"]}
    if op == "attend":
        kvb.kvb_sparse_attn(s["L"], s["Hq"], s["H"], s["d"], s["T"], s["cu"], s["B"], s["max_seq"], s["rows"],
                            s["cu_rows"], 1, s["max_rows"], s["q"], s["k_fresh"], s["v_fresh"], s["k_cache"],
                            s["v_cache"], None, s["d"] ** -0.5, s["out_dtype"], s["res"], s["attn_ws"],
                            s["attn_bytes"], v_status=s["status"])
        return {"k": s["k_cache"], "v": s["v_cache"], "out": s["res"]}
    if op == "stitch":
        kvb.kvb_stitch(s["pool"], s["P"], s["k_codes"], s["ks_scale"], s["ks_zero"], s["v_codes"], s["vs_scale"],
                       s["vs_zero"], s["chunks"], s["P"], s["rope_cos"], s["rope_sin"], s["T"], s["out_dtype"],
                       s["k_cache"], s["v_cache"])
        return {"k": s["k_cache"], "v": s["v_cache"]}
    if op == "stitch_deviation":
        _stitch_deviation(s)
        return {"k": s["k_cache"], "v": s["v_cache"], "delta": s["delta"]}
    if op == "deviation_topk":
        kvb.kvb_deviation_topk(s["L"], s["H"], s["d"], s["T"], s["cu"], s["B"], s["k_cache"], s["k_fresh"],
                               s["v_cache"], s["v_fresh"], 0, s["flags"], s["ks"], s["delta"], s["rows"],
                               s["cu_rows"], s["ws"], s["ws_bytes"])
        return {"delta": s["delta"], "rows": s["rows"], "cu_rows": s["cu_rows"]}
    if op == "select":
        _select(s)
        return {"rows": s["rows"], "cu_rows": s["cu_rows"]}
    L, H, d, P = s["L"], s["H"], s["d"], s["P"]
    kvb.kvb_rope_rows(d, P * L * H, C, 1, s["k_raw"], s["u"], s["src"], s["cos"], s["sin"], MAX_SRC + C, kvb.KVB_F64,
                      s["k_rot"])
    kvb.kvb_kivi_quantize(s["pool"], P, 0, L, kvb.KVB_F64, s["k_rot"], s["v_raw"], s["codes"][0], s["stats"][0],
                          s["stats"][1], s["codes"][1], s["stats"][2], s["stats"][3])
    s["importance"].zero_()  # new chunks start from nothing
    kvb.kvb_chunk_importance(s["pool"], P, L, kvb.KVB_F64, s["k_rot"], s["importance"])
    return {"k_rot": s["k_rot"], "codes": s["codes"], "stats": s["stats"], "importance": s["importance"]}


# ---- what a pass cannot do without ------------------------------------------------

def work(case):
    c = case
    cu, _, _, flags, ks = _layout(c)
    L, H, Hq, d, T = c.get("layers", 1), c["kv_heads"], c["q_heads"], c["dim"], int(cu[-1])
    cand, forced = int((flags & 1).sum()), int(((flags & 2) != 0).sum())
    both = int((flags == 3).sum())
    pick = int(ks.sum()) * (1 - both / cand) if cand else 0
    rows = forced + pick                      # expected size of a set
    row = H * d * 2                           # bytes of one tensor's bf16 row, all kv heads
    stat = 2 * 4 * (d / c["k_group"] + d / c["v_group"])
    pool = cand * H * (2 * d * c["bits"] / 8 + stat)
    op = c["op"]
    bytes_, flops = 0.0, 0.0
    if op in ("request", "stitch", "stitch_deviation"):
        bytes_ += L * (pool + 2 * cand * row * (2 if c.get("out") == "f32" else 1))
    if op == "stitch_deviation" or (op == "request" and cand):
        bytes_ += L * cand * (row + 4)
    if op == "deviation_topk":
        bytes_ += L * 4 * T * row + 4 * T
    if op in ("request", "select", "deviation_topk"):
        bytes_ += (1 if op == "deviation_topk" else L) * (4 * T + 4 * rows) + T
    if op in ("request", "attend"):
        bytes_ += L * 4 * rows * row          # patched rows, read and written
    if op == "request":
        bytes_ += L * T * row                 # the fp16 copy of V
    if op in ("request", "attend_layer", "attend"):
        out = 4 if c.get("out") == "f32" else 2
        bytes_ += L * (rows * Hq * d * (2 + out) + 2 * T * row)
        for b in range(len(cu) - 1):
            f = flags[cu[b]:cu[b + 1]]
            at = np.arange(1, len(f) + 1, dtype=np.float64)
            can = ((f & 1) != 0) & ((f & 2) == 0)
            n = max(1, int((f & 1).sum()))
            flops += L * 4.0 * d * Hq * (at[(f & 2) != 0].sum() + at[can].sum() * ks[b] / n)
    if op == "store":
        n = len(_layout(c)[1]) * L * H * C * d
        bytes_ += n * (4 + 8) + n * 8 + 2 * n * c["bits"] / 8 + n / d * stat
    return {"bytes": float(bytes_), "flops": float(flops)}


def tolerance(case):
    op = case["op"]
    if op in ("stitch", "select"):
        return "exact"                        # defined to the bit: one rounding of a 64-bit value; whole numbers
    if op == "store":
        return {"rel": 1e-12, "max": 1e-11}   # 64-bit sums in another order; codes are the same
    if op in ("stitch_deviation", "deviation_topk"):
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-4}  # fp32 roundings of 64-bit sums
    if case.get("out") == "f32":
        return {"rel": 8e-4, "max": 3e-2}     # fp16 probabilities
    # fp16 probabilities and a bf16 result; a tie at the last selected row
    return {"rel": 7e-3, "max": 1e-1, "differ": 1e-4}


# ---- the same in 64 bits ------------------------------------------------------------

def _stitched(c, i, to):
    """K and V rows of the cached chunks, f64 values rounded to `to`, into zeros or the cache."""
    L, H, d, T, P = (i[k] for k in ("L", "H", "d", "T", "P"))
    k = i["k_cache"].clone() if "k_cache" in i else torch.zeros((L, H, T, d), dtype=to, device="cuda")
    v = i["v_cache"].clone() if "v_cache" in i else torch.zeros((L, H, T, d), dtype=to, device="cuda")
    for p in range(P):
        x = _unpack(i["k_codes"][p], c["bits"]).unflatten(2, (C // c["k_group"], c["k_group"]))
        x = (x * i["ks_scale"][p].double()[:, :, :, None] + i["ks_zero"][p].double()[:, :, :, None]).flatten(2, 3)
        x = _rotate(x, i["rope_cos"][p][None].double(), i["rope_sin"][p][None].double())
        y = _unpack(i["v_codes"][p], c["bits"]).unflatten(3, (d // c["v_group"], c["v_group"]))
        y = (y * i["vs_scale"][p].double()[..., None] + i["vs_zero"][p].double()[..., None]).flatten(3, 4)
        r = int(i["chunks"][p, 2])
        k[:, :, r:r + C], v[:, :, r:r + C] = x.float().to(to), y.float().to(to)
    return k, v


def _cosine_loss(a, b):
    """1 - cosine of the rows of a and b, [L, H, T], in 64 bits."""
    out = []
    for l in range(a.shape[0]):
        x, y = a[l].double(), b[l].double()
        den = (x * x).sum(-1) * (y * y).sum(-1)
        none = ((x == 0).all(-1) & (y == 0).all(-1)).double()
        out.append(1.0 - torch.where(den == 0, none, (x * y).sum(-1) / den.clamp_min(1e-300).sqrt()))
    return torch.stack(out)


def _selected(c, i, delta):
    """Row lists by sorting each prompt's cached rows: largest first, lower row first."""
    n, T, cu = delta.shape[0], i["T"], i["cu_host"]
    rows = torch.full((n, T), -1, dtype=torch.int32, device="cuda")
    cr = torch.zeros((n, len(cu)), dtype=torch.int32, device="cuda")
    for s in range(n):
        at = 0
        for b in range(len(cu) - 1):
            f = i["flags"][int(cu[b]):int(cu[b + 1])]
            on = (f & 2) != 0
            can = torch.nonzero(f & 1).flatten()
            x = delta[s, int(cu[b]):int(cu[b + 1])][can]
            on[can[torch.sort(x, descending=True, stable=True).indices[:int(i["ks_host"][b])]]] = True
            r = torch.nonzero(on).flatten() + int(cu[b])
            rows[s, at:at + len(r)] = r.int()
            at += len(r)
            cr[s, b + 1] = at
    return rows, cr


def _attention(i, rows, cr, k, v):
    """Causal attention of the listed rows over the patched cache, zeros elsewhere."""
    L, H, Hq, d, T, cu = (i[n] for n in ("L", "H", "Hq", "d", "T", "cu_host"))
    out = torch.zeros((L, T, Hq, d), dtype=torch.float64, device="cuda")
    G = Hq // H
    for l in range(L):
        lim = cr[l].tolist()
        for b in range(len(cu) - 1):
            t = rows[l, lim[b]:lim[b + 1]].long()
            lo = int(cu[b])
            for part in t.split(1024):
                hi = int(part.max()) + 1 if len(part) else lo
                mask = torch.arange(lo, hi, device="cuda")[None, None] > part[:, None, None]
                for h in range(H):
                    q = i["q"][l, part, h * G:(h + 1) * G].double()
                    s = (q.flatten(0, 1) @ k[l, h, lo:hi].double().T.contiguous() * d ** -0.5).unflatten(0, (-1, G))
                    s = s.masked_fill(mask, -math.inf).softmax(-1)
                    out[l, part, h * G:(h + 1) * G] = (s.flatten(0, 1) @ v[l, h, lo:hi].double()).unflatten(0, (-1, G))
    return out


def exact(case, seed):
    c, i = case, _inputs(case, seed)
    op, L = c["op"], i["L"]
    if op == "select":
        rows, cr = _selected(c, i, i["delta"])
        return {"rows": rows, "cu_rows": cr}
    if op == "store":
        cos = i["cos"].double()[i["u"].long() + i["src"].long()[:, None]].unflatten(0, (i["P"], L, i["H"]))
        sin = i["sin"].double()[i["u"].long() + i["src"].long()[:, None]].unflatten(0, (i["P"], L, i["H"]))
        k = _rotate(i["k_raw"].double(), cos, sin)
        kc, k_scale, k_zero = _quantise(k, c["bits"], 3, c["k_group"])
        vc, v_scale, v_zero = _quantise(i["v_raw"], c["bits"], 4, c["v_group"])
        return {"k_rot": k, "codes": [_pack(kc, c["bits"]), _pack(vc, c["bits"])],
                "stats": [t.double() for t in (k_scale, k_zero, v_scale, v_zero)],
                "importance": k.square().sum(-1).sqrt().mean((1, 2, 3))}
    if op in ("stitch", "stitch_deviation", "request"):
        k, v = _stitched(c, i, DTYPES[c.get("out", "bf16")][1]) if i["P"] else (i["k_cache"], i["v_cache"])
        if op == "stitch":
            return {"k": k.double(), "v": v.double()}
        cand = (i["flags"] & 1).double()
        delta = _cosine_loss(k, i["k_fresh"]).mean(1) * cand
        if op == "stitch_deviation":
            return {"k": k.double(), "v": v.double(), "delta": delta}
        rows, cr = _selected(c, i, delta.float())
    elif op == "deviation_topk":
        delta = ((_cosine_loss(i["k_cache"], i["k_fresh"]) + _cosine_loss(i["v_cache"], i["v_fresh"])) / 2).mean((0, 1))
        rows, cr = _selected(c, i, delta.float()[None])
        return {"delta": delta[None], "rows": rows, "cu_rows": cr}
    else:
        rows, cr, k, v = i["rows"], i["cu_rows"], i["k_cache"], i["v_cache"]
    for l in range(L):
        r = rows[l, :int(cr[l, -1])].long()
        k[l][:, r], v[l][:, r] = i["k_fresh"][l][:, r], i["v_fresh"][l][:, r]
    out = _attention(i, rows, cr, k, v)
    if op == "attend_layer":
        return {"out": out}
    if op == "attend":
        return {"k": k.double(), "v": v.double(), "out": out}
    return {"k": k.double(), "v": v.double(), "v16": v.double(), "delta": delta if i["P"] else delta * 0,
            "rows": rows, "cu_rows": cr, "out": out}
