"""The decoder-layer calls that a serving program makes, as cases to time.

A case is one call of a public entry point over one batch: ``shape`` names the
model's layer shape, ``chunks`` the prompt chunks as "offset:length" texts
separated by blanks, ``decodes`` the decodes with context lengths drawn from
``ctx_lo`` .. ``ctx_hi``, ``seq`` the KV cache's positions per slot.  ``entry``
is the call: "hybrid" (one layer, at most one chunk), "mixed" (one layer, any
number of chunks) or "step" (``layers`` layers in one call).

Every case returns the output rows and the KV cache that the call updates in
place.
"""
from __future__ import annotations

import math

import torch

from paper_2308_16369_amd import sarathi as S

# Layer shapes of the paper's models (and the tiny one of the smoke test).
SHAPES = {
    "tiny": dict(hidden=256, n_heads=4, head_dim=64, ffn=688, norm="rms", act="swiglu", rope=1, eps=1e-6),
    "llama13b": dict(hidden=5120, n_heads=40, head_dim=128, ffn=13824, norm="rms", act="swiglu", rope=1, eps=1e-6),
    "llama33b": dict(hidden=6656, n_heads=52, head_dim=128, ffn=17920, norm="rms", act="swiglu", rope=1, eps=1e-6),
    "gpt3": dict(hidden=12288, n_heads=96, head_dim=128, ffn=49152, norm="layer", act="gelu", rope=0, eps=1e-5),
}
ROPE_BASE = 10000.0


def _case(name, shape, dtype, entry, chunks, decodes, ctx_lo, ctx_hi, seq, layers=1):
    c = {"shape": shape, "dtype": dtype, "entry": entry, "chunks": chunks, "decodes": decodes, "ctx_lo": ctx_lo,
         "ctx_hi": ctx_hi, "seq": seq, "layers": layers}
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest calls: the fp32 layer of the parity runs, a few dozen rows, all launches and latency.
        _case("tiny_f32_c64_b8", "tiny", "f32", "hybrid", "128:64", 8, 32, 128, 256),
        # A decode-only iteration with few requests (the batch of the per-token table): the weights stream once.
        _case("llama13b_decode_b4", "llama13b", "bf16", "hybrid", "", 4, 1024, 1024, 1088),
        # A decode-only iteration of a full server: long contexts, weights and KV both stream.
        _case("llama13b_decode_b48", "llama13b", "bf16", "hybrid", "", 48, 512, 2048, 2112),
        # The decode-maximal batch of the benchmark.
        _case("llama13b_c256_b64", "llama13b", "bf16", "hybrid", "512:256", 64, 256, 1024, 1088),
        # A whole prompt in one iteration with three decodes beside it: the largest prefill of the 1K study.
        _case("llama13b_c1021_b3", "llama13b", "bf16", "hybrid", "0:1021", 3, 1024, 1024, 1088),
        # Whole prompts of several requests plus every decode (mixed batching), ragged lengths.
        _case("llama13b_mixed3_b15", "llama13b", "bf16", "mixed", "0:683 0:910 0:347", 15, 300, 1000, 1088),
        # A short chunk over a long prefix, and a long one: the two ends of the chunk sizes on the 33B layer.
        _case("llama33b_c128_b32", "llama33b", "bf16", "hybrid", "2048:128", 32, 1024, 3072, 3136),
        _case("llama33b_c512_b32", "llama33b", "bf16", "hybrid", "2048:512", 32, 1024, 3072, 3136),
        # The widest layer: LayerNorm, GELU, no rotary embedding.
        _case("gpt3_c256_b27", "gpt3", "bf16", "hybrid", "1792:256", 27, 1024, 2048, 2112),
        # An iteration of a pipeline stage: several layers in one call, chunk and decodes on a tile multiple.
        _case("llama13b_step4_c239_b17", "llama13b", "bf16", "step", "478:239", 17, 683, 1023, 1088, 4),
        # The fp32 layer at a real width (reference runs beside the bf16 ones).
        _case("llama13b_f32_c128_b16", "llama13b", "f32", "hybrid", "256:128", 16, 256, 1024, 1088),
    ]


def _chunks(case):
    return [tuple(int(v) for v in t.split(":")) for t in case["chunks"].split()]


def draw(rng):
    """One more case of the same ranges, no costlier than the largest listed one."""
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = {d: max(_seconds(c) for c in listed() if c["dtype"] == d) for d in ("bf16", "f32")}
    while True:
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        shape = rng.choice(["tiny", "llama13b"] if dtype == "f32" else ["llama13b", "llama13b", "llama33b", "gpt3"])
        entry = rng.choice(["hybrid", "hybrid", "hybrid", "mixed", "step"])
        kind = rng.choice(["decode", "prefill", "both", "both"])
        seq = 256 if shape == "tiny" else rng.choice([1088, 2112, 3136])
        room = seq - 64
        chunks = []
        if kind != "decode":
            for _ in range(rng.randint(2, 4) if entry == "mixed" else 1):
                length = span(min(17, room), min(2048, room))
                left = room - length
                offset = 0 if rng.random() < 0.4 else rng.randint(0, left)
                chunks.append("%d:%d" % (offset, length))
        decodes = 0 if kind == "prefill" else span(1, 16 if shape == "tiny" else 80)
        if kind != "decode" and dtype == "f32" and sum(int(c.split(":")[1]) for c in chunks) > 160:
            continue
        lo = rng.randint(32, room // 2)
        case = _case(None, shape, dtype, entry, " ".join(chunks), decodes, lo, rng.randint(lo, room), seq,
                     rng.randint(2, 4) if entry == "step" else 1)
        if _seconds(case) <= most[dtype] and _kv_bytes(case) < 6e9:
            return case


def _kv_bytes(case):
    sh = SHAPES[case["shape"]]
    slots = len(_chunks(case)) + case["decodes"]
    return case["layers"] * slots * 2 * sh["n_heads"] * case["seq"] * sh["head_dim"] * (2 if case["dtype"] == "bf16" else 4)


def _seconds(case):
    w = work(case)
    return w["flops"] / (1.6e14 if case["dtype"] == "f32" else 2.5e15) + w["bytes"] / 8e12


def _contexts(case, seed):
    g = torch.Generator().manual_seed(seed * 7 + 1)
    n = len(_chunks(case)) + case["decodes"]
    slots = torch.randperm(n, generator=g).tolist()
    ctx = torch.randint(case["ctx_lo"], case["ctx_hi"] + 1, (case["decodes"],), generator=g).tolist()
    return slots, ctx


def _inputs(case, seed):
    """Tensors of one case on the GPU: weights 0.02 N(0,1), gains around 1, rows and cached K/V N(0,1)."""
    sh = SHAPES[case["shape"]]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    H, nh, hd, F = sh["hidden"], sh["n_heads"], sh["head_dim"], sh["ffn"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(dim, mean=0.0, std=0.02):
        return torch.empty(dim, dtype=dt, device="cuda").normal_(mean, std, generator=g)

    dims = {"w_qkv": (3 * nh * hd, H), "w_o": (H, nh * hd), "w_up": ((2 if sh["act"] == "swiglu" else 1) * F, H),
            "w_down": (H, F)}
    weights = []
    for _ in range(case["layers"]):
        w = {k: normal(d) for k, d in dims.items()}
        for n in ("norm1", "norm2"):
            w[n + "_g"] = normal((H,), 1.0)
            if sh["norm"] == "layer":
                w[n + "_b"] = normal((H,))
        weights.append(w)
    chunks = _chunks(case)
    slots, ctx = _contexts(case, seed)
    T = sum(c[1] for c in chunks) + case["decodes"]
    x = normal((T, H), 0.0, 1.0)
    kv = normal((case["layers"], len(slots), 2, nh, case["seq"], hd), 0.0, 1.0)
    return sh, weights, x, kv, chunks, slots, ctx


def prepare(case, seed):
    sh, weights, x, kv_t, chunks, slots, ctx = _inputs(case, seed)
    cfg = S.make_cfg(hidden=sh["hidden"], n_heads=sh["n_heads"], head_dim=sh["head_dim"], ffn=sh["ffn"],
                     n_layers=case["layers"], norm=S.NORM_RMS if sh["norm"] == "rms" else S.NORM_LAYER,
                     act=S.ACT_SWIGLU if sh["act"] == "swiglu" else S.ACT_GELU, rope=sh["rope"], rope_base=ROPE_BASE,
                     eps=sh["eps"], dtype=S.BF16 if case["dtype"] == "bf16" else S.F32)
    kv = S.sarathi_kv_alloc(cfg, len(slots), case["seq"], kv_t.data_ptr(), kv_t.numel() * kv_t.element_size())
    k = len(chunks)
    wabi = [S.make_weights({n: t.data_ptr() for n, t in w.items()}) for w in weights]
    if case["entry"] == "mixed":
        batch, keep = S.make_mixed_batch([(slots[i], o, n) for i, (o, n) in enumerate(chunks)], slots[k:], ctx)
        ws_bytes = S.sarathi_mixed_workspace_bytes(cfg, x.shape[0], k, case["seq"])
    else:
        slot, (offset, length) = (slots[0], chunks[0]) if chunks else (-1, (0, 0))
        batch, keep = S.make_batch(slot, offset, length, slots[k:], ctx)
        ws_bytes = S.sarathi_workspace_bytes(cfg, x.shape[0], len(ctx), case["seq"])
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    return dict(entry=case["entry"], cfg=cfg, weights=weights, wabi=wabi, kv=kv, kv_t=kv_t, batch=batch, keep=keep,
                x=x, y=torch.empty_like(x), ws=ws, ws_bytes=ws_bytes)


def run(state):
    s = state
    stream = torch.cuda.current_stream().cuda_stream
    args = (s["batch"], s["x"].data_ptr(), s["y"].data_ptr(), s["ws"].data_ptr(), s["ws_bytes"], stream)
    if s["entry"] == "hybrid":
        S.sarathi_hybrid_layer_forward(s["cfg"], s["wabi"][0], s["kv"], 0, *args)
    elif s["entry"] == "mixed":
        S.sarathi_mixed_layer_forward(s["cfg"], s["wabi"][0], s["kv"], 0, *args)
    else:
        S.sarathi_model_step(s["cfg"], s["wabi"], s["kv"], *args)
    return {"y": s["y"], "kv": s["kv_t"]}


def work(case):
    sh = SHAPES[case["shape"]]
    es = 2 if case["dtype"] == "bf16" else 4
    H, QD, F = sh["hidden"], sh["n_heads"] * sh["head_dim"], sh["ffn"]
    chunks = _chunks(case)
    T = sum(n for _, n in chunks) + case["decodes"]
    params = 3 * QD * H + H * QD + (3 if sh["act"] == "swiglu" else 2) * F * H
    ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2          # the mean context
    cached = sum(o for o, _ in chunks) + case["decodes"] * ctx
    pairs = sum(n * o + n * (n + 1) / 2 for o, n in chunks) + case["decodes"] * (ctx + 1)
    L = case["layers"]
    return {"bytes": L * es * (params + 2 * QD * (cached + T)) + 2 * es * T * H,
            "flops": L * (2.0 * T * params + 4.0 * pairs * QD)}


def tolerance(case):
    # About four times the distance of the outputs from the same layer(s) in
    # 64 bits.  Measured, rel / max: fp32 3.2e-6 / 1.7e-5 (sums in another
    # order); one bf16 layer 3.3e-3 .. 5.9e-3 / 3.4e-2 on the 13B shape, up to
    # 7.6e-3 / 4.4e-2 on the wider ones, a step of four 9.0e-3 / 6.0e-2
    # (activations rounded between the ops, and the output).
    if case["dtype"] == "f32":
        return {"rel": 1.3e-5, "max": 8e-5}
    wide = case["shape"] != "llama13b" or case["layers"] > 1
    return {"rel": 0.03 if wide else 0.02, "max": 0.2}


def exact(case, seed):
    """The layer(s) in float64 from the method's definition: every row attends to its own slot's keys up to its
    position."""
    sh, weights, x, kv_t, chunks, slots, ctx = _inputs(case, seed)
    nh, hd, F = sh["n_heads"], sh["head_dim"], sh["ffn"]
    kv = kv_t.double()
    del kv_t
    y = x.double()
    k = len(chunks)
    row_slot, row_pos, spans, r = [], [], [], 0
    for i, (o, n) in enumerate(chunks):
        spans.append((slots[i], r, n, o))
        r += n
    for i, c in enumerate(ctx):
        spans.append((slots[k + i], r + i, 1, c))
    for s, _, n, o in spans:
        row_slot += [s] * n
        row_pos += range(o, o + n)
    row_slot = torch.tensor(row_slot, device="cuda")
    row_pos = torch.tensor(row_pos, device="cuda")

    def norm(v, w, n):
        if sh["norm"] == "rms":
            return v / torch.sqrt((v * v).mean(-1, keepdim=True) + sh["eps"]) * w[n + "_g"].double()
        v = v - v.mean(-1, keepdim=True)
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + sh["eps"]) * w[n + "_g"].double() + w[n + "_b"].double()

    def rotate(v):
        i = torch.arange(hd // 2, device="cuda", dtype=torch.float64)
        ang = row_pos.double()[:, None] * ROPE_BASE ** (-2.0 * i / hd)
        c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
        a, b = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([a * c - b * s, a * s + b * c], -1)

    for layer, w in enumerate(weights):
        T = y.shape[0]
        qkv = norm(y, w, "norm1") @ w["w_qkv"].double().t()
        q, kn, vn = (t.reshape(T, nh, hd) for t in qkv.split(nh * hd, 1))
        if sh["rope"]:
            q, kn = rotate(q), rotate(kn)
        kv[layer, row_slot, 0, :, row_pos] = kn
        kv[layer, row_slot, 1, :, row_pos] = vn
        o = torch.empty_like(q)
        for s, r0, n, off in spans:
            keys, vals = kv[layer, s, 0, :, :off + n], kv[layer, s, 1, :, :off + n]
            mask = torch.arange(off + n, device="cuda")[None] > torch.arange(off, off + n, device="cuda")[:, None]
            for h in range(0, nh, 8):
                sc = torch.matmul(q[r0:r0 + n, h:h + 8].transpose(0, 1).contiguous(),
                                  keys[h:h + 8].transpose(1, 2).contiguous()) / math.sqrt(hd)
                p = torch.softmax(sc.masked_fill(mask, -math.inf), -1)
                o[r0:r0 + n, h:h + 8] = torch.matmul(p, vals[h:h + 8].contiguous()).transpose(0, 1)
        h_ = y + o.reshape(T, nh * hd) @ w["w_o"].double().t()
        z = norm(h_, w, "norm2") @ w["w_up"].double().t()
        if sh["act"] == "swiglu":
            m = torch.nn.functional.silu(z[:, :F]) * z[:, F:]
        else:
            m = torch.nn.functional.gelu(z)
        y = h_ + m @ w["w_down"].double().t()
    return {"y": y, "kv": kv}
