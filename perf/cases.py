"""Performance cases: the calls of a DeepSeek-V3 MLA decode that a program using this library makes,
through the Python binding, over the range of sizes it meets.

Seven kinds of case (the field ``kind``):

* ``gemv``       nmm_gemv, y = x . W with W row-major [K, N]: 1 to 32 rows, bf16 or fp16
* ``linear``     nmm_gemv_nt, the same product with a torch Linear weight [N, K]
* ``heads``      nmm_batched_gemv_bf16, the per-head absorbed products, 1 to 16 rows a head
* ``entry``      nmm_mla_kv_update, MatMul 2 with RMSNorm, RoPE and the latent-cache append
* ``attention``  nmm_latent_attention_bf16 over a latent cache
* ``step``       PreparedStep, one decode step with an independent attention beside the chain
* ``layer``      one whole MLA decode layer in its dependency order: PreparedQueryPath, attention
                 over the cache with this token's row, W_UV per head, W_O

Inputs are standard normal tokens and weights drawn N(0, 1/K), as the tests draw them.
"""
import math

import torch

import paper_2609_16009_amd as nmm

# DeepSeek-V3's MLA dimensions
HIDDEN, Q_LORA, KV_LORA, ROPE, NOPE, V_HEAD = 7168, 1536, 512, 64, 128, 128
DOWN = Q_LORA + KV_LORA + ROPE
QK = NOPE + ROPE
SCALE = 1.0 / math.sqrt(QK)
EPS, THETA = 1e-6, 10000.0
MAX_WEIGHT = 16384 * 7168          # elements of the largest weight (W_O)
MAX_SCORES = 128 * 65536           # heads x positions of the largest attention


def listed():
    return [
        # the smallest call: a 512 x 512 fp16 projection of one token, all launch latency
        {"name": "gemv_512_fp16", "kind": "gemv", "M": 1, "K": 512, "N": 512, "fp16": True},
        # the paper's MatMul 2 and its vector work, once per token and layer
        {"name": "entry_7168x576", "kind": "entry", "hidden": HIDDEN, "kv_lora": KV_LORA, "rope": ROPE, "rows": 4096,
         "position": 4000},
        # the fused down-projection W_DQ | W_DKV | W_KR of one token
        {"name": "gemv_down", "kind": "gemv", "M": 1, "K": HIDDEN, "N": DOWN, "fp16": False},
        # the output projection, the largest weight of the layer, for one token
        {"name": "gemv_w_o", "kind": "gemv", "M": 1, "K": 16384, "N": HIDDEN, "fp16": False},
        # W_UQ for eight tokens (speculative or small-batch decode), on the matrix cores
        {"name": "gemv_w_uq_8", "kind": "gemv", "M": 8, "K": Q_LORA, "N": 24576, "fp16": False},
        # a ragged fp16 product: no size a multiple of a tile
        {"name": "gemv_ragged_5", "kind": "gemv", "M": 5, "K": 4099, "N": 5003, "fp16": True},
        # the output projection kept as a torch Linear weight, for sixteen tokens
        {"name": "linear_w_o_16", "kind": "linear", "M": 16, "K": 16384, "N": HIDDEN, "fp16": False},
        # the absorbed per-head W_UK for four tokens of every head
        {"name": "heads_w_uk_4", "kind": "heads", "B": 128, "M": 4, "K": NOPE, "N": KV_LORA},
        # attention of one eighth of the heads (a tensor-parallel shard) over an odd cache length
        {"name": "attention_16x4097", "kind": "attention", "heads": 16, "seq": 4097, "d_qk": 576, "d_v": 512},
        # attention of all heads over a long context
        {"name": "attention_128x65536", "kind": "attention", "heads": 128, "seq": 65536, "d_qk": 576, "d_v": 512},
        # the decode step with attention beside the chain, all heads, 4096 positions
        {"name": "step_128x4096", "kind": "step", "heads": 128, "seq": 4096},
        # a whole MLA decode layer in dependency order on a quarter of the heads
        {"name": "layer_32x4096", "kind": "layer", "heads": 32, "seq": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size between lo and hi over its logarithm: half of them any number, half a multiple of 64."""
    v = _log(rng, lo, hi)
    return v if rng.random() < 0.5 else max(lo, v // 64 * 64)


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "linear", "linear", "heads", "heads", "entry", "attention", "attention",
                       "step", "layer"])
    if kind in ("gemv", "linear"):
        M = 1 if rng.random() < 0.3 else _log(rng, 1, 32)
        K = _size(rng, 512, 16384)
        N = _size(rng, 512, min(24576, MAX_WEIGHT // K))
        return {"kind": kind, "M": M, "K": K, "N": N, "fp16": rng.random() < 0.3}
    if kind == "heads":
        up = rng.random() < 0.5
        k, n = (_size(rng, 64, 256), _size(rng, 256, 1024)) if up else (_size(rng, 256, 1024), _size(rng, 64, 256))
        return {"kind": kind, "B": _log(rng, 8, 128), "M": _log(rng, 1, 16), "K": k, "N": n}
    if kind == "entry":
        rows = _log(rng, 512, 16384)
        return {"kind": kind, "hidden": _size(rng, 1024, 8192), "kv_lora": rng.choice([256, 384, 512]),
                "rope": rng.choice([32, 64]), "rows": rows, "position": rng.randrange(rows)}
    if kind == "attention":
        heads = _log(rng, 8, 128)
        d_qk, d_v = rng.choice([(576, 512), (576, 512), (576, 512), (320, 256)])
        return {"kind": kind, "heads": heads, "seq": _size(rng, 64, min(131072, MAX_SCORES // heads)), "d_qk": d_qk,
                "d_v": d_v}
    return {"kind": kind, "heads": rng.choice([8, 16, 32, 64, 128]) if rng.random() < 0.7 else _log(rng, 8, 128),
            "seq": _size(rng, 256, 4096 if kind == "step" else 8192)}


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _normal(g, shape, sigma=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * sigma).to(dtype)


def _rows(g, rows, cols, sigma=1.0, dtype=torch.bfloat16, lead=()):
    """A [..., rows, cols] matrix whose rows are padded to a multiple of 8 elements (whole 16-byte pieces)."""
    ld = (cols + 7) // 8 * 8
    return _normal(g, (*lead, rows, ld), sigma, dtype)


def _f32(*shape):
    return torch.zeros(shape, dtype=torch.float32, device="cuda")


def _bf16(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16, device="cuda")


def _layer_inputs(g, heads, chain):
    """The token, the weights of one MLA layer and the buffers of its intermediates."""
    b = {"x": _normal(g, (HIDDEN,)),
         "w_down": _normal(g, (HIDDEN, DOWN), HIDDEN ** -0.5),
         "w_uq": _normal(g, (Q_LORA, heads * QK), Q_LORA ** -0.5),
         "w_uk": _normal(g, (heads, NOPE, KV_LORA), NOPE ** -0.5),
         "w_uv": _normal(g, (heads, KV_LORA, V_HEAD), KV_LORA ** -0.5),
         "w_o": _normal(g, (heads * V_HEAD, HIDDEN), (heads * V_HEAD) ** -0.5),
         "down_f32": _f32(DOWN), "cq_bf16": _bf16(Q_LORA), "q_f32": _f32(heads * QK)}
    if chain:
        b.update(lat_f32=_f32(heads * KV_LORA), o_f32=_f32(heads * V_HEAD), y=_f32(HIDDEN),
                 qnope_bf16=_bf16(heads * NOPE), lat_bf16=_bf16(heads * KV_LORA), o_bf16=_bf16(heads * V_HEAD))
    else:
        b.update(kv_gamma=(1.0 + 0.1 * torch.randn(KV_LORA, generator=g, device="cuda")).to(torch.bfloat16),
                 q_bf16=_bf16(heads * QK), qlat_f32=_f32(heads * KV_LORA), query=_bf16(heads, KV_LORA + ROPE))
    return b


def _dims(heads):
    return dict(hidden=HIDDEN, q_lora=Q_LORA, kv_lora=KV_LORA, rope=ROPE, heads=heads, nope=NOPE, v_head=V_HEAD)


def prepare(case, seed):
    g = _gen(seed)
    s = {"case": case}
    kind = case["kind"]
    if kind in ("gemv", "linear"):
        M, K, N = case["M"], case["K"], case["N"]
        dt = torch.float16 if case["fp16"] else torch.bfloat16
        s["x"] = _rows(g, M, K, 1.0, dt)
        s["W"] = _rows(g, K, N, K ** -0.5, dt) if kind == "gemv" else _rows(g, N, K, K ** -0.5, dt)
        s["y"] = _f32(M, N)
    elif kind == "heads":
        B, M, K, N = case["B"], case["M"], case["K"], case["N"]
        s["x"] = _rows(g, M, K, 1.0, lead=(B,))
        s["W"] = _rows(g, K, N, K ** -0.5, lead=(B,))
        s["y"], s["yb"] = _f32(B, M, N), _bf16(B, M, N)
    elif kind == "entry":
        n = case["kv_lora"] + case["rope"]
        s["h"] = _rows(g, 1, case["hidden"])[0]
        s["w"] = _rows(g, case["hidden"], n, case["hidden"] ** -0.5)
        s["gamma"] = (1.0 + 0.1 * torch.randn(case["kv_lora"], generator=g, device="cuda")).to(torch.bfloat16)
        s["mm"] = _f32(n)
        s["cache"] = _normal(g, (case["rows"], n))
        s["entry"] = s["cache"][case["position"]]
    elif kind == "attention":
        s["q"] = _normal(g, (case["heads"], case["d_qk"]))
        s["kv"] = _normal(g, (case["seq"], max(case["d_qk"], case["d_v"])))
        s["out"], s["outb"] = _f32(case["heads"], case["d_v"]), _bf16(case["heads"], case["d_v"])
        s["scale"] = SCALE if case["d_qk"] == 576 else case["d_qk"] ** -0.5
    elif kind == "step":
        heads = case["heads"]
        b = _layer_inputs(g, heads, True)
        a = dict(q=_normal(g, (heads, KV_LORA + ROPE)), kv=_normal(g, (case["seq"], KV_LORA + ROPE)),
                 out=_f32(heads, KV_LORA), out_bf16=_bf16(heads, KV_LORA), scale=SCALE)
        s["step"] = nmm.PreparedStep(_dims(heads), b, a)
        s["outs"] = {"down": b["down_f32"], "q": b["q_f32"], "lat": b["lat_f32"], "o": b["o_f32"], "y": b["y"],
                     "out": a["out"], "out_bf16": a["out_bf16"]}
    else:
        heads, seq = case["heads"], case["seq"]
        b = _layer_inputs(g, heads, False)
        b["kv_cache"] = _normal(g, (seq + 1, KV_LORA + ROPE))
        s["b"] = b
        s["path"] = nmm.PreparedQueryPath(_dims(heads), b, eps=EPS, theta=THETA, position=seq)
        s["att"], s["att_b"] = _f32(heads, KV_LORA), _bf16(heads, KV_LORA)
        s["att_rows"] = s["att_b"].view(heads, 1, KV_LORA)
        s["o"], s["o_b"] = _f32(heads, 1, V_HEAD), _bf16(heads, 1, V_HEAD)
        s["o_row"] = s["o_b"].view(1, heads * V_HEAD)
        s["y"] = _f32(1, HIDDEN)
        s["outs"] = {"down": b["down_f32"], "q": b["q_f32"], "qlat": b["qlat_f32"], "query": b["query"],
                     "entry": b["kv_cache"][seq], "att": s["att"], "o": s["o"], "y": s["y"]}
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "gemv":
        return nmm.nmm_gemv(s["x"], s["W"], s["y"], N=case["N"])
    if kind == "linear":
        return nmm.nmm_gemv_nt(s["x"], s["W"], s["y"], K=case["K"])
    if kind == "heads":
        nmm.nmm_batched_gemv_bf16(s["x"], s["W"], s["yb"], y=s["y"], N=case["N"])
        return s["y"], s["yb"]
    if kind == "entry":
        nmm.nmm_mla_kv_update(s["h"], s["w"], s["gamma"], s["mm"], s["cache"], kv_lora=case["kv_lora"],
                              rope=case["rope"], eps=EPS, theta=THETA, position=case["position"])
        return s["mm"], s["entry"], s["cache"]
    if kind == "attention":
        nmm.nmm_latent_attention_bf16(s["q"], s["kv"], s["out"], s["outb"], s["scale"], d_qk=case["d_qk"],
                                      d_v=case["d_v"])
        return s["out"], s["outb"]
    if kind == "step":
        s["step"].launch()
        return s["outs"]
    b = s["b"]
    s["path"].launch()
    nmm.nmm_latent_attention_bf16(b["query"], b["kv_cache"], s["att"], s["att_b"], SCALE)
    nmm.nmm_batched_gemv_bf16(s["att_rows"], b["w_uv"], s["o_b"], y=s["o"])
    nmm.nmm_gemv(s["o_row"], b["w_o"], s["y"])
    return s["outs"]


def _chain_work(heads):
    """Elements of the weights and of the fp32 results of one layer's five MatMuls."""
    w = HIDDEN * DOWN + Q_LORA * heads * QK + heads * NOPE * KV_LORA + heads * KV_LORA * V_HEAD + \
        heads * V_HEAD * HIDDEN
    return w, DOWN + heads * (QK + KV_LORA + V_HEAD) + HIDDEN


def work(case):
    kind = case["kind"]
    if kind in ("gemv", "linear", "heads"):
        B, M, K, N = case.get("B", 1), case["M"], case["K"], case["N"]
        out = 6 if kind == "heads" else 4
        return {"bytes": B * (M * K * 2 + K * N * 2 + M * N * out), "flops": 2 * B * M * K * N}
    if kind == "entry":
        n = case["kv_lora"] + case["rope"]
        return {"bytes": case["hidden"] * (n + 1) * 2 + n * 6 + case["kv_lora"] * 2, "flops": 2 * case["hidden"] * n}
    if kind == "attention":
        h, t, dq, dv = case["heads"], case["seq"], case["d_qk"], case["d_v"]
        return {"bytes": h * dq * 2 + t * max(dq, dv) * 2 + h * dv * 6, "flops": 2 * h * t * (dq + dv)}
    h, t, d = case["heads"], case["seq"], KV_LORA + ROPE
    w, outs = _chain_work(h)
    return {"bytes": 2 * w + 4 * outs + HIDDEN * 2 + t * d * 2 + h * d * 2 + h * KV_LORA * 6,
            "flops": 2 * w + 2 * h * t * (d + KV_LORA)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("gemv", "linear"):
        return {"rel": 2e-6}                    # fp32 sums of up to 16384 exact products: 1e-7 to 5e-7 measured
    if kind in ("heads", "entry"):
        return {"rel": 1e-3, "max": 8e-3}       # bf16 results: a rounding may fall the other way at a tie
    if kind in ("attention", "step"):
        return {"rel": 8e-3, "max": 4e-2}       # probabilities rounded to bf16: up to 2e-3 measured
    return {"rel": 1e-2, "max": 5e-2}           # the same, with bf16 hand-offs between the products


def _rope64(v, position):
    """RoPE of the last dimension's adjacent pairs, in 64 bits."""
    n = v.shape[-1]
    i = torch.arange(n // 2, dtype=torch.float64, device=v.device)
    a = float(position) * THETA ** (-2.0 * i / n)
    a = torch.remainder(a, 2 * math.pi)
    c, s = torch.cos(a), torch.sin(a)
    k0, k1 = v[..., 0::2], v[..., 1::2]
    return torch.stack((k0 * c - k1 * s, k0 * s + k1 * c), -1).reshape(v.shape)


def _entry64(mm, gamma, kv_lora, position):
    c = mm[:kv_lora]
    norm = c / torch.sqrt((c * c).mean() + EPS) * gamma.double()
    return torch.cat((norm, _rope64(mm[kv_lora:], position)))


def _attention64(q, kv, d_qk, d_v, scale):
    kv = kv.double()
    p = torch.softmax(scale * (q[:, :d_qk].double() @ kv[:, :d_qk].T.contiguous()), dim=-1)
    return p @ kv[:, :d_v].contiguous()


def _b(t):
    """Rounded to bf16, as the next product's operand is."""
    return t.to(torch.bfloat16).double()


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "gemv":
        return s["x"][:, :case["K"]].double() @ s["W"][:, :case["N"]].double().contiguous()
    if kind == "linear":
        return s["x"][:, :case["K"]].double() @ s["W"][:, :case["K"]].double().T.contiguous()
    if kind == "heads":
        y = torch.bmm(s["x"][..., :case["K"]].double().contiguous(), s["W"][..., :case["N"]].double().contiguous())
        return y, y
    if kind == "entry":
        n = case["kv_lora"] + case["rope"]
        mm = (s["h"][:case["hidden"]].double()[None] @ s["w"][:, :n].double().contiguous())[0]
        entry = _entry64(mm, s["gamma"], case["kv_lora"], case["position"])
        cache = s["cache"].double()
        cache[case["position"]] = entry
        return mm, entry, cache
    if kind == "attention":
        out = _attention64(s["q"], s["kv"], case["d_qk"], case["d_v"], s["scale"])
        return out, out
    heads, seq = case["heads"], case["seq"]
    b = s["step"]._bufs if kind == "step" else s["b"]
    down = (b["x"].double()[None] @ b["w_down"].double())[0]
    q = (_b(down[:Q_LORA])[None] @ b["w_uq"].double())[0]
    qh = q.view(heads, QK)
    lat = torch.bmm(_b(qh[:, None, :NOPE]).contiguous(), b["w_uk"].double())[:, 0]
    if kind == "step":
        o = torch.bmm(_b(lat)[:, None], b["w_uv"].double())
        y = _b(o).view(1, -1) @ b["w_o"].double()
        a = s["step"]._attn_bufs
        out = _attention64(a["q"], a["kv"], KV_LORA + ROPE, KV_LORA, SCALE)
        return {"down": down, "q": q, "lat": lat.reshape(-1), "o": o.reshape(-1), "y": y[0], "out": out,
                "out_bf16": out}
    query = torch.cat((lat, _rope64(qh[:, NOPE:], seq)), -1)
    entry = _entry64(down[Q_LORA:], b["kv_gamma"], KV_LORA, seq)
    cache = b["kv_cache"].double()
    cache[seq] = _b(entry)
    att = _attention64(_b(query), cache, KV_LORA + ROPE, KV_LORA, SCALE)
    o = torch.bmm(_b(att)[:, None], b["w_uv"].double())
    y = _b(o).view(1, -1) @ b["w_o"].double()
    return {"down": down, "q": q, "qlat": lat.reshape(-1), "query": query, "entry": entry, "att": att, "o": o, "y": y}
