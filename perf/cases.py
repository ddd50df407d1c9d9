"""The work whose speed counts: attention training steps, attention for serving, and the row-wise
kernels around them, each through the package's public entry points.

Four kinds of case (`op`):
  "step"    one attention training step, forward and backward.  api "call": attn_fwd + attn_bwd on
            the tensors of a program that drives the library itself; api "autograd": fused_attention
            under torch's autograd, as a model's layer uses it.
  "serve"   one attention forward of a serving program (attn_fwd_rect): new rows against a
            key/value cache, decoding (Sq = 1), a few speculative tokens, or a prefill chunk;
            rope: with the rotary embedding of the new rows fused in (attn_fwd_rope).
  "norm"    kind "layernorm": LayerNorm forward and backward; kind "rmsnorm": RMSNorm forward.
  "rotary"  the rotary embedding of one tensor.
"""
import math

import torch

import paper_2601_16238_amd as attn
from paper_2601_16238_amd import rowops
from paper_2601_16238_amd.autograd import fused_attention

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16}


def _step(api, B, Hq, Hkv, S, D, causal, dtype="bf16", sigma=1.0, outliers=0.0):
    return {"op": "step", "api": api, "B": B, "Hq": Hq, "Hkv": Hkv, "S": S, "D": D,
            "causal": causal, "dtype": dtype, "sigma": sigma, "outliers": outliers}


def _serve(B, Hq, Hkv, Sq, Sk, D, rope):
    return {"op": "serve", "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Sk": Sk, "D": D, "rope": rope}


def _norm(kind, rows, cols):
    return {"op": "norm", "kind": kind, "rows": rows, "cols": cols}


def _rotary(B, H, S, D):
    return {"op": "rotary", "B": B, "H": H, "S": S, "D": D}


def listed():
    return [
        # the smallest call: two short heads, where latency and launches are all there is
        dict(_step("call", 1, 2, 2, 128, 64, False), name="tiny_step"),
        # a CIFAR ViT layer: 64 patches and a class token, ragged, many short heads
        dict(_step("autograd", 128, 6, 6, 65, 64, False), name="vit_step"),
        # a character-level GPT's layer
        dict(_step("autograd", 8, 8, 8, 1024, 64, True, sigma=0.5), name="minigpt_step"),
        # the shape that fused attention kernels are usually compared at
        dict(_step("call", 4, 32, 32, 4096, 128, False), name="sdpa_step"),
        # long context on few heads; some rows of Q and K are large
        dict(_step("call", 1, 16, 16, 16384, 128, True, outliers=0.01), name="long_step"),
        # grouped heads, fp16, a head dimension between the kernels' own and a length off every tile
        dict(_step("autograd", 2, 16, 4, 1537, 96, True, dtype="f16"), name="grouped_f16_step"),
        # the largest head dimension
        dict(_step("call", 4, 16, 16, 4096, 256, True), name="headdim256_step"),
        # one new token per sequence against an 8K cache
        dict(_serve(8, 32, 8, 1, 8192, 128, False), name="decode"),
        # 512 new rows after 3584 cached ones, queries rotated on the way
        dict(_serve(1, 32, 8, 512, 4096, 128, True), name="prefill_chunk_rope"),
        # the norm of the ViT layer above: 128 x 65 tokens of 6 x 64 columns
        dict(_norm("layernorm", 8320, 384), name="vit_layernorm"),
        # the norm of a large language model's serving step
        dict(_norm("rmsnorm", 4096, 8192), name="rmsnorm"),
        # the queries (or keys) of a 2048-token batch
        dict(_rotary(4, 8, 2048, 128), name="rotary"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "serve", "serve", "norm", "norm", "rotary"])
    if op == "step":
        S = _log(rng, 17, 16384)
        D = rng.choice([64, 64, 128, 128, 128, 32, 80, 96, 256])
        causal = rng.random() < 0.6
        # work up to that of the largest listed step, and a bounded number of elements
        heads = max(1, int(min(2e11 / (float(S) * S * D), 3e7 / (float(S) * D), 1024)))
        Hkv = rng.choice([h for h in (1, 2, 4, 5, 6, 8, 12, 16) if h <= heads])
        G = rng.choice([g for g in (1, 1, 1, 2, 4) if g * Hkv <= heads])
        B = _log(rng, 1, heads // (Hkv * G))
        api = "autograd" if G > 1 else rng.choice(["call", "autograd"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16"]) if api == "autograd" else "bf16"
        return _step(api, B, Hkv * G, Hkv, S, D, causal, dtype)
    if op == "serve":
        Hkv = rng.choice([1, 2, 4, 8])
        G = rng.choice([1, 4, 8])
        D = rng.choice([64, 128, 128])
        Sq = rng.choice([1, 1, rng.randint(2, 8), _log(rng, 33, 1024)])
        Sk = Sq + _log(rng, 200, 32768)
        most = max(1, int(min(1.3e8 / (Hkv * Sk * D), 3e11 / (4.0 * Hkv * G * Sq * Sk * D))))
        return _serve(_log(rng, 1, min(most, 64)), Hkv * G, Hkv, Sq, Sk, D, rng.random() < 0.3)
    if op == "norm":
        cols = 8 * _log(rng, 32, 1024)
        rows = _log(rng, 64, min(65536, 33554432 // cols))
        return _norm(rng.choice(["layernorm", "rmsnorm"]), rows, cols)
    D = rng.choice([64, 128, 96, 256])
    H, S = rng.choice([4, 8, 12, 16, 32]), _log(rng, 60, 8192)
    return _rotary(_log(rng, 1, max(2, 33554432 // (H * S * D))), H, S, D)


def _scale(D):
    return float(D) ** -0.5


def _tables(S, D):
    """cos and sin of the rotary positions, fp32 [S, D/2]."""
    inv = 10000.0 ** (-torch.arange(0, D, 2, dtype=torch.float64, device="cuda") / D)
    ang = torch.arange(S, dtype=torch.float64, device="cuda")[:, None] * inv[None, :]
    return ang.cos().float(), ang.sin().float()


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, dtype=torch.bfloat16, sigma=1.0, mean=0.0):
        x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
        return (x * sigma + mean).to(dtype)

    st = dict(case)
    if case["op"] == "step":
        B, Hq, Hkv, S, D = (case[k] for k in ("B", "Hq", "Hkv", "S", "D"))
        for name, H in (("q", Hq), ("k", Hkv), ("v", Hkv), ("do", Hq)):
            st[name] = normal(B, H, S, D, dtype=DTYPES[case["dtype"]], sigma=case["sigma"])
        if case["outliers"]:
            for name in ("q", "k"):
                rows = st[name].view(-1, D)
                pick = torch.randperm(rows.shape[0], generator=g, device="cuda")
                rows[pick[:int(round(case["outliers"] * rows.shape[0]))]] *= 8.0
        if case["api"] == "autograd":
            for name in ("q", "k", "v"):
                st[name].requires_grad_()
    elif case["op"] == "serve":
        B, Hq, Hkv, Sq, Sk, D = (case[k] for k in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
        st["q"], st["k"], st["v"] = normal(B, Hq, Sq, D), normal(B, Hkv, Sk, D), normal(B, Hkv, Sk, D)
        if case["rope"]:  # the cache holds rotated keys; these stand for them
            st["cos"], st["sin"] = _tables(Sk, D)
    elif case["op"] == "norm":
        rows, cols = case["rows"], case["cols"]
        st["x"] = normal(rows, cols, sigma=2.0, mean=0.25)
        st["w"] = normal(cols, dtype=torch.float32, sigma=0.5, mean=1.0)
        if case["kind"] == "layernorm":
            st["b"], st["dy"] = normal(cols, dtype=torch.float32, sigma=0.3), normal(rows, cols)
    else:
        st["x"] = normal(case["B"], case["H"], case["S"], case["D"])
        st["cos"], st["sin"] = _tables(case["S"], case["D"])
    return st


def run(st):
    if st["op"] == "step":
        q, k, v, do, causal, scale = st["q"], st["k"], st["v"], st["do"], st["causal"], _scale(st["D"])
        if st["api"] == "autograd":
            o = fused_attention(q, k, v, causal=causal, scale=scale)
            dq, dk, dv = torch.autograd.grad(o, (q, k, v), do)
            return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
        o, lse = attn.attn_fwd(q, k, v, scale, causal)
        dq, dk, dv = attn.attn_bwd(q, k, v, o, do, lse, scale, causal)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if st["op"] == "serve":
        if st["rope"]:
            o, lse, _ = attn.attn_fwd_rope(st["q"], st["k"], st["v"], st["cos"], st["sin"], _scale(st["D"]),
                                           True, want_q_rot=False)
        else:
            o, lse = attn.attn_fwd_rect(st["q"], st["k"], st["v"], _scale(st["D"]), True)
        return {"o": o, "lse": lse}
    if st["op"] == "norm":
        if st["kind"] == "rmsnorm":
            return {"y": rowops.rmsnorm_fwd(st["x"], st["w"], 1e-6)}
        y, mean, rstd = rowops.layernorm_fwd(st["x"], st["w"], st["b"], 1e-5)
        dx, dw, db = rowops.layernorm_bwd(st["dy"], st["x"], st["w"], mean, rstd)
        return {"y": y, "mean": mean, "rstd": rstd, "dx": dx, "dw": dw, "db": db}
    return {"y": rowops.rotary_fwd(st["x"], st["cos"], st["sin"])}


def _pairs(Sq, Sk, causal):
    """Visible (query, key) pairs of one head; a causal mask is aligned to the last row and key."""
    return Sq * (Sk - Sq) + Sq * (Sq + 1) // 2 if causal else Sq * Sk


def work(case):
    if case["op"] == "step":
        B, Hq, Hkv, S, D = (case[k] for k in ("B", "Hq", "Hkv", "S", "D"))
        # q, do in and o, dq out; k, v in and dk, dv out; two products forward, five backward
        return {"bytes": 8 * B * (Hq + Hkv) * S * D, "flops": 14 * B * Hq * _pairs(S, S, case["causal"]) * D}
    if case["op"] == "serve":
        B, Hq, Hkv, Sq, Sk, D = (case[k] for k in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
        rope = 4 * Sq * D if case["rope"] else 0
        return {"bytes": 4 * B * (Hq * Sq + Hkv * Sk) * D + rope + 4 * B * Hq * Sq,
                "flops": 4 * B * Hq * _pairs(Sq, Sk, True) * D}
    if case["op"] == "norm":
        n = case["rows"] * case["cols"]
        if case["kind"] == "rmsnorm":
            return {"bytes": 4 * n + 4 * case["cols"], "flops": 4 * n}
        # x, dy in and y, dx out, once each
        return {"bytes": 8 * n + 16 * case["cols"] + 8 * case["rows"], "flops": 20 * n}
    n = case["B"] * case["H"] * case["S"] * case["D"]
    return {"bytes": 4 * n + 4 * case["S"] * case["D"], "flops": 3 * n}


def tolerance(case):
    """About four times the distance to the result in 64 bits that was measured (bf16 0.0017 for a
    row-wise result, 0.0023 .. 0.0025 for attention, 0.005 with outlier rows; fp16 0.0003): a 16-bit
    result is rounded once, and the gradients carry the rounding of P, dS and O."""
    if case["op"] == "step":
        if case["dtype"] == "f16":
            return {"rel": 1.3e-3}
        return {"rel": 2e-2} if case["outliers"] else {"rel": 1e-2}
    return {"rel": 1e-2} if case["op"] == "serve" else {"rel": 7e-3}


def _rotated(x, cos, sin):
    hd = x.shape[-1] // 2
    x1, x2 = x[..., :hd], x[..., hd:]
    return torch.cat([x1 * cos - x2 * sin, x2 * cos + x1 * sin], dim=-1)


def _exact_attention(q, k, v, do, scale, causal, chunk_bytes=2 << 30):
    """O, LSE and (do given) dQ, dK, dV in 64 bits; q, do [B,Hq,Sq,D], k, v [B,Hkv,Sk,D].  A few
    K/V heads at a time, each against the query heads that read it."""
    B, Hq, Sq, D = q.shape
    Hkv, Sk = k.shape[1], k.shape[2]
    G = Hq // Hkv
    q, k, v = (t.detach().double() for t in (q, k, v))
    qg = q.reshape(B * Hkv, G, Sq, D)
    kf, vf = k.reshape(B * Hkv, Sk, D), v.reshape(B * Hkv, Sk, D)
    o, lse = torch.empty_like(qg), torch.empty(qg.shape[:3], dtype=torch.float64, device=q.device)
    if do is not None:
        dog = do.double().reshape(B * Hkv, G, Sq, D)
        dq, dk, dv = torch.empty_like(qg), torch.empty_like(kf), torch.empty_like(vf)
    hidden = None
    if causal:
        row = torch.arange(Sq, device=q.device)[:, None] + (Sk - Sq)
        hidden = torch.arange(Sk, device=q.device)[None, :] > row
    n = max(1, int(chunk_bytes // (8 * Sq * Sk)))
    for i in range(0, B * Hkv, n):
        kc, vc = kf[i:i + n], vf[i:i + n]
        kt, vt = kc.transpose(1, 2).contiguous(), vc.transpose(1, 2).contiguous()
        for j in range(G):
            qc = qg[i:i + n, j].contiguous()
            s = torch.matmul(qc, kt).mul_(scale)
            if hidden is not None:
                s.masked_fill_(hidden, -math.inf)
            le = torch.logsumexp(s, dim=-1)
            p = s.sub_(le[..., None]).exp_()
            oc = torch.matmul(p, vc)
            o[i:i + n, j], lse[i:i + n, j] = oc, le
            if do is None:
                continue
            doc = dog[i:i + n, j].contiguous()
            pt = p.transpose(1, 2).contiguous()
            gv = torch.matmul(pt, doc)
            ds = torch.matmul(doc, vt).sub_((doc * oc).sum(-1, keepdim=True)).mul_(p).mul_(scale)
            del p, pt, s
            dq[i:i + n, j] = torch.matmul(ds, kc)
            gk = torch.matmul(ds.transpose(1, 2).contiguous(), qc)
            if j == 0:
                dk[i:i + n], dv[i:i + n] = gk, gv
            else:
                dk[i:i + n] += gk
                dv[i:i + n] += gv
    out = {"o": o.reshape(q.shape), "lse": lse.reshape(B, Hq, Sq)}
    if do is not None:
        out.update(dq=dq.reshape(q.shape), dk=dk.reshape(k.shape), dv=dv.reshape(v.shape))
    return out


def exact(case, seed):
    st = prepare(case, seed)
    if case["op"] == "step":
        with torch.no_grad():
            out = _exact_attention(st["q"], st["k"], st["v"], st["do"], _scale(case["D"]), case["causal"])
        if case["api"] == "autograd":
            del out["lse"]
        return out
    if case["op"] == "serve":
        q = st["q"]
        if case["rope"]:  # the rotated rows are 16-bit rows: rounded once, like the keys
            at = slice(case["Sk"] - case["Sq"], case["Sk"])
            q = _rotated(q.double(), st["cos"][at].double(), st["sin"][at].double()).to(q.dtype)
        return _exact_attention(q, st["k"], st["v"], None, _scale(case["D"]), True)
    x = st["x"].double()
    if case["op"] == "rotary":
        return {"y": _rotated(x, st["cos"].double(), st["sin"].double())}
    w = st["w"].double()
    if case["kind"] == "rmsnorm":
        return {"y": x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6) * w}
    mean = x.mean(-1, keepdim=True)
    xc = x - mean
    rstd = torch.rsqrt(xc.square().mean(-1, keepdim=True) + 1e-5)
    xhat, dy = xc * rstd, st["dy"].double()
    gr = dy * w
    dx = rstd * (gr - gr.mean(-1, keepdim=True) - xhat * (gr * xhat).mean(-1, keepdim=True))
    return {"y": xhat * w + st["b"].double(), "mean": mean[:, 0], "rstd": rstd[:, 0],
            "dx": dx, "dw": (dy * xhat).sum(0), "db": dy.sum(0)}
