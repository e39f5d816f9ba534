"""The measured cases: what a user of this library calls, over the sizes it is called with.

Three kinds of call:

* ``enc``  -- one encoder forward (MiniLM-L6 shape: hidden 384, 12 heads of 32,
  FFN 1536, 6 layers) on a right-padded batch of token ids, the library's main
  path: single queries, ordinary and bulk batches, long documents, fp32,
  weight-only int8 / int4, pooled embeddings or hidden states;
* ``mlp``  -- a transformer MLP, two matmuls with fused epilogues
  (up + bias + GELU, down + bias + residual) on dense or quantised weights:
  one decode step (M = 1), a batched decode step, a prefill chunk;
* ``attn`` / ``mx`` -- the masked-attention and block-scaled minifloat matmul
  entry points on their own.

``listed`` holds the fixed cases, ``draw`` gives others from the same ranges.
Inputs come from the seed alone and are made on the GPU.  Sequence lengths are
evenly spaced over the case's range and shuffled by the seed, so the work of a
case does not depend on the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2609_37916_amd as rlx

HIDDEN, HEADS, HEAD_DIM, FFN, LAYERS = 384, 12, 32, 1536, 6
VOCAB, MAX_POS, TYPE_VOCAB, LN_EPS = 30522, 512, 2, 1e-12

# Weight schemes of the matmul: (library scheme, group size or 0 for per channel, bits, has zeros / mins)
SCHEMES = {
    "bf16": (rlx.Q_NONE, 0, 16, False),
    "f32": (rlx.Q_NONE, 0, 32, False),
    "int8": (rlx.Q_INT8_PER_CHANNEL, 0, 8, False),
    "int4": (rlx.Q_INT4_GROUP_ZP, 32, 4, True),
    "int8_group": (rlx.Q_INT8_GROUP, 32, 8, False),
    "int4_min": (rlx.Q_INT4_GROUP_MIN, 32, 4, True),
    "int8_group16": (rlx.Q_INT8_GROUP16, 16, 8, False),
}
# Minifloat formats: (exponent bits, mantissa bits, bias, exponent of the largest value)
MX = {"e4m3": (4, 3, 7, 8), "e5m2": (5, 2, 15, 15), "e2m3": (2, 3, 1, 2), "e3m2": (3, 2, 3, 4), "e2m1": (2, 1, 1, 2)}
KINDS = {"none": rlx.MASK_NONE, "causal": rlx.MASK_CAUSAL, "sliding": rlx.MASK_SLIDING_WINDOW,
         "custom": rlx.MASK_CUSTOM}


def _enc(name, batch, seq, lo, dtype="bf16", quant="none", output="pooled", full=0):
    c = {"kind": "enc", "batch": batch, "seq": seq, "lo": lo, "full": full, "dtype": dtype, "quant": quant,
         "output": output}
    return {"name": name, **c} if name else c


def _mlp(name, scheme, m, hidden, ffn):
    c = {"kind": "mlp", "scheme": scheme, "m": m, "hidden": hidden, "ffn": ffn}
    return {"name": name, **c} if name else c


def _attn(name, mask, batch, seq, lo, dtype="bf16", window=0):
    c = {"kind": "attn", "mask": mask, "batch": batch, "seq": seq, "lo": lo, "dtype": dtype, "window": window}
    return {"name": name, **c} if name else c


def _mx(name, fx, fw, m, n, k):
    c = {"kind": "mx", "fx": fx, "fw": fw, "m": m, "n": n, "k": k}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one search query or short document embedded by itself: latency
        _enc("enc_bf16_b1_s128", 1, 128, 96),
        # the benchmark's default batch: an embedding service's ordinary request
        _enc("enc_bf16_b32_s128", 32, 128, 16),
        # bulk indexing of a corpus: throughput
        _enc("enc_bf16_b256_s128", 256, 128, 8),
        # long documents, half of them at the model's limit
        _enc("enc_bf16_b8_s512", 8, 512, 64, full=4),
        # the fp32 model, for users who compare or fine-tune against it
        _enc("enc_f32_b64_s128", 64, 128, 8, dtype="f32"),
        # weight-only quantised model at the ordinary batch
        _enc("enc_int4_b32_s128", 32, 128, 16, quant="int4"),
        # attention over long sequences by itself, causal
        _attn("attn_causal_b8_s512", "causal", 8, 512, 512),
        # one decode step through a quantised MLP
        _mlp("mlp_int4_m1", "int4", 1, 4096, 14336),
        # a batched decode step, the layout that Q4_K and Q4_1 weights are repacked into
        _mlp("mlp_int4_min_m16", "int4_min", 16, 4096, 14336),
        # a ragged prefill chunk on int8 weights
        _mlp("mlp_int8_m509", "int8", 509, 4096, 14336),
        # a long prefill on dense weights: the largest product
        _mlp("mlp_bf16_m2048", "bf16", 2048, 4096, 14336),
        # FP8 block-scaled product of the encoder's FFN-down shape over a bulk batch
        _mx("mx_e4m3_m18048_n384_k1536", "e4m3", "e4m3", 18048, 384, 1536),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    u = rng.random()
    if u < 0.45:
        dtype, quant = rng.choice([("bf16", "none")] * 5 + [("f32", "none")] * 2 + [("bf16", "int8"), ("bf16", "int4")])
        most = 8192 if dtype == "f32" else 32768
        seq = _log(rng, 16, 512)
        batch = _log(rng, 1, min(256, most // seq))
        lo = rng.randint(1, seq)
        full = rng.choice([0, 0, batch // 2])
        return _enc(None, batch, seq, lo, dtype, quant, rng.choice(["pooled"] * 3 + ["hidden"]), full)
    if u < 0.60:
        seq = _log(rng, 16, 512)
        batch = _log(rng, 1, min(64, 16384 // seq))
        mask = rng.choice(["none", "causal", "sliding", "custom"])
        lo = rng.randint(1, seq) if mask == "custom" else seq
        return _attn(None, mask, batch, seq, lo, rng.choice(["bf16", "bf16", "bf16", "f32"]),
                     rng.randint(1, seq) if mask == "sliding" else 0)
    if u < 0.88:
        scheme = rng.choice(["bf16", "bf16", "f32", "int8", "int4", "int4", "int4_min", "int4_min", "int8_group",
                             "int8_group16"])
        m = _log(rng, 1, 256 if scheme == "f32" else 2048)
        return _mlp(None, scheme, m, 64 * _log(rng, 6, 64), 64 * _log(rng, 24, 224))
    fx, fw = rng.choice([("e4m3", "e4m3"), ("e4m3", "e4m3"), ("e5m2", "e4m3"), ("e4m3", "e2m1"), ("e2m3", "e2m3"),
                         ("e3m2", "e3m2"), ("e2m1", "e2m1"), ("e2m1", "e2m1")])
    return _mx(None, fx, fw, _log(rng, 1, 18048), 128 * _log(rng, 1, 32), 128 * _log(rng, 1, 32))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape, std=1.0):
    return torch.randn(*shape, generator=g, device="cuda") * std


def _lengths(c):
    """Token counts: ``full`` rows of ``seq``, the others evenly spaced over [lo, seq]."""
    n = c["batch"] - c.get("full", 0)
    lens = [c["lo"] + int((c["seq"] - c["lo"] + 1) * (i + 0.5) / n) for i in range(n)]
    return lens + [c["seq"]] * (c["batch"] - n)


def _mask(c, g):
    lens = torch.tensor(_lengths(c), device="cuda")[torch.randperm(c["batch"], generator=g, device="cuda")]
    return (torch.arange(c["seq"], device="cuda")[None, :] < lens[:, None]).to(torch.uint8).contiguous()


def _quantise(w, scheme):
    """w [N, K] f32 -> (codes, scales, zeros) in the library's documented layouts."""
    _, group, bits, has_zeros = SCHEMES[scheme]
    n, k = w.shape
    if group == 0:
        s = (w.abs().amax(1) / 127).to(torch.float16)
        return (w / s.float()[:, None]).round().clamp(-127, 127).to(torch.int8), s, None
    gw = w.view(n, k // group, group)
    if bits == 8:
        s = (gw.abs().amax(2) / 127).to(torch.float16)
        q = (gw / s.float()[..., None]).round().clamp(-127, 127).to(torch.int8).view(n, k)
        return q, s, None
    mn, mx = gw.amin(2), gw.amax(2)
    s = ((mx - mn) / 15).to(torch.float16)
    if scheme == "int4_min":
        z = mn.to(torch.float16)
        q = ((gw - z.float()[..., None]) / s.float()[..., None]).round().clamp(0, 15)
    else:
        z = (-mn / s.float()).round().clamp(0, 15).to(torch.float16)
        q = (gw / s.float()[..., None]).round().add(z.float()[..., None]).clamp(0, 15)
    q = q.to(torch.uint8).view(n, k)
    return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous(), s, z


def _linear(g, n, k, scheme, std=0.02):
    w = _randn(g, n, k, std=std)
    if scheme in ("bf16", "f32"):
        return {"w": w.to(torch.bfloat16) if scheme == "bf16" else w, "scales": None, "zeros": None}
    q, s, z = _quantise(w, scheme)
    return {"w": q, "scales": s, "zeros": z}


def _dequant64(lin, scheme):
    """The weights the library is given, as float64."""
    _, group, bits, _ = SCHEMES[scheme]
    w, s, z = lin["w"], lin["scales"], lin["zeros"]
    if bits >= 16:
        return w.double()
    if bits == 4:
        w = torch.stack([w & 15, w >> 4], -1).view(w.shape[0], -1)
    if group == 0:
        return w.double() * s.double()[:, None]
    gw = w.double().view(w.shape[0], -1, group)
    if bits == 8:
        gw = gw * s.double()[..., None]
    elif scheme == "int4_min":
        gw = gw * s.double()[..., None] + z.double()[..., None]
    else:
        gw = (gw - z.double()[..., None]) * s.double()[..., None]
    return gw.view(w.shape[0], -1)


def _enc_inputs(c, seed):
    g = _gen(seed)
    act = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    scheme = c["quant"] if c["quant"] != "none" else c["dtype"]
    mask = _mask(c, g)
    ids = torch.randint(1000, VOCAB, (c["batch"], c["seq"]), generator=g, device="cuda", dtype=torch.int32)
    ids = ids * mask

    def ln():
        return 1 + _randn(g, HIDDEN, std=0.1), _randn(g, HIDDEN, std=0.1)

    w = {"word": _randn(g, VOCAB, HIDDEN, std=0.02).to(act), "pos": _randn(g, MAX_POS, HIDDEN, std=0.02).to(act),
         "type": _randn(g, TYPE_VOCAB, HIDDEN, std=0.02).to(act), "layers": []}
    w["emb_gamma"], w["emb_beta"] = ln()
    for _ in range(LAYERS):
        d = {}
        for nm, n, k in (("wqkv", 3 * HIDDEN, HIDDEN), ("wo", HIDDEN, HIDDEN), ("w1", FFN, HIDDEN), ("w2", HIDDEN, FFN)):
            lin = _linear(g, n, k, scheme)
            d[nm] = lin["w"]
            if lin["scales"] is not None:
                d[nm + "_scales"] = lin["scales"]
            if lin["zeros"] is not None:
                d[nm + "_zeros"] = lin["zeros"]
            d["b" + nm[1:]] = _randn(g, n, std=0.02)
        d["ln1_g"], d["ln1_b"] = ln()
        d["ln2_g"], d["ln2_b"] = ln()
        w["layers"].append(d)
    return w, ids, mask


def _mlp_inputs(c, seed):
    g = _gen(seed)
    act = torch.float32 if c["scheme"] == "f32" else torch.bfloat16
    h, f = c["hidden"], c["ffn"]
    return {"x": _randn(g, c["m"], h).to(act), "up": _linear(g, f, h, c["scheme"]), "down": _linear(g, h, f, c["scheme"]),
            "b1": _randn(g, f, std=0.02), "b2": _randn(g, h, std=0.02)}


def _attn_inputs(c, seed):
    g = _gen(seed)
    act = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    qkv = _randn(g, c["batch"] * c["seq"], 3 * HIDDEN).to(act)
    return {"qkv": qkv, "key_mask": _mask(c, g) if c["mask"] == "custom" else None}


def _mx_values(fmt):
    """Decoded value of every code of the format; NaN and Inf codes as NaN."""
    e_bits, m_bits, bias, _ = MX[fmt]
    out = []
    for code in range(1 << (1 + e_bits + m_bits)):
        e, m = (code >> m_bits) & ((1 << e_bits) - 1), code & ((1 << m_bits) - 1)
        v = math.ldexp(1 + m / (1 << m_bits), e - bias) if e else math.ldexp(m / (1 << m_bits), 1 - bias)
        if fmt == "e4m3" and (code & 0x7F) == 0x7F or fmt == "e5m2" and e == 31:
            v = math.nan
        out.append(-v if code >> (e_bits + m_bits) else v)
    return out


def _mx_operand(g, rows, k, fmt):
    """N(0, 1) rows rounded to the nearest block-scaled value: (packed rows, scales, codes)."""
    e_bits, m_bits, _, emax = MX[fmt]
    bits = 1 + e_bits + m_bits
    x = _randn(g, rows, k // 32, 32)
    e = torch.floor(torch.log2(x.abs().amax(2))) - emax
    y = (x * torch.exp2(-e)[..., None]).view(rows, k)
    vals = _mx_values(fmt)[: 1 << (bits - 1)]
    grid = torch.tensor([v for v in vals if not math.isnan(v)], device="cuda")  # ascending in the code
    code = torch.bucketize(y.abs(), (grid[1:] + grid[:-1]) / 2).to(torch.uint8)
    code = code | ((y < 0).to(torch.uint8) << (bits - 1))
    scales = (e + 127).to(torch.uint8).contiguous()
    if bits == 8:
        packed = code
    elif bits == 4:
        packed = code[:, 0::2] | (code[:, 1::2] << 4)
    else:
        q = code.view(rows, k // 4, 4).to(torch.int32)
        word = q[..., 0] | (q[..., 1] << 6) | (q[..., 2] << 12) | (q[..., 3] << 18)
        packed = torch.stack([word & 255, (word >> 8) & 255, (word >> 16) & 255], -1).to(torch.uint8).view(rows, -1)
    return packed.contiguous(), scales, code


def _mx_inputs(c, seed):
    g = _gen(seed)
    return _mx_operand(g, c["m"], c["k"], c["fx"]), _mx_operand(g, c["n"], c["k"], c["fw"])


def prepare(case, seed):
    k = case["kind"]
    if k == "enc":
        w, ids, mask = _enc_inputs(case, seed)
        enc = rlx.Encoder(dtype=case["dtype"], quant=case["quant"], output_kind=case["output"], max_batch=case["batch"],
                          max_seq=case["seq"], weights=w)
        return {"case": case, "enc": enc, "ids": ids, "mask": mask}
    if k == "mlp":
        return {"case": case, **_mlp_inputs(case, seed)}
    if k == "attn":
        return {"case": case, **_attn_inputs(case, seed)}
    (x, xs, _), (w, ws, _) = _mx_inputs(case, seed)
    return {"case": case, "x": x, "x_scales": xs, "w": w, "w_scales": ws}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    c = state["case"]
    if c["kind"] == "enc":
        return state["enc"].forward(state["ids"], state["mask"])
    if c["kind"] == "mlp":
        scheme, group, _, _ = SCHEMES[c["scheme"]]
        up, down = state["up"], state["down"]
        h = rlx.dequant_matmul(state["x"], up["w"], scheme=scheme, scales=up["scales"], zeros=up["zeros"],
                               group_size=group or 32, bias=state["b1"], epi=rlx.EPI_BIAS_GELU)
        y = rlx.dequant_matmul(h, down["w"], scheme=scheme, scales=down["scales"], zeros=down["zeros"],
                               group_size=group or 32, bias=state["b2"], residual=state["x"],
                               epi=rlx.EPI_BIAS_RESIDUAL)
        return {"h": h, "y": y}
    if c["kind"] == "attn":
        qkv = state["qkv"]
        return rlx.masked_attention(qkv[:, :HIDDEN], qkv[:, HIDDEN:2 * HIDDEN], qkv[:, 2 * HIDDEN:], B=c["batch"],
                                    S=c["seq"], heads=HEADS, kind=KINDS[c["mask"]], key_mask=state["key_mask"],
                                    window=c["window"])
    return rlx.scaled_matmul(state["x"], state["x_scales"], c["fx"], state["w"], state["w_scales"], c["fw"], K=c["k"])


# ---------------------------------------------------------------------------
# work and tolerances
# ---------------------------------------------------------------------------

def _weight_bytes(n, k, scheme):
    _, group, bits, has_zeros = SCHEMES[scheme]
    b = n * k * bits / 8
    if bits < 16:
        b += 2 * n * (k // group if group else 1) * (2 if has_zeros else 1)
    return b


def _visible(c):
    """Visible (query, key) pairs of one head."""
    s, n = c["seq"], c["batch"]
    if c["mask"] == "causal":
        return n * s * (s + 1) // 2
    if c["mask"] == "sliding":
        return n * sum(min(i + 1, c["window"]) for i in range(s))
    return s * sum(_lengths(c))


def work(case):
    c = case
    if c["kind"] == "enc":
        a = 2 if c["dtype"] == "bf16" else 4
        scheme = c["quant"] if c["quant"] != "none" else c["dtype"]
        lens = _lengths(c)
        t = sum(lens)
        weights = sum(_weight_bytes(n, k, scheme) + 4 * n for n, k in
                      ((3 * HIDDEN, HIDDEN), (HIDDEN, HIDDEN), (FFN, HIDDEN), (HIDDEN, FFN))) + 16 * HIDDEN
        out = (c["batch"] if c["output"] == "pooled" else c["batch"] * c["seq"]) * HIDDEN * 4
        nbytes = LAYERS * weights + (t + max(lens)) * HIDDEN * a + c["batch"] * c["seq"] * 5 + out
        flops = LAYERS * (2 * t * (4 * HIDDEN * HIDDEN + 2 * HIDDEN * FFN) + 4 * HIDDEN * sum(n * n for n in lens))
        return {"bytes": nbytes, "flops": flops}
    if c["kind"] == "mlp":
        a = 4 if c["scheme"] == "f32" else 2
        m, h, f = c["m"], c["hidden"], c["ffn"]
        nbytes = _weight_bytes(f, h, c["scheme"]) + _weight_bytes(h, f, c["scheme"]) + 4 * (h + f) + a * m * (2 * h + f)
        return {"bytes": nbytes, "flops": 4 * m * h * f}
    if c["kind"] == "attn":
        a = 2 if c["dtype"] == "bf16" else 4
        rows = c["batch"] * c["seq"]
        kv = sum(_lengths(c)) if c["mask"] == "custom" else rows
        return {"bytes": a * HIDDEN * (2 * rows + 2 * kv) + (rows if c["mask"] == "custom" else 0),
                "flops": 4 * HIDDEN * _visible(c)}
    bits = {f: 1 + v[0] + v[1] for f, v in MX.items()}
    m, n, k = c["m"], c["n"], c["k"]
    return {"bytes": m * k * bits[c["fx"]] / 8 + n * k * bits[c["fw"]] / 8 + (m + n) * k / 32 + 4 * m * n,
            "flops": 2 * m * n * k}


def tolerance(case):
    """About four times the distance from ``exact`` that the sizes above show.

    Measured: bf16 pooled embeddings 1.0e-3 .. 1.7e-3, bf16 hidden states
    5.9e-3 .. 8.2e-3 (LayerNormed rows, six layers), bf16 attention 1.9e-3 ..
    2.1e-3, MLP products rounded to bf16 1.6e-3 .. 3.2e-3, fp32 encoder 0.9e-7 ..
    4.2e-7, fp32 attention 2.0e-7 .. 3.9e-7, fp32 MLP 1.5e-7 .. 2.2e-6 (K up to
    14336), minifloat products 0 .. 1.5e-5 (the matrix cores' aligned adder).
    """
    c = case
    if c["kind"] == "mx":
        return {"rel": 6e-5}
    if c["kind"] == "mlp":
        return {"rel": 8e-6 if c["scheme"] == "f32" else 1.2e-2}
    if c["dtype"] == "f32":
        return {"rel": 2e-6}
    if c["kind"] == "attn":
        return {"rel": 8e-3}
    return {"rel": 2.4e-2 if c["output"] == "hidden" else 7e-3}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _gelu64(x):
    return 0.5 * x * (1 + torch.erf(x / math.sqrt(2)))


def _ln64(x, gamma, beta):
    d = x - x.mean(-1, keepdim=True)
    return d / torch.sqrt((d * d).mean(-1, keepdim=True) + LN_EPS) * gamma.double() + beta.double()


def _attention64(q, k, v, visible):
    """q, k, v [B, heads, S, d]; visible broadcastable to [B, heads, S, S]; every query sees a key."""
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(HEAD_DIM)
    return torch.matmul(torch.softmax(s.masked_fill(~visible, -math.inf), -1), v)


def _heads(x, b, s):
    return x.reshape(b, s, HEADS, HEAD_DIM).transpose(1, 2).contiguous()


def _enc64(c, seed):
    w, ids, mask = _enc_inputs(c, seed)
    b, s = mask.shape
    scheme = c["quant"] if c["quant"] != "none" else c["dtype"]
    x = w["word"].double()[ids.long()] + w["pos"].double()[None, :s] + w["type"].double()[0]
    x = _ln64(x, w["emb_gamma"], w["emb_beta"])

    def linear(x, lw, nm):
        lin = {"w": lw[nm], "scales": lw.get(nm + "_scales"), "zeros": lw.get(nm + "_zeros")}
        return torch.matmul(x, _dequant64(lin, scheme).t()) + lw["b" + nm[1:]].double()

    keys = mask.bool()[:, None, None, :]
    for lw in w["layers"]:
        q, k, v = linear(x, lw, "wqkv").split(HIDDEN, -1)
        ctx = _attention64(_heads(q, b, s), _heads(k, b, s), _heads(v, b, s), keys)
        x = _ln64(x + linear(ctx.transpose(1, 2).reshape(b, s, HIDDEN), lw, "wo"), lw["ln1_g"], lw["ln1_b"])
        x = _ln64(x + linear(_gelu64(linear(x, lw, "w1")), lw, "w2"), lw["ln2_g"], lw["ln2_b"])
    x = x * mask.double()[..., None]
    if c["output"] == "hidden":
        return x
    p = x.sum(1) / mask.double().sum(1, keepdim=True)
    return p / p.norm(dim=1, keepdim=True)


def exact(case, seed):
    c = case
    if c["kind"] == "enc":
        return _enc64(c, seed)
    if c["kind"] == "mlp":
        st = _mlp_inputs(c, seed)
        x = st["x"].double()
        h = _gelu64(torch.matmul(x, _dequant64(st["up"], c["scheme"]).t()) + st["b1"].double())
        y = torch.matmul(h, _dequant64(st["down"], c["scheme"]).t()) + st["b2"].double() + x
        return {"h": h, "y": y}
    if c["kind"] == "attn":
        st = _attn_inputs(c, seed)
        b, s = c["batch"], c["seq"]
        q, k, v = (_heads(t, b, s) for t in st["qkv"].double().split(HIDDEN, -1))
        i = torch.arange(s, device="cuda")
        if c["mask"] == "custom":
            vis = st["key_mask"].bool()[:, None, None, :]
        else:
            vis = torch.ones(s, s, dtype=torch.bool, device="cuda")
            if c["mask"] != "none":
                vis = i[None, :] <= i[:, None]
            if c["mask"] == "sliding":
                vis = vis & (i[None, :] > i[:, None] - c["window"])
        return _attention64(q, k, v, vis).transpose(1, 2).reshape(b * s, HIDDEN)
    ops = []
    for (_, scales, codes), fmt in zip(_mx_inputs(c, seed), (c["fx"], c["fw"])):
        vals = torch.tensor(_mx_values(fmt), dtype=torch.float64, device="cuda")[codes.long()]
        ops.append(vals * torch.exp2(scales.double() - 127).repeat_interleave(32, 1))
    return torch.matmul(ops[0], ops[1].t().contiguous())
