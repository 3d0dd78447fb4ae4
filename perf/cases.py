"""What a user of the packed forward has it do, as cases that can be timed and compared.

Three kinds of call, each through the package's public entry points:

  step   one packed step of a whole (small) model, ``packed_forward``: embedding, every layer,
         final norm, LM head and greedy tokens.  The fp32 decoder (2 layers, d 256) is the
         latency-bound end; the 7B-shape model has 4 of its 32 layers, since two correct bf16
         implementations drift apart by about 1.2e-3 of the norm per layer and 32 layers would
         leave nothing to compare.
  layer  one 7B-shape decoder layer in place on its hidden rows, ``packed_layer_forward``: the
         norms, four projections, rotary embedding and ring write, attention and residuals.  The
         step of the 32-layer model is 32 of these.  The rows' keys and values go to the ring,
         where the same call's attention reads them: every one of them enters the returned rows.
  head   final norm, LM head and greedy argmax of the emitting rows, ``op_lm_head_argmax``.

A packed step holds ``pipes`` prefill segments of ``P`` rows (0: none) that start at position
``ctx`` of their requests (0 for a whole prefill, more for a later chunk of one) and ``d`` single
decode rows.  Ranges: P 0..512, d 0..63, pipes 1..8, at most 2264 rows; decode rows with 1..544
positions of history.
"""
import math

import torch

import paper_2512_20276_amd as af
import workload as wl

MAX_ROWS = 2264


def _case(name, kind, **kw):
    c = {"kind": kind, "pipes": 1, "P": 0, "d": 0, "ctx": 0, "history": 0}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the tiny fp32 decoder's packed step, K = 3 and L_P = 32: launches and latency only
        _case("tiny_f32_step", "step", model="tiny", P=32, d=2, history=33),
        # one request alone, one action token: the step of the sequential baseline's decode phase
        _case("layer_decode_1", "layer", d=1, history=280),
        # decode rows only (every pipeline between two prefills), 15 requests in flight
        _case("layer_decode_15", "layer", d=15, history=283),
        # a short prompt (128 rows) packed with 7 decode rows
        _case("layer_p128_d7", "layer", P=128, d=7, history=132),
        # the benchmark's step, K = 7: 276 prefill rows and 6 decode rows
        _case("layer_p276_d6", "layer", P=276, d=6, history=280),
        # a long action chunk, K = 32: 276 prefill rows and 31 decode rows
        _case("layer_p276_d31", "layer", P=276, d=31, history=290),
        # a long instruction (256 vision and 256 text rows) with 15 decode rows
        _case("layer_p512_d15", "layer", P=512, d=15, history=516),
        # the second chunk of a prefill (positions 200..299) beside 3 decode rows
        _case("layer_chunk100_d3", "layer", P=100, d=3, ctx=200, history=301),
        # eight pipelines of depth 8 in one forward: 8 x 276 prefill rows and 56 decode rows
        _case("layer_stress_8x276_d56", "layer", pipes=8, P=276, d=56, history=280),
        # the head of the K = 7 step and of the eight-pipeline step
        _case("head_7", "head", d=7),
        _case("head_64", "head", d=64),
        # a whole K = 7 step through four layers and the head
        _case("step_4layers_p276_d6", "step", model="7b4", P=276, d=6, history=280),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny", "head", "decode", "decode", "layer", "layer", "layer", "pipes", "chunk", "step"])
    if kind == "tiny":
        return _case(None, "step", model="tiny", P=_log_int(rng, 8, 200), d=rng.randint(1, 15), history=rng.randint(1, 200))
    if kind == "head":
        return _case(None, "head", d=_log_int(rng, 1, 64))
    if kind == "decode":
        return _case(None, "layer", d=_log_int(rng, 1, 63), history=rng.randint(1, 544))
    if kind == "chunk":
        return _case(None, "layer", P=_log_int(rng, 2, 256), ctx=rng.randint(1, 256), d=_log_int(rng, 1, 31),
                     history=rng.randint(1, 512))
    if kind == "step":
        P = _log_int(rng, 32, 512)
        return _case(None, "step", model="7b4", P=P, d=_log_int(rng, 1, 31), history=P + rng.randint(0, 31))
    pipes = 1 if kind == "layer" else rng.randint(2, 8)
    P = _log_int(rng, 16, 512 if pipes == 1 else 276)
    d = pipes * _log_int(rng, 1, 31 if pipes == 1 else 7)
    return _case(None, "layer", pipes=pipes, P=min(P, MAX_ROWS // pipes), d=d, history=P + rng.randint(0, 31))


# ----------------------------------------------------------------------------- shapes
def _shape(case):
    if case["kind"] == "step":
        return wl.TINY if case["model"] == "tiny" else wl.LLAMA7B.with_layers(4)
    return wl.LLAMA7B.with_layers(1 if case["kind"] == "layer" else 0)


def _specs(case):
    """(request, pos0, q_len) of the step's segments: the prefills, then the decode rows, whose
    contexts vary a little around ``history``."""
    segs = [(100 + p, case["ctx"], case["P"]) for p in range(case["pipes"])] if case["P"] else []
    lo = max(1, case["history"] - 3)
    return segs + [(1000 + i, min(544, lo + i % 7), 1) for i in range(case["d"])]


def _rows(case):
    return sum(q for _, _, q in _specs(case))


# ----------------------------------------------------------------------------- inputs
def _normal(gen, shape, dtype, std=1.0):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _weights(gen, shape):
    """Random weights of ``shape``: N(0, 0.02) matrices, norm gains around 1."""
    D, F, V, dt = shape.d_model, shape.d_ff, shape.vocab, shape.torch_dtype
    gain = lambda: torch.randn(D, generator=gen, device="cuda").mul_(0.1).add_(1.0).to(dt)  # noqa: E731
    g = {"embed": _normal(gen, (V, D), dt, wl.WEIGHT_STD), "final_norm": gain(),
         "lm_head": _normal(gen, (V, D), dt, wl.WEIGHT_STD)}
    layers = []
    for _ in range(shape.n_layers):
        lw = {n: _normal(gen, s, dt, wl.WEIGHT_STD) for n, s in (
            ("wq", (D, D)), ("wk", (D, D)), ("wv", (D, D)), ("wo", (D, D)), ("w_gate", (F, D)), ("w_up", (F, D)),
            ("w_down", (D, F)))}
        lw["attn_norm"], lw["mlp_norm"] = gain(), gain()
        layers.append(lw)
    return g, layers


def _inputs(case, seed):
    """Every tensor of the case from the seed alone: weights, rows, ids and the slots' history."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)
    shape = _shape(case)
    x = {"shape": shape, "specs": _specs(case)}
    x["globals"], x["layers"] = _weights(gen, shape)
    M = _rows(case)
    if case["kind"] == "head":
        x["rows"] = _normal(gen, (M, shape.d_model), shape.torch_dtype)
        return x
    x["rows"] = _normal(gen, (M, shape.d_model), shape.torch_dtype)
    if case["kind"] == "step":
        # the 7B prefill is vision rows and then 20 instruction ids; the tiny one is all ids
        ids = torch.randint(0, shape.vocab, (M,), generator=gen, device="cuda").to(torch.int32)
        if case["model"] != "tiny":
            n_pre = case["pipes"] * case["P"]
            ids[:max(0, n_pre - 20)] = -1
        x["ids"] = ids
    x["kv"] = {}
    for rid, pos0, _ in x["specs"]:
        for layer in range(shape.n_layers):
            if pos0:
                kv = (pos0, shape.n_heads, shape.head_dim)
                x["kv"][rid, layer] = (_normal(gen, kv, shape.torch_dtype), _normal(gen, kv, shape.torch_dtype))
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    shape, specs = x["shape"], x["specs"]
    st = {"case": dict(case), "w": af.Weights(shape, x["globals"], x["layers"])}
    M, V = _rows(case), shape.vocab
    if case["kind"] == "head":
        st["hidden"] = x["rows"]
        # every row the last one of its own request
        st["segs"] = [af.Segment(i, 1, i, 0, 1000 + i, af.AF_SEG_EMIT, 0) for i in range(M)]
        st["logits"] = torch.empty((M, V), dtype=torch.float32, device="cuda")
        st["tokens"] = torch.empty(M, dtype=torch.int32, device="cuda")
        return st
    max_pos = max(p + q for _, p, q in specs)
    ring = af.Ring(shape.n_layers, len(specs) + 1, (max_pos + 31) // 32 * 32, shape.n_heads, shape.head_dim,
                   dtype=shape.torch_dtype)
    segs, row = [], 0
    for rid, pos0, q_len in specs:
        if pos0:
            slot = ring.append(rid, pos0).slot
            for layer in range(shape.n_layers):
                ring.write_kv(layer, slot, 0, *x["kv"][rid, layer])
        s = ring.append(rid, q_len)
        s.q_start, s.flags = row, af.AF_SEG_EMIT
        segs.append(s)
        row += q_len
    st.update(ring=ring, segs=af.segments_array(segs), rows=x["rows"])
    st["hidden"] = torch.empty((M, shape.d_model), dtype=shape.torch_dtype, device="cuda")
    if case["kind"] == "step":
        n = len(specs)
        st["ids"] = x["ids"]
        st["logits"] = torch.empty((n, V), dtype=torch.float32, device="cuda")
        st["tokens"] = torch.empty(n, dtype=torch.int32, device="cuda")
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "head":
        af.op_lm_head_argmax(st["w"], st["hidden"], st["segs"], st["logits"], st["tokens"])
        return {"logits": st["logits"], "tokens": st["tokens"]}
    if kind == "layer":
        # the layer works in place on the residual stream
        st["hidden"].copy_(st["rows"])
        af.packed_layer_forward(st["w"], 0, st["hidden"], st["segs"], st["ring"])
        return {"hidden": st["hidden"]}
    af.packed_forward(st["w"], st["ids"], st["rows"], st["segs"], st["ring"], st["hidden"], st["logits"], st["tokens"])
    # the greedy tokens follow from the logits; between two implementations a near tie may go
    # either way after four bf16 layers, so they are compared in the head cases
    return {"hidden": st["hidden"], "logits": st["logits"]}


# ----------------------------------------------------------------------------- what it takes
def work(case):
    shape, specs = _shape(case), _specs(case)
    D, F, V, L = shape.d_model, shape.d_ff, shape.vocab, shape.n_layers
    es = 2 if shape.dtype == "bf16" else 4
    M, n = _rows(case), len(specs)
    by = fl = 0.0
    if case["kind"] != "head":
        mats = 4 * D * D + 3 * D * F  # q, k, v, o, gate, up, down
        by += L * (mats + 2 * D) * es + 2 * M * D * es  # the weights; the rows in and out
        fl += L * 2.0 * M * mats
        for _, pos0, q in specs:
            by += L * 2 * (pos0 + q) * D * es  # history read, new keys and values written
            fl += L * 4.0 * D * (q * pos0 + q * (q + 1) / 2)
    if case["kind"] != "layer":
        by += (V * D + D) * es + n * V * 4 + n * 4 + (n * D * es if case["kind"] == "head" else 0)
        fl += 2.0 * n * V * D
    return {"bytes": by, "flops": fl}


def tolerance(case):
    shape = _shape(case)
    if shape.dtype == "f32":
        return {"rel": 1e-5}  # two layers of 32-bit sums
    if case["kind"] == "head":
        # the normed row is stored in bf16 (equal on both sides but for single ulps), the sums
        # are fp32; the largest logits lie far further apart than that
        return {"rel": 2e-3, "differ": 0.005}
    # one layer lies 0.004 to 0.005 of the norm from the 64-bit result, four layers 0.011 to 0.014
    return {"rel": 0.015 if case["kind"] == "layer" else 0.03, "max": 0.3}


# ----------------------------------------------------------------------------- 64-bit result
def _norm64(x, g, eps):
    return x * torch.rsqrt(x.square().mean(dim=1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, theta):
    """x [M, H, hd] rotated at positions pos, pairs (j, j + hd/2)."""
    half = x.shape[2] // 2
    ang = pos.double()[:, None] * theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=2)


def _layer64(shape, lw, x, specs, kv):
    D, H, hd = shape.d_model, shape.n_heads, shape.head_dim
    M = x.shape[0]
    pos = torch.cat([torch.arange(p, p + q, device=x.device) for _, p, q in specs])
    xn = _norm64(x, lw["attn_norm"], shape.rms_eps)
    q, k, v = ((xn @ lw[n].double().t()).view(M, H, hd) for n in ("wq", "wk", "wv"))
    q, k = _rope64(q, pos, shape.rope_theta), _rope64(k, pos, shape.rope_theta)
    out = torch.empty_like(q)
    row = 0
    for rid, pos0, n in specs:
        r = slice(row, row + n)
        ks, vs = k[r], v[r]
        if pos0:
            hk, hv = kv[rid]
            ks, vs = torch.cat([hk.double(), ks]), torch.cat([hv.double(), vs])
        qh = q[r].transpose(0, 1).contiguous()                       # [H, n, hd]
        kt = ks.permute(1, 2, 0).contiguous()                        # [H, hd, n_keys]
        sc = torch.bmm(qh, kt) / math.sqrt(hd)
        seen = torch.arange(pos0 + n, device=x.device)[None, :] <= pos[r][:, None]
        pr = torch.softmax(sc.masked_fill(~seen[None], float("-inf")), dim=2)
        out[r] = torch.bmm(pr, vs.transpose(0, 1).contiguous()).transpose(0, 1)
        row += n
    x = x + out.reshape(M, D) @ lw["wo"].double().t()
    xn = _norm64(x, lw["mlp_norm"], shape.rms_eps)
    act = torch.nn.functional.silu(xn @ lw["w_gate"].double().t()) * (xn @ lw["w_up"].double().t())
    return x + act @ lw["w_down"].double().t()


def exact(case, seed):
    x = _inputs(case, seed)
    shape, specs, g = x["shape"], x["specs"], x["globals"]
    h = x["rows"].double()
    if case["kind"] == "step":
        ids = x["ids"].long()
        h = torch.where(ids[:, None] >= 0, g["embed"].double()[ids.clamp(min=0)], h)
    for layer in range(shape.n_layers):
        kv = {rid: x["kv"][rid, layer] for rid, pos0, _ in specs if pos0}
        h = _layer64(shape, x["layers"][layer], h, specs, kv)
    if case["kind"] == "layer":
        return {"hidden": h}
    last = torch.tensor([q for _, _, q in specs], device="cuda").cumsum(0) - 1
    z = _norm64(h[last], g["final_norm"], shape.rms_eps) @ g["lm_head"].double().t()
    if case["kind"] == "head":
        return {"logits": z, "tokens": None}
    return {"hidden": h, "logits": z}

