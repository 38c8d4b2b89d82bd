"""The work that programs built on this library have it do, as measurable cases.

A program that serves a decoder model with block-quantized weights quantizes its matrices once (`quantize`), now and then reads
one back (`dequant`), multiplies a prompt's tokens with them (a prefill: `qgemm` with hundreds to thousands of vectors), and
then decodes: one token at a time (a layer as separate launches, or the whole stack in one), or a handful to a few dozen live
queries at once (`qgemm_fused`, `qgemm`), each step attending over the cached keys and values (`attn_decode`).  The listed cases
are one point of each of these; `draw` picks further points of the same ranges, over all nine formats.

Shapes are those of the repository's benchmark and tests: 4096 / 11008 (7B layers), 8192 / 28672 with 64 query and 8
key/value heads (70B layers), the 1024 x 1024 matrix of the smallest configuration.
"""
import math

import torch

from paper_2401_08294_amd import iflow

HEAD_DIM = 128
EPS = 1e-5
ROPE_BASE = 10000.0
DEVICE = "cuda"
MAX_MAC = 28672 * 8192 * 2000          # multiply-adds of the largest listed case

# format -> (levels - 1, block, bits per weight stored)
FORMAT = {"Q8_B32": (255, 32, 9.0), "Q8_B64": (255, 64, 8.5), "Q6_B64": (63, 64, 6.5), "Q5_B64": (31, 64, 5.5), "Q4_B32": (15, 32, 5.0),
          "Q4_B64": (15, 64, 4.5), "Q3H_B64": (10, 64, 4.0), "Q3_B32": (7, 32, 4.0), "Q2_B32": (3, 32, 3.0)}


def listed():
    return [
        # the smallest call: one token through one 1024 x 1024 projection (latency and host work count)
        {"name": "gemv_1024", "kind": "gemv", "format": "Q3H_B64", "rows": 1024, "cols": 1024},
        # one decoder layer's decode step as the six calls a program issues per layer, grouped-query attention at a short context
        {"name": "layer_step_7b", "kind": "layer", "format": "Q4_B64", "heads": 32, "kv_heads": 8, "ffn": 11008, "position": 511, "max_seq": 1024},
        # a decode step of eight whole layers in one planned launch, multi-head attention at a full kilotoken of context
        {"name": "decode_stack_7b", "kind": "stack", "format": "Q3H_B64", "layers": 8, "heads": 32, "kv_heads": 32, "ffn": 11008, "position": 1000,
         "max_seq": 1024},
        # decode attention alone: multi-head over a context that ends in the middle of a block
        {"name": "attn_mha_3k", "kind": "attn", "heads": 32, "kv_heads": 32, "seq_len": 3001, "max_seq": 4096},
        # ... and eight query heads per key/value head over a long context
        {"name": "attn_gqa_16k", "kind": "attn", "heads": 64, "kv_heads": 8, "seq_len": 16001, "max_seq": 16384},
        # dynamic batching, few live queries: the normalized gate projection of eight tokens
        {"name": "batch8_fused", "kind": "gemm_fused", "format": "Q3H_B64", "rows": 11008, "cols": 4096, "batch": 8, "op": "rms"},
        # dynamic batching, an odd number of queries against long rows, 8-bit weights
        {"name": "batch33_down", "kind": "gemm", "format": "Q8_B64", "rows": 4096, "cols": 11008, "batch": 33},
        # a short prompt, or many live queries: batch between the small and the dense sizes
        {"name": "batch200_proj", "kind": "gemm", "format": "Q5_B64", "rows": 4096, "cols": 4096, "batch": 200},
        # a prompt chunk of 512 tokens through a feed-forward projection
        {"name": "prefill512_ffn", "kind": "gemm", "format": "Q3H_B64", "rows": 11008, "cols": 4096, "batch": 512},
        # the largest: a 2000-token prompt through a feed-forward projection of a large model
        {"name": "prefill2000_ffn", "kind": "gemm", "format": "Q4_B64", "rows": 28672, "cols": 8192, "batch": 2000},
        # loading a model: one fp32 matrix to packed 3.5-bit
        {"name": "quantize_ffn", "kind": "quantize", "format": "Q3H_B64", "rows": 11008, "cols": 4096},
        # reading weights back as fp16
        {"name": "dequant_ffn", "kind": "dequant", "format": "Q6_B64", "rows": 4096, "cols": 11008},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: any format, odd row counts, any multiple of 64 columns, any batch."""
    kind = rng.choice(["gemv", "layer", "stack", "attn", "gemm_fused", "gemm", "gemm", "gemm", "quantize", "dequant"])
    fmt = rng.choice(sorted(FORMAT))
    if kind == "attn":
        kv = rng.choice([1, 2, 4, 8, 16, 32])
        group = rng.choice([1, 1, 2, 3, 4, 8, 16])
        seq = _log_int(rng, 64, 16384 if kv <= 8 else 4096)
        return {"kind": kind, "heads": min(kv * group, 128) // kv * kv, "kv_heads": kv, "seq_len": seq, "max_seq": seq + rng.randrange(1, 600)}
    if kind in ("layer", "stack"):
        heads = rng.choice([8, 16, 32])
        kv = heads // rng.choice([1, 2, 4, 8])
        position = rng.randrange(0, 1500)
        case = {"kind": kind, "format": fmt, "heads": heads, "kv_heads": kv, "ffn": 64 * _log_int(rng, 16, 172), "position": position,
                "max_seq": position + rng.randrange(1, 200)}
        if kind == "stack":
            case["layers"] = rng.randrange(1, 9)
        return case
    cols = 64 * _log_int(rng, 16, 448)
    rows = min(_log_int(rng, 512, 28672), MAX_MAC // 2000 // cols)
    case = {"kind": kind, "format": fmt, "rows": rows, "cols": cols}
    if kind == "gemm_fused":
        case.update(batch=rng.randrange(2, 17), op=rng.choice(["plain", "rms", "silu"]))
    elif kind == "gemm":
        case["batch"] = min(_log_int(rng, 2, 2048), MAX_MAC // (rows * cols))
    return case


# ---- inputs -----------------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _normal(g, shape, sigma=1.0):
    return torch.empty(shape, dtype=torch.float32, device=DEVICE).normal_(0.0, sigma, generator=g)


def _half(g, shape, sigma=1.0, mean=0.0):
    return (_normal(g, shape, sigma) + mean).half()


def _weights(g, rows, cols, sigma=0.02):
    """Zero-mean Gaussian weights with one entry in a thousand ten times larger."""
    w = _normal(g, (rows, cols), sigma)
    return w.mul_(1.0 + 9.0 * (torch.rand((rows, cols), device=DEVICE, generator=g) < 1e-3))


def _layer_shapes(case):
    hidden, kvd, ffn = case["heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM, case["ffn"]
    # name: (rows, cols, gain): entries have the deviation gain / sqrt(cols), so that a layer neither grows nor shrinks its input
    return {"wq": (hidden, hidden, 1.0), "wk": (kvd, hidden, 1.0), "wv": (kvd, hidden, 1.0), "wo": (hidden, hidden, 0.5),
            "w_gate": (ffn, hidden, 2.0), "w_up": (ffn, hidden, 1.0), "w_down": (hidden, ffn, 0.5)}


def _layer_seed(seed, layer):
    return seed * 1009 + layer


def _layer_inputs(case, seed, layer):
    """(matrices fp32 one by one, then gains and caches) of one layer: a generator, so that only one fp32 matrix is held at a time."""
    g = _generator(_layer_seed(seed, layer))
    for name, (rows, cols, gain) in _layer_shapes(case).items():
        yield name, _weights(g, rows, cols, gain / math.sqrt(cols))
    hidden = case["heads"] * HEAD_DIM
    for name in ("norm1", "norm2"):
        yield name, _half(g, (hidden,), 0.2, 1.0)
    cache = torch.zeros((2, case["kv_heads"], case["max_seq"], HEAD_DIM), dtype=torch.float16, device=DEVICE)
    cache[:, :, :case["position"]] = _half(g, (2, case["kv_heads"], case["position"], HEAD_DIM))
    yield "cache", cache


def _hidden_state(case, seed):
    return _half(_generator(seed + 77), (case["heads"] * HEAD_DIM,))


def _gemm_inputs(case, seed):
    g = _generator(seed)
    rows, cols, batch = case["rows"], case["cols"], case.get("batch", 1)
    w = _weights(g, rows, cols)
    x = _half(g, (batch, cols))
    op = case.get("op", "plain")
    aux = _half(g, (cols,), 0.2, 1.0) if op == "rms" else _half(g, (batch, cols)) if op == "silu" else None
    residual = _half(g, (batch, rows)) if case["kind"] == "gemm_fused" else None
    return w, x, aux, residual


def _attn_inputs(case, seed):
    g = _generator(seed)
    q = _half(g, (case["heads"], HEAD_DIM))
    cache = _half(g, (2, case["kv_heads"], case["max_seq"], HEAD_DIM))
    return q, cache


def _pack(fmt, w):
    rows, cols = w.shape
    code = iflow.FORMATS[fmt]
    n = iflow.packed_bytes(code, rows, cols)
    packed = torch.empty((n,), dtype=torch.uint8, device=DEVICE)
    iflow.quantize(code, w, rows, cols, packed, n)
    return packed


def _out(*shape):
    return torch.empty(shape, dtype=torch.float16, device=DEVICE)


def _prepare_layer(case, seed, layer):
    st = {}
    for name, t in _layer_inputs(case, seed, layer):
        st[name] = _pack(case["format"], t) if name.startswith("w") else t
    st["k_cache"], st["v_cache"] = st["cache"][0], st["cache"][1]
    return st


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "kind": kind}
    if "format" in case:
        st["fmt"] = iflow.FORMATS[case["format"]]
    if kind in ("gemv", "gemm", "gemm_fused"):
        w, st["x"], st["aux"], st["residual"] = _gemm_inputs(case, seed)
        st["packed"] = _pack(case["format"], w)
        st["y"] = _out(case.get("batch", 1), case["rows"])
    elif kind == "quantize":
        st["w"] = _weights(_generator(seed), case["rows"], case["cols"])
        st["n"] = iflow.packed_bytes(st["fmt"], case["rows"], case["cols"])
        st["packed"] = torch.empty((st["n"],), dtype=torch.uint8, device=DEVICE)
    elif kind == "dequant":
        st["packed"] = _pack(case["format"], _weights(_generator(seed), case["rows"], case["cols"]))
        st["w16"] = _out(case["rows"], case["cols"])
    elif kind == "attn":
        st["q"], cache = _attn_inputs(case, seed)
        st["k"], st["v"] = cache[0], cache[1]
        st["ws_bytes"] = iflow.attn_decode_workspace_bytes(case["heads"])
        st["ws"] = torch.empty((st["ws_bytes"],), dtype=torch.uint8, device=DEVICE)
        st["out"] = _out(case["heads"], HEAD_DIM)
    elif kind == "layer":
        st.update(_prepare_layer(case, seed, 0))
        hidden, kvd = case["heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM
        st["h"] = _hidden_state(case, seed)
        st["q"], st["k"], st["v"], st["t"] = _out(hidden), _out(kvd), _out(kvd), _out(hidden)
        st["h1"], st["a"], st["h2"] = _out(hidden), _out(case["ffn"]), _out(hidden)
        st["ws_bytes"] = iflow.attn_decode_workspace_bytes(case["heads"])
        st["ws"] = torch.empty((st["ws_bytes"],), dtype=torch.uint8, device=DEVICE)
    elif kind == "stack":
        hidden, n = case["heads"] * HEAD_DIM, case["layers"]
        st["layers"] = [_prepare_layer(case, seed, i) for i in range(n)]
        st["h"], st["h_out"] = _hidden_state(case, seed), _out(hidden)
        shape = (st["fmt"], hidden, case["ffn"], case["heads"], case["kv_heads"], case["max_seq"], EPS, ROPE_BASE, iflow.ROPE_HALVES)
        scratch, plan, ws = iflow.decode_stack_sizes(iflow.decode_stack(*shape, n_layers=n))
        st["scratch"] = torch.zeros((n, scratch // 2 // n), dtype=torch.float16, device=DEVICE)
        st["plan"] = torch.empty((plan,), dtype=torch.uint8, device=DEVICE)
        st["ws"] = torch.empty((ws,), dtype=torch.uint8, device=DEVICE)
        desc = iflow.decode_stack(*shape, layers=st["layers"], h_in=st["h"], h_out=st["h_out"], scratch=st["scratch"])
        st["chain"] = iflow.decode_stack_plan(desc, st["plan"], plan, st["ws"], ws)
    return st


def run(st):
    case, kind = st["case"], st["kind"]
    if kind == "gemv":
        iflow.qgemv(st["fmt"], st["packed"], case["rows"], case["cols"], st["x"], st["y"])
        return st["y"]
    if kind == "gemm":
        iflow.qgemm(st["fmt"], st["packed"], case["rows"], case["cols"], st["x"], case["batch"], st["y"])
        return st["y"]
    if kind == "gemm_fused":
        op = {"plain": iflow.X_PLAIN, "rms": iflow.X_RMS_GAIN, "silu": iflow.X_SILU_MUL}[case["op"]]
        iflow.qgemm_fused(st["fmt"], st["packed"], case["rows"], case["cols"], st["x"], case["batch"], st["y"], op, st["aux"], EPS, st["residual"])
        return st["y"]
    if kind == "quantize":
        iflow.quantize(st["fmt"], st["w"], case["rows"], case["cols"], st["packed"], st["n"])
        return st["packed"]
    if kind == "dequant":
        iflow.dequant(st["fmt"], st["packed"], case["rows"], case["cols"], st["w16"])
        return st["w16"]
    if kind == "attn":
        iflow.attn_decode(st["q"], st["k"], st["v"], case["heads"], case["kv_heads"], HEAD_DIM, case["seq_len"], case["max_seq"],
                          HEAD_DIM ** -0.5, st["out"], st["ws"], st["ws_bytes"])
        return st["out"]
    if kind == "layer":
        fmt, heads, kv, ffn, pos = st["fmt"], case["heads"], case["kv_heads"], case["ffn"], case["position"]
        hidden, kvd = heads * HEAD_DIM, kv * HEAD_DIM
        iflow.qgemv_fused(fmt, [st["wq"], st["wk"], st["wv"]], [hidden, kvd, kvd], hidden, st["h"], [st["q"], st["k"], st["v"]],
                          iflow.X_RMS_GAIN, st["norm1"], EPS)
        iflow.rope_append(st["q"], st["k"], st["v"], heads, kv, HEAD_DIM, pos, case["max_seq"], ROPE_BASE, iflow.ROPE_HALVES, st["k_cache"],
                          st["v_cache"])
        iflow.attn_decode(st["q"], st["k_cache"], st["v_cache"], heads, kv, HEAD_DIM, pos + 1, case["max_seq"], HEAD_DIM ** -0.5, st["t"],
                          st["ws"], st["ws_bytes"])
        iflow.qgemv_fused(fmt, [st["wo"]], [hidden], hidden, st["t"], [st["h1"]], residual_list=[st["h"]])
        iflow.qgemv_gated(fmt, st["w_gate"], st["w_up"], ffn, hidden, st["h1"], st["a"], iflow.X_RMS_GAIN, st["norm2"], EPS)
        iflow.qgemv_fused(fmt, [st["w_down"]], [hidden], ffn, st["a"], [st["h2"]], residual_list=[st["h1"]])
        return [st[name] for name in ("q", "k", "v", "t", "h1", "a", "h2", "cache")]
    iflow.decode_stack_launch(st["chain"], case["position"])
    return [st["h_out"], st["scratch"]] + [layer["cache"] for layer in st["layers"]]


# ---- what a pass cannot do without --------------------------------------------------------------------------------------------

def _packed(case, rows, cols):
    return rows * cols * FORMAT[case["format"]][2] / 8


def work(case):
    kind = case["kind"]
    if kind in ("gemv", "gemm", "gemm_fused"):
        rows, cols, batch = case["rows"], case["cols"], case.get("batch", 1)
        nbytes = _packed(case, rows, cols) + 2 * batch * (rows + cols)
        if kind == "gemm_fused":
            nbytes += 2 * batch * rows + {"plain": 0, "rms": 2 * cols, "silu": 2 * batch * cols}[case["op"]]
        return {"bytes": nbytes, "flops": 2.0 * rows * cols * batch}
    if kind == "quantize":
        return {"bytes": 4.0 * case["rows"] * case["cols"] + _packed(case, case["rows"], case["cols"]), "flops": 0.0}
    if kind == "dequant":
        return {"bytes": 2.0 * case["rows"] * case["cols"] + _packed(case, case["rows"], case["cols"]), "flops": 0.0}
    if kind == "attn":
        return {"bytes": 4.0 * case["kv_heads"] * case["seq_len"] * HEAD_DIM + 4.0 * case["heads"] * HEAD_DIM,
                "flops": 4.0 * case["heads"] * case["seq_len"] * HEAD_DIM}
    layers = case.get("layers", 1)
    weights = sum(r * c for r, c, _ in _layer_shapes(case).values())
    attended = case["position"] + 1
    vectors = 2 * (6 * case["heads"] * HEAD_DIM + 4 * case["kv_heads"] * HEAD_DIM + case["ffn"])
    return {"bytes": layers * (_packed(case, 1, weights) + 4.0 * case["kv_heads"] * attended * HEAD_DIM + vectors),
            "flops": layers * (2.0 * weights + 4.0 * case["heads"] * attended * HEAD_DIM)}


def tolerance(case):
    """About four times the distance from the 64-bit results that the path shows (2-norm): 2.1e-4 to 2.9e-4 for one product, 2.0e-4 to
    2.6e-4 for the attention (one fp16 rounding of the output each), 5.3e-4 over one layer's stages, 1.5e-3 after eight layers."""
    kind = case["kind"]
    if kind in ("quantize", "dequant"):
        return "exact"
    if kind == "layer":
        return {"rel": 2.5e-3, "max": 2e-2}
    if kind == "stack":
        return {"rel": 6e-3, "max": 6e-2}
    return {"rel": 1.2e-3, "max": 8e-3}


# ---- the same results in 64 bits ------------------------------------------------------------------------------------------------

def _read_back(fmt, w):
    """The weights as the format holds them: per block the fp16 pair (scale, offset) and whole levels, Eq.1 to Eq.3 of the paper."""
    top, block, _ = FORMAT[fmt]
    rows, cols = w.shape
    out = torch.empty((rows, cols), dtype=torch.float64, device=w.device)
    step = max(1, (1 << 26) // cols)
    for r0 in range(0, rows, step):                            # (a slice of rows at a time: 64-bit copies are large)
        wb = w[r0:r0 + step].reshape(-1, cols // block, block)
        mn, mx = wb.amin(-1, keepdim=True), wb.amax(-1, keepdim=True)
        scale = (((mx - mn).double() / top).float()).half().double()
        offset = mn.half().double()
        t = ((wb.double() - offset).float().double() / scale).float().double()
        level = (t.floor() + ((t - t.floor()) >= 0.5)).clamp(0, top)
        level = torch.where(scale == 0, torch.zeros_like(level), level)
        out[r0:r0 + step] = (level * scale + offset).reshape(-1, cols)
    return out


def _held(fmt, w):
    """... rounded to the fp16 values that every product is defined on."""
    return _read_back(fmt, w).half().double()


def _rms(x, gain):
    return x * gain / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)


def _silu(x):
    return x * torch.sigmoid(x)


def _attend(q, k, v):
    """q [heads][128] over k, v [kv heads][positions][128], all 64-bit."""
    group = q.shape[0] // k.shape[0]
    out = torch.empty_like(q)
    for i in range(q.shape[0]):
        p = torch.softmax(k[i // group] @ q[i] * HEAD_DIM ** -0.5, 0)
        out[i] = v[i // group].T.contiguous() @ p
    return out


def _rotate(x, position):
    half = HEAD_DIM // 2
    angle = position * torch.pow(torch.tensor(ROPE_BASE, dtype=torch.float64, device=x.device),
                                 -torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a, b = x[:, :half], x[:, half:]
    return torch.cat([a * angle.cos() - b * angle.sin(), a * angle.sin() + b * angle.cos()], 1)


def _exact_layer(case, seed, layer, h):
    parts, w = {}, {}
    for name, t in _layer_inputs(case, seed, layer):
        if name.startswith("w"):
            w[name] = _held(case["format"], t)
        else:
            parts[name] = t.double()
    heads, kv, pos = case["heads"], case["kv_heads"], case["position"]
    n1 = _rms(h, parts["norm1"])
    q, k, v = w["wq"] @ n1, w["wk"] @ n1, w["wv"] @ n1
    rotated = _rotate(q.view(heads, HEAD_DIM), pos)
    cache = parts["cache"]
    cache[0, :, pos] = _rotate(k.view(kv, HEAD_DIM), pos)
    cache[1, :, pos] = v.view(kv, HEAD_DIM)
    t = _attend(rotated, cache[0, :, :pos + 1], cache[1, :, :pos + 1]).reshape(-1)
    h1 = h + w["wo"] @ t
    n2 = _rms(h1, parts["norm2"])
    a = _silu(w["w_gate"] @ n2) * (w["w_up"] @ n2)
    h2 = h1 + w["w_down"] @ a
    return {"q": q, "rotated": rotated.reshape(-1), "k": k, "v": v, "t": t, "h1": h1, "a": a, "h2": h2, "cache": cache}


def exact(case, seed):
    kind = case["kind"]
    if kind == "quantize":
        return None                                            # bytes
    if kind == "dequant":
        return _read_back(case["format"], _weights(_generator(seed), case["rows"], case["cols"]))
    if kind == "attn":
        q, cache = _attn_inputs(case, seed)
        kv = cache[:, :, :case["seq_len"]].double()
        return _attend(q.double(), kv[0], kv[1])
    if kind in ("gemv", "gemm", "gemm_fused"):
        w, x, aux, residual = _gemm_inputs(case, seed)
        x = x.double()
        op = case.get("op", "plain")
        if op == "rms":
            x = _rms(x, aux.double())
        elif op == "silu":
            x = _silu(x) * aux.double()
        y = torch.empty((x.shape[0], case["rows"]), dtype=torch.float64, device=DEVICE)
        for r0 in range(0, case["rows"], 4096):
            y[:, r0:r0 + 4096] = x @ _held(case["format"], w[r0:r0 + 4096]).T.contiguous()
        return y if residual is None else y + residual.double()
    h = _hidden_state(case, seed).double()
    if kind == "layer":
        s = _exact_layer(case, seed, 0, h)
        return [s["rotated"], s["k"], s["v"], s["t"], s["h1"], s["a"], s["h2"], s["cache"]]
    caches, n = [], case["layers"]
    round_up = lambda m: (m + 127) // 128 * 128
    per_layer = sum(round_up(m) for m in (h.numel(), case["kv_heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM, h.numel(), h.numel(),
                                          case["ffn"], h.numel()))
    scratch = torch.zeros((n, per_layer), dtype=torch.float64, device=DEVICE)
    for layer in range(n):
        s = _exact_layer(case, seed, layer, h)
        at = 0
        for name in ("q", "k", "v", "t", "h1", "a", "h2"):
            if not (name == "h2" and layer == n - 1):          # the last layer's output goes to h_out instead
                scratch[layer, at:at + s[name].numel()] = s[name]
            at += round_up(s[name].numel())
        caches.append(s["cache"])
        h = s["h2"]
    return [h, scratch] + caches
