"""The work whose speed counts: unit-scaled linear layers, FFN layers, attention, layer norm, the softmax cross-entropy
and the scaled FP8 cast, called as a training or inference program calls them.

``listed()`` names the cases, ``draw(rng)`` gives others of the same ranges.  ``prepare`` makes what a program has in hand
before the call (inputs from the seed, buffers, workspace, the GELU tables, and, where the weights do not change from call to
call, their FP8 copies), ``run`` makes one pass and returns its results, ``work`` counts the bytes and operations the pass
cannot do without, ``tolerance`` how far another correct implementation at the same precision may be off.
"""
import math

import torch

import paper_2303_11257_amd as us

DEV = "cuda:0"
ACTS = {"none": 0, "gelu": us.ACT_GELU, "relu": us.ACT_RELU, "tanh": us.ACT_TANH, "sigmoid": us.ACT_SIGMOID}
EPI_ACT = {"gelu": 0, "relu": us.EPI_ACT_RELU, "tanh": us.EPI_ACT_TANH, "sigmoid": us.EPI_ACT_SIGMOID}
MAX_FFN_FLOPS = 12.0 * 32768 * 4096 * 16384


def listed():
    return [
        # one small linear layer, FP16, forward and backward: latency and launches count
        dict(name="linear_small", kind="linear", b=256, m=256, n=1024, fp8=False, act="none", back=True),
        # one FP8 linear layer with a ReLU in its epilogue and odd sizes, few tiles and a ragged last tile everywhere
        dict(name="linear_ragged_relu", kind="linear", b=2000, m=1552, n=2064, fp8=True, act="relu", back=True),
        # BERT-base FFN in FP16, forward and backward: the ordinary mixed-precision training step
        dict(name="ffn_f16_base", kind="ffn", tokens=4096, d=768, f=3072, fp8=False, variant="plain", back=True),
        # BERT-large FFN in FP8 with its casts, forward and backward: the headline training step
        dict(name="ffn_fp8_large", kind="ffn", tokens=8192, d=1024, f=4096, fp8=True, variant="plain", back=True),
        # LLM-size FFN in FP8, forward and backward: the largest call
        dict(name="ffn_fp8_llm", kind="ffn", tokens=32768, d=4096, f=16384, fp8=True, variant="plain", back=True),
        # FFN with bias rows and their gradients, FP16, on a batch of packed sequences whose token count is no multiple of a tile
        dict(name="ffn_f16_bias_ragged", kind="ffn", tokens=4016, d=1008, f=4000, fp8=False, variant="bias", back=True),
        # residual FFN layer in FP8, forward only, on the tokens of a small inference batch; the weights' FP8 copies are kept
        dict(name="ffn_fp8_infer", kind="ffn", tokens=64, d=1024, f=4096, fp8=True, variant="residual", back=False),
        # attention over 512 tokens, 256 heads, forward and backward
        dict(name="attention_512", kind="attention", heads=256, s=512, d=64, back=True),
        # attention of a BERT-large layer on sequences of 128 (64 sequences, 16 heads each)
        dict(name="attention_128", kind="attention", heads=1024, s=128, d=64, back=True),
        # the layer norm between two such layers, forward and backward
        dict(name="layer_norm", kind="layer_norm", b=8192, n=1024, back=True),
        # the end of a language model: loss and gradient over a vocabulary of 30528
        dict(name="xent_vocab", kind="xent", rows=8192, s=30528),
        # range stress: both operands cast from FP32 to E4M3 with saturation counters, then their product
        dict(name="range_stress", kind="cast_matmul", b=4096, m=4096, n=4096, sigma=8.0),
    ]


def _size(rng, lo, hi, unit=16):
    """A multiple of `unit` in lo .. hi, spread over the logarithm; every other one a multiple of 128 where that fits."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5 and v >= 128:
        unit = 128
    return int(min(hi // unit * unit, max(lo, round(v / unit) * unit)))


def draw(rng):
    kind = rng.choice(["linear", "linear", "ffn", "ffn", "ffn", "attention", "attention", "layer_norm", "xent", "cast_matmul"])
    if kind == "linear":
        return dict(kind=kind, b=_size(rng, 16, 16384), m=_size(rng, 128, 4096), n=_size(rng, 128, 4096),
                    fp8=rng.random() < 0.5, act=rng.choice(["none", "none", "gelu", "relu", "tanh", "sigmoid"]),
                    back=rng.random() < 0.7)
    if kind == "ffn":
        while True:
            d = _size(rng, 128, 4096)
            case = dict(kind=kind, tokens=_size(rng, 16, 32768), d=d, f=int(d * rng.choice([2, 3, 4, 4, 4])) // 16 * 16,
                        fp8=rng.random() < 0.6, variant=rng.choice(["plain", "plain", "bias", "residual"]),
                        back=rng.random() < 0.7)
            if work(case)["flops"] * (1 if case["fp8"] else 2.2) <= MAX_FFN_FLOPS:
                return case
    if kind == "attention":
        s, d = _size(rng, 32, 2048), rng.choice([32, 48, 64, 64, 64, 80, 96, 128])
        most = max(1, min(1024, 2 ** 26 // (s * s)))
        return dict(kind=kind, heads=int(math.exp(rng.uniform(0.0, math.log(most)))), s=s, d=d, back=rng.random() < 0.8)
    if kind == "layer_norm":
        return dict(kind=kind, b=int(math.exp(rng.uniform(math.log(64), math.log(65536)))), n=_size(rng, 128, 4096),
                    back=rng.random() < 0.7)
    if kind == "xent":
        return dict(kind=kind, rows=int(math.exp(rng.uniform(math.log(64), math.log(16384)))), s=_size(rng, 256, 65536, 8))
    return dict(kind=kind, b=_size(rng, 256, 8192), m=_size(rng, 256, 8192), n=_size(rng, 256, 8192),
                sigma=rng.choice([1.0 / 64, 1.0 / 8, 1.0, 8.0, 64.0]))


# ---- what a program has in hand ---------------------------------------------------------------------------------------

class _Buffers:
    """Tensors of one case by name; p(name) is the device address the library takes (None for a tensor that is not there)."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)
        self.t = {}

    def normal(self, name, *shape, sigma=1.0, dtype=torch.float16):
        x = torch.empty(shape, dtype=dtype, device=DEV)
        x.normal_(0.0, sigma, generator=self.gen)
        self.t[name] = x
        return x

    def empty(self, name, *shape, dtype=torch.float16):
        self.t[name] = torch.empty(shape, dtype=dtype, device=DEV)
        return self.t[name]

    def codes(self, name, *shape):
        return self.empty(name, *shape, dtype=torch.uint8)

    def p(self, name):
        x = self.t.get(name)
        return None if x is None else x.data_ptr()

    def results(self, *names):
        return {n: self.t[n] for n in names if n in self.t}


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _cast(B, *pairs):
    """One batched cast: (source, destination, FP8 type) by name."""
    us.cast_fp8_batch([B.p(s) for s, _, _ in pairs], [B.p(d) for _, d, _ in pairs], [B.t[s].numel() for s, _, _ in pairs],
                      [f for _, _, f in pairs], _stream())


def _workspace(B, nbytes, tables):
    B.empty("ws", max(nbytes, us.TABLE_AREA_BYTES), dtype=torch.uint8)
    B.wsb = B.t["ws"].numel()
    if tables:                    # built once per run of a program, like the workspace itself
        us.gelu_tables(B.p("ws"), B.wsb, 0.0, 0.0, _stream())


def prepare(case, seed):
    B = _Buffers(seed)
    B.case = case
    _PREPARE[case["kind"]](B, case)
    B.gen = None
    return B


def _prepare_linear(B, c):
    b, m, n = c["b"], c["m"], c["n"]
    B.normal("X", b, m)
    B.normal("W", m, n)
    B.empty("Y", b, n)
    if c["act"] != "none":
        B.codes("A8", b, n) if c["fp8"] else B.empty("A", b, n)
    if c["fp8"]:
        B.codes("X8", b, m), B.codes("W8", m, n)
    if c["back"]:
        B.normal("G", b, n)
        if c["fp8"]:
            B.codes("G8", b, n)
        if c["act"] != "none":
            B.normal("Zpre", b, m)           # the pre-activation that this layer's input came from
            if c["fp8"]:
                B.codes("dX8", b, m)
        B.empty("dX", b, m), B.empty("dW", m, n)
    elif c["fp8"]:
        _cast(B, ("W", "W8", us.E4M3))       # inference: the weights' codes are kept
    _workspace(B, us.workspace_bytes(b, m, n), c["act"] == "gelu")


def _prepare_ffn(B, c):
    T, d, f = c["tokens"], c["d"], c["f"]
    B.normal("X", T, d), B.normal("W1", d, f), B.normal("W2", f, d)
    if c["variant"] == "bias":
        B.normal("b1", f, sigma=0.1), B.normal("b2", d, sigma=0.1)
    B.empty("Z", T, f), B.empty("Y", T, d)
    B.codes("H", T, f) if c["fp8"] else B.empty("H", T, f)
    if c["fp8"]:
        B.codes("X8", T, d), B.codes("W1_8", d, f), B.codes("W2_8", f, d)
    if c["back"]:
        B.normal("G", T, d)
        if c["fp8"]:
            B.codes("G8", T, d), B.codes("dZ8", T, f)
        else:
            B.empty("dZ", T, f)
        B.empty("dX", T, d), B.empty("dW1", d, f), B.empty("dW2", f, d)
        if c["variant"] == "bias":
            B.empty("db1", f), B.empty("db2", d)
    elif c["fp8"]:
        _cast(B, ("W1", "W1_8", us.E4M3), ("W2", "W2_8", us.E4M3))
    _workspace(B, us.ffn_bias_workspace_bytes(T, d, f) if c["variant"] == "bias" else us.ffn_workspace_bytes(T, d, f), True)


def _prepare_attention(B, c):
    h, s, d = c["heads"], c["s"], c["d"]
    for n in ("Q", "K", "V"):
        B.normal(n, h, s, d)
    B.empty("A", h, s, s), B.empty("P", h, s, s), B.empty("O", h, s, d)
    if c["back"]:
        B.normal("dO", h, s, d)
        B.empty("dP", h, s, s), B.empty("dA", h, s, s)
        for n in ("dQ", "dK", "dV"):
            B.empty(n, h, s, d)


def _prepare_layer_norm(B, c):
    b, n = c["b"], c["n"]
    B.normal("X", b, n), B.normal("w", n), B.normal("c", n, sigma=0.1), B.empty("Y", b, n)
    if c["back"]:
        B.normal("G", b, n), B.empty("dX", b, n), B.empty("dw", n), B.empty("dc", n)
        B.wsb = us.layer_norm_workspace_bytes(b, n)
        B.empty("ws", max(16, B.wsb), dtype=torch.uint8)


def _prepare_xent(B, c):
    rows, s = c["rows"], c["s"]
    B.normal("X", rows, s)
    t = torch.randint(0, s, (rows,), generator=B.gen, device=DEV, dtype=torch.int32)
    skip = torch.rand((rows,), generator=B.gen, device=DEV) < 0.1        # positions without a label
    B.t["target"] = torch.where(skip, torch.full_like(t, -1), t)
    B.empty("loss", rows, dtype=torch.float32), B.empty("dX", rows, s)


def _prepare_cast_matmul(B, c):
    b, m, n = c["b"], c["m"], c["n"]
    for name, shape in (("X", (b, m)), ("W", (m, n))):
        x = B.normal(name, *shape, sigma=c["sigma"], dtype=torch.float32)
        at = torch.randint(0, x.numel(), (x.numel() // 1000,), generator=B.gen, device=DEV)
        x.view(-1)[at] = torch.where(at % 2 == 0, 1000.0, -1000.0).to(x.dtype)      # one in a thousand an outlier
        B.codes(name + "8", *shape)
    B.empty("Y", b, n)
    B.empty("stats", 2, 4, dtype=torch.int64)


_PREPARE = dict(linear=_prepare_linear, ffn=_prepare_ffn, attention=_prepare_attention, layer_norm=_prepare_layer_norm,
                xent=_prepare_xent, cast_matmul=_prepare_cast_matmul)


# ---- one pass -----------------------------------------------------------------------------------------------------------

def run(state):
    return _RUN[state.case["kind"]](state, state.case)


def _run_linear(B, c):
    b, m, n, st, p = c["b"], c["m"], c["n"], _stream(), B.p
    x = w = g = us.F16
    X, W, G = "X", "W", "G"
    if c["fp8"]:
        X, W, G, x, w, g = "X8", "W8", "G8", us.E4M3, us.E4M3, us.E5M2
        if c["back"]:
            _cast(B, ("X", "X8", us.E4M3), ("W", "W8", us.E4M3), ("G", "G8", us.E5M2))
        else:
            _cast(B, ("X", "X8", us.E4M3))
    act = c["act"] != "none"
    ready = us.EPI_TABLES_READY if c["act"] == "gelu" else 0
    fwd = (us.EPI_GELU | EPI_ACT[c["act"]] | ready) if act else us.EPI_NONE
    us.linear_fwd(p(X), p(W), p("Y"), b, m, n, x, w, us.F16, 0.0, fwd, 0.0, p("A"), p("A8"), p("ws"), B.wsb, st)
    if c["back"]:
        bwd = (us.EPI_GELU_GRAD | EPI_ACT[c["act"]] | ready) if act else us.EPI_NONE
        us.linear_bwd(p(X), p(W), p(G), p("dX"), p("dW"), b, m, n, x, w, g, us.F16, 0.0, 0.0, bwd, 0.0, p("Zpre"), p("dX8"),
                      p("ws"), B.wsb, st)
    return B.results("Y", "A", "A8", "dX", "dX8", "dW")


def _run_ffn(B, c):
    T, d, f, st, p = c["tokens"], c["d"], c["f"], _stream(), B.p
    X, W1, W2, G = "X", "W1", "W2", "G"
    if c["fp8"]:
        X, W1, W2, G = "X8", "W1_8", "W2_8", "G8"
        if c["back"]:
            _cast(B, ("X", X, us.E4M3), ("W1", W1, us.E4M3), ("W2", W2, us.E4M3), ("G", G, us.E5M2))
        else:
            _cast(B, ("X", X, us.E4M3))
    mode = (us.FFN_FP8 if c["fp8"] else 0) | us.FFN_TABLES_READY
    ws = (p("ws"), B.wsb, st)
    if c["variant"] == "bias":
        us.ffn_bias_fwd(p(X), p(W1), p("b1"), p(W2), p("b2"), p("Z"), p("H"), p("Y"), T, d, f, mode, *ws)
        if c["back"]:
            us.ffn_bias_bwd(p(X), p(W1), p(W2), p("Z"), p("H"), p(G), p("G"), p("dZ"), p("dZ8"), p("dX"), p("dW1"), p("dW2"),
                            p("db1"), p("db2"), T, d, f, mode, *ws)
    elif c["variant"] == "residual":
        us.ffn_res_fwd(p("X"), p(X), p(W1), p(W2), p("Z"), p("H"), p("Y"), T, d, f, 0.5, mode, *ws)
        if c["back"]:
            us.ffn_res_bwd(p(X), p(W1), p(W2), p("Z"), p("H"), p("G"), p(G), p("dZ"), p("dZ8"), p("dX"), p("dW1"), p("dW2"),
                           T, d, f, 0.5, mode, *ws)
    else:
        us.ffn_fwd(p(X), p(W1), p(W2), p("Z"), p("H"), p("Y"), T, d, f, mode, *ws)
        if c["back"]:
            us.ffn_bwd(p(X), p(W1), p(W2), p("Z"), p("H"), p(G), p("dZ"), p("dZ8"), p("dX"), p("dW1"), p("dW2"), T, d, f,
                       mode, *ws)
    return B.results("Y", "dX", "dW1", "dW2", "db1", "db2")


def _run_attention(B, c):
    h, s, d, st, p = c["heads"], c["s"], c["d"], _stream(), B.p
    us.attention_fwd(p("Q"), p("K"), p("V"), p("A"), p("P"), p("O"), h, s, d, st)
    if c["back"]:
        us.attention_bwd(p("Q"), p("K"), p("V"), p("A"), p("P"), p("dO"), p("dP"), p("dA"), p("dQ"), p("dK"), p("dV"), h, s, d, st)
    return B.results("O", "A", "P", "dP", "dA", "dQ", "dK", "dV")


def _run_layer_norm(B, c):
    b, n, st, p = c["b"], c["n"], _stream(), B.p
    us.layer_norm_fwd(p("X"), p("w"), p("c"), p("Y"), b, n, 1e-5, st)
    if c["back"]:
        us.layer_norm_bwd(p("X"), p("w"), p("G"), p("dX"), p("dw"), p("dc"), b, n, 1e-5, 0.0, p("ws"), B.wsb, st)
    return B.results("Y", "dX", "dw", "dc")


def _run_xent(B, c):
    us.softmax_xent(B.p("X"), B.p("target"), B.p("loss"), B.p("dX"), c["rows"], c["s"], 0.0, 0.0, _stream())
    return B.results("loss", "dX")


def _run_cast_matmul(B, c):
    b, m, n, st, p = c["b"], c["m"], c["n"], _stream(), B.p
    scale = 1.0 / c["sigma"]
    B.t["stats"].zero_()                                   # the counters are the caller's to clear
    at = p("stats")
    us.cast_fp8(p("X"), us.F32, p("X8"), us.E4M3, b * m, scale, at, st)
    us.cast_fp8(p("W"), us.F32, p("W8"), us.E4M3, m * n, scale, at + 32, st)
    us.linear_fwd(p("X8"), p("W8"), p("Y"), b, m, n, us.E4M3, us.E4M3, us.F16, 0.0, us.EPI_NONE, 0.0, None, None, None, 0, st)
    return B.results("X8", "W8", "stats", "Y")


_RUN = dict(linear=_run_linear, ffn=_run_ffn, attention=_run_attention, layer_norm=_run_layer_norm, xent=_run_xent,
            cast_matmul=_run_cast_matmul)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def work(case):
    """Every tensor that an entry point takes is read once and every one that it fills is written once, per call; a matmul
    is 2 operations per product, everything else counts as traffic."""
    c, k = case, case["kind"]
    if k == "linear":
        b, m, n = c["b"], c["m"], c["n"]
        es, act, back = (1 if c["fp8"] else 2), c["act"] != "none", c["back"]
        fwd = es * (b * m + m * n) + 2 * b * n + (es * b * n if act else 0)
        bwd = es * (b * m + m * n + b * n) + 2 * (b * m + m * n) + ((2 + (1 if c["fp8"] else 0)) * b * m if act else 0)
        cast = 3 * (b * m + (m * n + b * n if back else 0)) if c["fp8"] else 0
        return {"bytes": float(cast + fwd + (bwd if back else 0)), "flops": 2.0 * b * m * n * (3 if back else 1)}
    if k == "ffn":
        T, d, f, back = c["tokens"], c["d"], c["f"], c["back"]
        es = 1 if c["fp8"] else 2
        res, bias = c["variant"] == "residual", c["variant"] == "bias"
        fwd = es * (T * d + 2 * d * f + T * f) + (2 + es) * T * f + 2 * T * d + (2 * T * d if res else 0)
        bwd = es * (2 * T * d + 2 * d * f + 2 * T * f) + 2 * T * f + es * T * f + 2 * (T * d + 2 * d * f) + (2 * T * d if res or bias else 0)
        cast = 3 * (T * d + (T * d + 2 * d * f if back else 0)) if c["fp8"] else 0
        return {"bytes": float(cast + fwd + (bwd if back else 0)), "flops": 4.0 * T * d * f * (3 if back else 1)}
    if k == "attention":
        h, s, d, back = c["heads"], c["s"], c["d"], c["back"]
        fwd = 2 * h * (4 * s * d + 2 * s * s)
        bwd = 2 * h * (7 * s * d + 4 * s * s)
        return {"bytes": float(fwd + (bwd if back else 0)), "flops": 4.0 * h * s * s * d * (3 if back else 1)}
    if k == "layer_norm":
        e = c["b"] * c["n"]
        return {"bytes": float(4 * e + (6 * e if c["back"] else 0)), "flops": 0.0}
    if k == "xent":
        return {"bytes": float(4 * c["rows"] * c["s"] + 8 * c["rows"]), "flops": 0.0}
    b, m, n = c["b"], c["m"], c["n"]
    return {"bytes": float(6 * (b * m + m * n) + 2 * b * n), "flops": 2.0 * b * m * n}


def tolerance(case):
    """Four times what the library and the same chain in float64 (with the same rounding points) were seen to differ by, over the
    listed cases (the two largest scaled down) and 24 drawn ones.  FP16 results of FP32 sums differ by single flips of the last
    place; behind a chain of products a flip of an FP8 code at a rounding boundary moves one product by up to an eighth, and the
    matrix core adds FP8 products with about 14 bits."""
    c, k = case, case["kind"]
    if k == "linear":        # seen: FP16 2.4e-5, at most 1.5e-3; FP8 7.7e-5, at most 1.8e-3, codes 3.9e-4 of the values
        return {"rel": 3e-4, "max": 8e-3, "differ": 2e-3} if c["fp8"] else {"rel": 1e-4, "max": 6e-3}
    if k == "ffn":           # seen: FP16 1.1e-4, at most 1.9e-3; FP8 1.6e-3, at most 0.11
        return {"rel": 6e-3, "max": 0.4} if c["fp8"] else {"rel": 4e-4, "max": 8e-3}
    if k == "attention":     # seen: 5.4e-5, at most 3.1e-3
        return {"rel": 2e-4, "max": 1.2e-2}
    if k == "layer_norm":    # seen: 8.1e-6, at most 9.8e-4
        return {"rel": 3e-5, "max": 4e-3}
    if k == "xent":          # seen: 6.6e-6, at most 6.4e-4
        return {"rel": 3e-5, "max": 4e-3}
    return {"rel": 1e-3, "max": 2.5e-2, "differ": 0.0}       # seen: 2.5e-4, at most 6.3e-3; codes and counters are exact
