"""The calls this library exists for, as measurable cases.

A case is one pass of work as a program that runs quantized layers issues it: a decode or prefill
linear layer, the products of an encoder block, convolution layers, matrices no tile divides, 16-bit
operands.  ``prepare`` makes what such a program holds before the call (device buffers, packed
weights, filter sums, workspaces), ``run`` issues the pass through the public entry points,
``exact`` forms the same outputs in 64-bit arithmetic with plain torch.

Sizes come from the workloads of this repository (decode layers of a LLaMA-7B-shaped model, linear
and attention products of BERT-shaped encoder blocks, ResNet-50-shaped convolutions, squares, odd
sizes with padded leading dimensions); ``draw`` spreads over the same ranges.
"""
import math

import torch

import paper_2506_11728_amd as M

ROW, COL = M.ROW_MAJOR, M.COL_MAJOR
OVERWRITE, ACCUMULATE = M.OVERWRITE, M.ACCUMULATE

# (h_i = w_i, c_i, c_o, h_f = w_f, stride, pad): the distinct kinds of layer of a ResNet-50-type
# network, from the 3-channel stem to the last expansions
CONV_LAYERS = (
    (224, 3, 64, 7, 2, 3),
    (56, 64, 64, 1, 1, 0), (56, 64, 64, 3, 1, 1), (56, 64, 256, 1, 1, 0), (56, 256, 64, 1, 1, 0),
    (56, 256, 128, 1, 1, 0), (56, 128, 128, 3, 2, 1), (56, 256, 512, 1, 2, 0),
    (28, 128, 128, 3, 1, 1), (28, 128, 512, 1, 1, 0), (28, 512, 128, 1, 1, 0), (28, 512, 1024, 1, 2, 0),
    (14, 256, 256, 3, 1, 1), (14, 256, 1024, 1, 1, 0), (14, 1024, 256, 1, 1, 0), (14, 1024, 2048, 1, 2, 0),
    (7, 512, 512, 3, 1, 1), (7, 512, 2048, 1, 1, 0), (7, 2048, 512, 1, 1, 0),
)

# an encoder block of a BERT-Large-type model
ENCODER_D, ENCODER_HEADS = 1024, 16


def _gemm(name, m, n, k, entry="s8s8", out="s32", orders="rrr", pad=0, panels=1):
    """entry: operand types of A and B; out: s32, f32 (dequantised) or s8 (requantised); orders: r / c
    for A, B, C; pad: added to every smallest legal leading dimension; panels: k arrives in that many
    parts, the first overwriting C and the others accumulating onto it."""
    return {"name": name, "kind": "gemm", "m": m, "n": n, "k": k, "entry": entry, "out": out,
            "orders": orders, "pad": pad, "panels": panels}


def _packed(name, m, n, k, entry):
    return {"name": name, "kind": "packed", "m": m, "n": n, "k": k, "entry": entry}


def _conv(name, b, layer, out, sums):
    hi, ci, co, hf, stride, pad = layer
    return {"name": name, "kind": "conv", "b": b, "hi": hi, "ci": ci, "co": co, "hf": hf,
            "stride": stride, "pad": pad, "out": out, "sums": sums}


def listed():
    return [
        # one token through a 4096 x 4096 layer whose weights were packed at load time
        _packed("decode_1_token_packed", 1, 4096, 4096, "s8s8"),
        # sixteen sequences decoding together, weights as they came (k x n, row-major), result
        # dequantised for the floating-point step that follows
        _gemm("decode_16_tokens_f32", 16, 11008, 4096, out="f32"),
        # sixty-four sequences, uint8 activations, packed weights with a long k
        _packed("decode_64_tokens_u8_packed", 64, 4096, 11008, "u8s8"),
        # a product small enough that launching it is most of its time, k in two panels
        _gemm("small_256_two_panels", 256, 256, 512, panels=2),
        # every GEMM of one encoder block on 512 tokens, the per-head products as batched calls
        {"name": "encoder_block_512", "kind": "encoder", "l": 512},
        # a prompt of 1000 tokens through an up-projection, weights stored n x k, uint8 activations,
        # result dequantised
        _gemm("prefill_1000_tokens_f32", 1000, 11008, 4096, entry="u8s8", out="f32", orders="rcr"),
        # a mid-size layer between two quantized layers: int8 in, int8 out
        _gemm("square_2048_s8_out", 2048, 2048, 2048, out="s8"),
        # the large product the throughput of such a library is quoted on
        _gemm("square_8192", 8192, 8192, 8192),
        # nothing is a multiple of anything and no row is aligned
        _gemm("unaligned_4095x4097x4099", 4095, 4097, 4099, pad=17),
        # a 3 x 3 layer of a convolutional network at batch 32, int8 output for the next layer
        _conv("conv_3x3_b32_s8_out", 32, (28, 128, 128, 3, 1, 1), "s8", True),
        # its 3-channel first layer at batch 32
        _conv("conv_stem_b32", 32, (224, 3, 64, 7, 2, 3), "s32", False),
        # 16-bit operands through a feed-forward layer
        {"name": "s16_1024x3072x768", "kind": "s16", "m": 1024, "n": 3072, "k": 768, "orders": "rcr"},
    ]


def _size(rng, lo, hi):
    """Log-uniform in lo .. hi; a third of them whole multiples of 64 (where large enough), a third
    multiples of 16, a third as drawn."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    unit = rng.choice((64, 16, 1))
    if x >= unit:
        x = x // unit * unit
    return max(lo, min(hi, x))


def draw(rng):
    kind = rng.choice(("packed", "gemm", "gemm", "gemm", "encoder", "conv", "conv", "s16"))
    if kind == "packed":
        case = _packed("", _size(rng, 1, 128), _size(rng, 512, 16384), _size(rng, 512, 16384),
                       rng.choice(("s8s8", "u8s8")))
    elif kind == "gemm":
        m, n, k = _size(rng, 16, 8192), _size(rng, 64, 12288), _size(rng, 64, 8192)
        while m * n * k > 8192 ** 3:
            k = max(64, k // 2)
        out = rng.choice(("s32", "s32", "f32", "s8"))
        case = _gemm("", m, n, k, entry=rng.choice(("s8s8", "u8s8", "s8u8")), out=out,
                     orders=rng.choice(("rrr", "rcr", "rrr", "rcr", "crr", "rrc")),
                     pad=rng.choice((0, 0, 0, 16, 17)),
                     panels=rng.choice((1, 1, 2)) if out == "s32" else 1)
    elif kind == "encoder":
        case = {"kind": "encoder", "l": _size(rng, 64, 1024)}
    elif kind == "conv":
        out = rng.choice(("s32", "f32", "s8"))
        case = _conv("", rng.choice((1, 2, 4, 8, 16, 32)), rng.choice(CONV_LAYERS), out,
                     rng.choice((True, False)))
    else:
        case = {"kind": "s16", "m": _size(rng, 16, 4096), "n": _size(rng, 64, 4096),
                "k": _size(rng, 64, 4096), "orders": rng.choice(("rrr", "rcr", "crr", "rrc"))}
    case.pop("name", None)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

_TORCH = {"s8": torch.int8, "u8": torch.uint8}
_OUT = {"s32": torch.int32, "f32": torch.float32, "s8": torch.int8}


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + stream)


def _values(gen, rows, cols, kind):
    """Operand values: uint8 activations uniform, int8 ones clipped normal (as layers produce them),
    "any8" and "s16" uniform over their type."""
    if kind == "u8":
        return torch.randint(0, 256, (rows, cols), generator=gen, device="cuda", dtype=torch.uint8)
    if kind == "any8":
        return torch.randint(-128, 128, (rows, cols), generator=gen, device="cuda", dtype=torch.int8)
    if kind == "s16":
        return torch.randint(-32768, 32768, (rows, cols), generator=gen, device="cuda", dtype=torch.int16)
    x = torch.randn((rows, cols), generator=gen, device="cuda") * 24.0
    return x.round_().clamp_(-128, 127).to(torch.int8)


def _ld(rows, cols, order, pad):
    return (cols if order == "r" else rows) + pad


def _store(x, order, pad):
    """The matrix x in a flat buffer with leading dimension smallest + pad."""
    y = x if order == "r" else x.t()
    if pad == 0:
        return y.contiguous()
    buf = torch.zeros((y.shape[0], y.shape[1] + pad), dtype=x.dtype, device="cuda")
    buf[:, :y.shape[1]] = y
    return buf


def _order(c):
    return ROW if c == "r" else COL


def _operand_kinds(case):
    a, b = case["entry"][:2], case["entry"][2:]
    if case["m"] == case["n"] == case["k"]:
        a, b = ("any8" if t == "s8" else t for t in (a, b))
    return a, b


def _gemm_values(case, seed):
    a, b = _operand_kinds(case)
    return (_values(_generator(seed, 1), case["m"], case["k"], a),
            _values(_generator(seed, 2), case["k"], case["n"], b))


def _scale(case):
    """A float32 value that leaves requantised results spread over the int8 range."""
    depth = case["k"] if "k" in case else case["ci"] * case["hf"] ** 2
    spread = 24.0 * 24.0 if case.get("entry") == "s8s8" else 24.0 * 147.0
    return float(torch.tensor(40.0 / (spread * math.sqrt(depth)), dtype=torch.float32))


def _panel_edges(case):
    p = case["panels"]
    return [case["k"] * i // p for i in range(p + 1)]


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def prepare(case, seed):
    return {"gemm": _prepare_gemm, "packed": _prepare_packed, "encoder": _prepare_encoder,
            "conv": _prepare_conv, "s16": _prepare_s16}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


# ---- GEMM ----

def _prepare_gemm(case, seed):
    A, B = _gemm_values(case, seed)
    oa, ob, oc = case["orders"]
    pad, m, n = case["pad"], case["m"], case["n"]
    edges = _panel_edges(case)
    size = M.mipgemm_workspace_size if case["out"] == "s32" else M.mipgemm_workspace_size_f32
    panels, ws = [], 0
    for lo, hi in zip(edges, edges[1:]):
        a, b = A[:, lo:hi], B[lo:hi, :]
        panels.append((hi - lo, _store(a, oa, pad), _ld(m, hi - lo, oa, pad),
                       _store(b, ob, pad), _ld(hi - lo, n, ob, pad)))
        ws = max(ws, size(m, n, hi - lo, _order(oa), _order(ob), _order(oc)))
    C = _store(torch.zeros((m, n), dtype=_OUT[case["out"]], device="cuda"), oc, pad)
    view = C[:, :n] if oc == "r" else C[:, :m].t()
    extra = {} if case["out"] == "s32" else {"scale": _scale(case)}
    return {"run": _run_gemm, "fn": getattr(M, "mipgemm_" + case["entry"] + case["out"]), "m": m, "n": n,
            "panels": panels, "orders": [_order(c) for c in case["orders"]], "C": C,
            "ldc": _ld(m, n, oc, pad), "view": view, "ws": _workspace(ws), "ws_bytes": ws, "extra": extra}


def _run_gemm(s):
    oa, ob, oc = s["orders"]
    mode = OVERWRITE
    for k, A, lda, B, ldb in s["panels"]:
        s["fn"](s["m"], s["n"], k, A, lda, oa, B, ldb, ob, s["C"], s["ldc"], oc, mode,
                workspace=s["ws"], workspace_bytes=s["ws_bytes"], **s["extra"])
        mode = ACCUMULATE
    return s["view"]


# ---- packed weights ----

def _prepare_packed(case, seed):
    A, B = _gemm_values(case, seed)
    m, n, k = case["m"], case["n"], case["k"]
    packed = torch.empty(M.mipgemm_packed_weights_bytes(k, n), dtype=torch.uint8, device="cuda")
    M.mipgemm_pack_weights(k, n, B.contiguous(), n, ROW, packed)
    ws = M.mipgemm_workspace_size(m, n, k, ROW, COL, ROW)
    return {"run": _run_packed, "fn": getattr(M, "mipgemm_" + case["entry"] + "s32_packed"), "m": m, "n": n,
            "k": k, "A": A.contiguous(), "packed": packed, "ws": _workspace(ws), "ws_bytes": ws,
            "C": torch.zeros((m, n), dtype=torch.int32, device="cuda")}


def _run_packed(s):
    s["fn"](s["m"], s["n"], s["k"], s["A"], s["k"], ROW, s["packed"], s["C"], s["n"], ROW, OVERWRITE,
            workspace=s["ws"], workspace_bytes=s["ws_bytes"])
    return s["C"]


# ---- encoder block ----
# M1-M3 the Q, K, V projections (one batch that shares the activations), M5 K^T Q and M7 V E_1 for
# every head (E_1, the attention weights after the softmax, unsigned), M9 the output projection,
# F11 and F13 the feed-forward pair.  The steps between the products (softmax, normalisation,
# re-quantisation) belong to the caller: every product has operands of its own.

def _encoder_values(case, seed):
    l, d, h = case["l"], ENCODER_D, ENCODER_HEADS
    v = lambda i, r, c, kind="s8": _values(_generator(seed, i), r, c, kind)
    return {"Wqkv": v(1, 3 * d, d), "X": v(2, d, l), "K": v(3, d, l), "Q": v(4, d, l), "V": v(5, d, l),
            "E": v(6, h * l, l, "u8"), "W9": v(7, d, d), "X9": v(8, d, l), "W11": v(9, 4 * d, d),
            "X11": v(10, d, l), "W13": v(11, d, 4 * d), "X13": v(12, 4 * d, l)}


def _prepare_encoder(case, seed):
    l, d, h = case["l"], ENCODER_D, ENCODER_HEADS
    s = _encoder_values(case, seed)
    out = lambda *shape: torch.zeros(shape, dtype=torch.int32, device="cuda")
    s.update(run=_run_encoder, l=l, C1=out(3, d, l), C5=out(h, l, l), C7=out(d, l), C9=out(d, l),
             C11=out(4 * d, l), C13=out(d, l))
    ws = max(M.mipgemm_workspace_size(m, l, k, ROW, ROW, ROW)
             for m, k in ((d, d), (d // h, l), (l, d // h), (4 * d, d), (d, 4 * d)))
    s.update(ws=_workspace(ws), ws_bytes=ws)
    return s


def _run_encoder(s):
    l, d, h = s["l"], ENCODER_D, ENCODER_HEADS
    dk = d // h
    w = {"workspace": s["ws"], "workspace_bytes": s["ws_bytes"]}
    M.mipgemm_s8s8s32_batched(d, l, d, s["Wqkv"], d, ROW, d * d, s["X"], l, ROW, 0,
                              s["C1"], l, ROW, d * l, 3, OVERWRITE, **w)
    # (K^i)^T is the d/h x l slice of K read column-major
    M.mipgemm_s8s8s32_batched(l, l, dk, s["K"], l, COL, dk * l, s["Q"], l, ROW, dk * l,
                              s["C5"], l, ROW, l * l, h, OVERWRITE, **w)
    M.mipgemm_s8u8s32_batched(dk, l, l, s["V"], l, ROW, dk * l, s["E"], l, ROW, l * l,
                              s["C7"], l, ROW, dk * l, h, OVERWRITE, **w)
    M.mipgemm_s8s8s32(d, l, d, s["W9"], d, ROW, s["X9"], l, ROW, s["C9"], l, ROW, OVERWRITE, **w)
    M.mipgemm_s8s8s32(4 * d, l, d, s["W11"], d, ROW, s["X11"], l, ROW, s["C11"], l, ROW, OVERWRITE, **w)
    M.mipgemm_s8s8s32(d, l, 4 * d, s["W13"], 4 * d, ROW, s["X13"], l, ROW, s["C13"], l, ROW, OVERWRITE, **w)
    return {"qkv": s["C1"], "scores": s["C5"], "attention": s["C7"], "projection": s["C9"],
            "hidden": s["C11"], "output": s["C13"]}


# ---- convolution ----

def _out_size(case):
    return (case["hi"] + 2 * case["pad"] - case["hf"]) // case["stride"] + 1


def _conv_values(case, seed):
    hi, ci, co, hf = case["hi"], case["ci"], case["co"], case["hf"]
    image = _values(_generator(seed, 1), case["b"] * hi * hi, ci, "u8").view(case["b"], hi, hi, ci)
    return image, _values(_generator(seed, 2), co, hf * hf * ci, "s8")


def _geometry(case):
    return (case["b"], case["hi"], case["hi"], case["ci"], case["co"], case["hf"], case["hf"],
            case["stride"], case["pad"])


def _prepare_conv(case, seed):
    image, filters = _conv_values(case, seed)
    ho = _out_size(case)
    geo = _geometry(case)
    ws = M.mipgemm_conv_workspace_size(*geo)
    args = {"workspace": _workspace(ws), "workspace_bytes": ws}
    sums = None
    if case["sums"]:
        sums = torch.empty(case["co"], dtype=torch.int32, device="cuda")
        M.mipgemm_conv_filter_sums(case["co"], filters.shape[1], filters, sums)
    name = "mipgemm_conv_s8u8" + case["out"]
    mode = (OVERWRITE,)
    if case["out"] == "s8":
        args["filter_sums"] = sums
    elif sums is not None:
        name += "_with_sums"
        mode = (OVERWRITE, sums)
    if case["out"] != "s32":
        args["scale"] = _scale(case)
    O = torch.zeros((case["b"], ho, ho, case["co"]), dtype=_OUT[case["out"]], device="cuda")
    return {"run": _run_conv, "fn": getattr(M, name), "geo": geo, "F": filters, "I": image, "O": O,
            "mode": mode, "args": args}


def _run_conv(s):
    s["fn"](*s["geo"], s["F"], s["I"], s["O"], *s["mode"], **s["args"])
    return s["O"]


# ---- 16-bit operands ----

def _s16_values(case, seed):
    return (_values(_generator(seed, 1), case["m"], case["k"], "s16"),
            _values(_generator(seed, 2), case["k"], case["n"], "s16"))


def _prepare_s16(case, seed):
    A, B = _s16_values(case, seed)
    m, n, k = case["m"], case["n"], case["k"]
    oa, ob, oc = case["orders"]
    C = torch.zeros((m, n) if oc == "r" else (n, m), dtype=torch.int32, device="cuda")
    ws = M.mipgemm_workspace_size_s16(m, n, k)
    return {"run": _run_s16, "m": m, "n": n, "k": k, "A": _store(A, oa, 0), "lda": _ld(m, k, oa, 0),
            "B": _store(B, ob, 0), "ldb": _ld(k, n, ob, 0), "C": C, "ldc": _ld(m, n, oc, 0),
            "orders": [_order(c) for c in case["orders"]], "view": C if oc == "r" else C.t(),
            "ws": _workspace(ws), "ws_bytes": ws}


def _run_s16(s):
    oa, ob, oc = s["orders"]
    M.mipgemm_s16s16s32(s["m"], s["n"], s["k"], s["A"], s["lda"], oa, s["B"], s["ldb"], ob, s["C"],
                        s["ldc"], oc, OVERWRITE, workspace=s["ws"], workspace_bytes=s["ws_bytes"])
    return s["view"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it has to give
# ---------------------------------------------------------------------------

_OUT_BYTES = {"s32": 4, "f32": 4, "s8": 1}


def work(case):
    """Operands once, outputs once; two operations per multiply-accumulate of the named type."""
    if case["kind"] == "encoder":
        l, d, h = case["l"], ENCODER_D, ENCODER_HEADS
        products = [(d, l, d)] * 4 + [(l, l, d // h)] * h + [(d // h, l, l)] * h + [(4 * d, l, d), (d, l, 4 * d)]
        nbytes = sum(m * k + k * n + 4 * m * n for m, n, k in products) - 2 * d * l  # X is shared by M1-M3
        return {"bytes": nbytes, "flops": sum(2 * m * n * k for m, n, k in products)}
    if case["kind"] == "conv":
        positions = case["b"] * _out_size(case) ** 2
        depth = case["ci"] * case["hf"] ** 2
        return {"bytes": case["b"] * case["hi"] ** 2 * case["ci"] + case["co"] * depth
                + _OUT_BYTES[case["out"]] * positions * case["co"],
                "flops": 2 * positions * case["co"] * depth}
    m, n, k = case["m"], case["n"], case["k"]
    element = 2 if case["kind"] == "s16" else 1
    return {"bytes": element * (m * k + k * n) + _OUT_BYTES[case.get("out", "s32")] * m * n,
            "flops": 2 * m * n * k}


def tolerance(case):
    """Integer results are exact in any order of summation.  A dequantised result is a 32-bit
    conversion and one 32-bit multiplication: 2^-24 of each, 2.5e-8 measured in the 2-norm."""
    if case.get("out") == "f32":
        return {"rel": 1e-7}
    return "exact"


def _product(A, B):
    """A B as 64-bit integers: every partial sum is below 2^53, so double arithmetic is exact."""
    return (A.to(torch.float64) @ B.to(torch.float64)).to(torch.int64)


def _finish(S, case):
    out = case.get("out", "s32")
    if out == "s32":
        return S.to(torch.int32)  # modulo 2^32
    scale = _scale(case)
    if out == "f32":
        return S.to(torch.float64) * scale
    # requantisation is defined in float32: conversion, one product, ties to even, saturation
    return (S.to(torch.float32) * torch.tensor(scale, dtype=torch.float32, device=S.device)
            ).round().clamp(-128, 127).to(torch.int8)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gemm", "packed"):
        return _finish(_product(*_gemm_values(case, seed)), case)
    if kind == "s16":
        return _finish(_product(*_s16_values(case, seed)), case)
    if kind == "conv":
        image, filters = _conv_values(case, seed)
        b, hi, ci, hf = case["b"], case["hi"], case["ci"], case["hf"]
        pad, stride, ho, co = case["pad"], case["stride"], _out_size(case), case["co"]
        padded = torch.zeros((b, hi + 2 * pad, hi + 2 * pad, ci), dtype=torch.float64, device="cuda")
        padded[:, pad:pad + hi, pad:pad + hi, :] = image.to(torch.float64)
        taps = filters.to(torch.float64).view(co, hf, hf, ci)
        S = torch.zeros((b * ho * ho, co), dtype=torch.float64, device="cuda")
        reach = stride * (ho - 1) + 1
        for y in range(hf):
            for x in range(hf):
                window = padded[:, y:y + reach:stride, x:x + reach:stride, :].reshape(-1, ci)
                S += window @ taps[:, y, x, :].t().contiguous()
        return _finish(S.to(torch.int64).view(b, ho, ho, co), case)
    l, d, h = case["l"], ENCODER_D, ENCODER_HEADS
    v = _encoder_values(case, seed)
    heads = lambda X: X.view(h, d // h, l)
    K, Q, V, E = heads(v["K"]), heads(v["Q"]), heads(v["V"]), v["E"].view(h, l, l)
    res = {"qkv": _product(v["Wqkv"], v["X"]).view(3, d, l),
           "scores": torch.stack([_product(K[i].t().contiguous(), Q[i]) for i in range(h)]),
           "attention": torch.cat([_product(V[i], E[i]) for i in range(h)]),
           "projection": _product(v["W9"], v["X9"]), "hidden": _product(v["W11"], v["X11"]),
           "output": _product(v["W13"], v["X13"])}
    return {key: S.to(torch.int32) for key, S in res.items()}
