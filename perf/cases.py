"""The cases this framework's speed is measured on.

They are the calls a serving program makes with quantized linear layers of a
7B-class decoder (hidden 4096, MLP 11008) and the small and ragged sizes around
them, through the package's public entry points: the GEMM from unpacked
activations for any number of tokens (codes or fp16), the decode GEMM, the GEMM
on packed operands, the zero-point GEMM and the fp16 quantizer + packer.
Weights are packed once, before the call, as a program does when it loads a
model; everything the activations need happens inside the call.
"""
import math

import torch

import paper_2508_19087_amd as apt

#: (weight bits, activation bits) in use: the paper's widths and their neighbours.
BITS = [(1, 1), (1, 2), (1, 4), (2, 2), (2, 4), (2, 8), (3, 3), (3, 4), (3, 8), (4, 4), (4, 8),
        (5, 5), (6, 6), (8, 8)]
#: 2 M N K of the largest listed case: no drawn case does more.
MOST = 2 * 2048 * 11008 * 4096


def listed():
    return [
        # the paper's smallest kernel size: one launch, where latency is everything
        {"name": "tile_w1a2_16x512x512", "kind": "packed", "M": 16, "N": 512, "K": 512, "p": 1, "q": 2,
         "out": "int32"},
        # one token through one gate projection, called eagerly from the codes
        {"name": "token_w2a2_1x11008x4096", "kind": "decode", "M": 1, "N": 11008, "K": 4096, "p": 2,
         "q": 2, "src": "codes", "out": "both"},
        # one token through the linears of eight decoder layers (q/k/v fused, o, gate/up fused,
        # down), each from its fp16 input: a decode step, captured once and replayed per token.
        # The weights (405 MB) do not fit the caches, as a model's do not.
        {"name": "decode_layers_w2a4_m1", "kind": "layers", "M": 1, "hidden": 4096, "mlp": 11008,
         "layers": 8, "p": 2, "q": 4},
        # the same for eight sequences at once and 4-bit weights, four layers (405 MB)
        {"name": "decode_layers_w4a4_m8", "kind": "layers", "M": 8, "hidden": 4096, "mlp": 11008,
         "layers": 4, "p": 4, "q": 4},
        # a batch of 64 sequences in decode, or a short prompt
        {"name": "batch_w4a4_64x11008x4096", "kind": "act", "M": 64, "N": 11008, "K": 4096, "p": 4,
         "q": 4, "src": "fp16", "out": "fp16"},
        # sizes that divide by nothing: unaligned rows, partial tiles, a partial last chunk
        {"name": "ragged_w3a8_333x5003x2999", "kind": "act", "M": 333, "N": 5003, "K": 2999, "p": 3,
         "q": 8, "src": "codes", "out": "both"},
        # a down projection of a 512-token prompt at mixed widths, on packed operands
        {"name": "down_w4a8_512x4096x11008", "kind": "packed", "M": 512, "N": 4096, "K": 11008, "p": 4,
         "q": 8, "out": "int32"},
        # the narrow widths in prefill: gate projection of 1024 tokens from fp16
        {"name": "gate_w2a2_1024x11008x4096", "kind": "act", "M": 1024, "N": 11008, "K": 4096, "p": 2,
         "q": 2, "src": "fp16", "out": "fp16"},
        # quantizers with zero-points, W2A4 as in the layer set
        {"name": "gate_affine_w2a4_1024x11008x4096", "kind": "affine", "M": 1024, "N": 11008, "K": 4096,
         "p": 2, "q": 4},
        # the widest operands: fused q/k/v projection of 1024 tokens from fp16
        {"name": "qkv_w8a8_1024x12288x4096", "kind": "act", "M": 1024, "N": 12288, "K": 4096, "p": 8,
         "q": 8, "src": "fp16", "out": "fp16"},
        # the headline prefill: 2048 tokens, W4A4, from the codes to int32
        {"name": "prefill_w4a4_2048x11008x4096", "kind": "act", "M": 2048, "N": 11008, "K": 4096, "p": 4,
         "q": 4, "src": "codes", "out": "int32"},
        # the activation side alone: quantize and pack 2048 fp16 tokens of the MLP width
        {"name": "quantize_q4_2048x11008", "kind": "quantize", "M": 2048, "K": 11008, "q": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A width: half of them multiples of 128 as models have, half as they come."""
    v = _log(rng, lo, hi)
    return max(lo, v // 128 * 128) if v >= 256 and rng.random() < 0.5 else v


def draw(rng):
    kind = rng.choice(["packed", "decode", "layers", "act", "act", "act", "affine", "quantize"])
    p, q = rng.choice(BITS)
    if kind == "quantize":
        return {"kind": kind, "M": _log(rng, 1, 4096), "K": _size(rng, 256, 11008), "q": q}
    if kind == "layers":
        hidden = 128 * rng.randint(8, 32)
        p, q = rng.choice([b for b in BITS if b[0] <= 4 and b[1] <= 4])
        return {"kind": kind, "M": rng.randint(1, 8), "hidden": hidden,
                "mlp": 32 * rng.randint(hidden // 16, hidden // 12), "layers": rng.randint(1, 4),
                "p": p, "q": q}
    M = rng.randint(1, 8) if kind == "decode" else _log(rng, 9, 2048)
    N, K = _size(rng, 256, 12288), _size(rng, 256, 11008)
    M = max(1, min(M, MOST // (2 * N * K)))
    case = {"kind": kind, "M": M, "N": N, "K": K, "p": p, "q": q}
    if kind in ("decode", "act"):
        case["src"] = rng.choice(["codes", "fp16"])
    if kind != "affine":
        case["out"] = rng.choice(["int32", "fp16", "both"])
    return case


# ---- inputs ---------------------------------------------------------------------

def _generator(seed, *sub):
    g = torch.Generator(device="cuda")
    for s in sub:
        seed = (seed * 1000003 + s + 17) % (1 << 62)
    g.manual_seed(seed)
    return g


def _codes(g, rows, K, bits):
    """Signed codes, uniform over the 2^bits values."""
    half = 1 << (bits - 1)
    return torch.randint(-half, half, (rows, K), dtype=torch.int8, device="cuda", generator=g)


def _activations(g, rows, K):
    """fp16 activations of a decoder layer's linear: a Gaussian body with a per-token spread
    (log-normal) and 1% outlier channels, 10 to 50 times larger."""
    x = torch.randn((rows, K), device="cuda", generator=g)
    x *= torch.exp(0.75 * torch.randn((rows, 1), device="cuda", generator=g))
    boost = 10.0 + 40.0 * torch.rand(K, device="cuda", generator=g)
    pick = torch.rand(K, device="cuda", generator=g) < 0.01
    return (x * torch.where(pick, boost, torch.ones_like(boost))).half()


def _scales(g, n, lo, hi):
    return (lo + (hi - lo) * torch.rand(n, device="cuda", generator=g)).half()


def _zeros(g, scale, bits):
    half = scale.float() * ((1 << bits) - 1)
    return ((torch.rand(scale.shape, device="cuda", generator=g) - 0.5) * 0.5 * half).half()


def _linears(case):
    """(N, K) of one decoder layer's linears."""
    h, m = case["hidden"], case["mlp"]
    return [(3 * h, h), (h, h), (2 * m, h), (h, m)]


def _gemm_inputs(case, seed):
    """Every tensor of a single-GEMM case, before packing."""
    M, N, K, p, q = (case[k] for k in "MNKpq")
    v = {"w": _codes(_generator(seed, 1), N, K, p),
         "ws": _scales(_generator(seed, 2), N, 0.005, 0.05)}
    if case.get("src") == "fp16":
        v["x"] = _activations(_generator(seed, 3), M, K)
    else:
        v["x"] = _codes(_generator(seed, 3), M, K, q)
        v["as"] = _scales(_generator(seed, 4), M, 0.01, 0.1)
    if case["kind"] == "affine":
        v["wz"] = _zeros(_generator(seed, 5), v["ws"], p)
        v["az"] = _zeros(_generator(seed, 6), v["as"], q)
    return v


def _layer_inputs(case, seed, i, j):
    """Weight codes, weight scales and fp16 input of linear j of layer i."""
    N, K = _linears(case)[j]
    return (_codes(_generator(seed, 10, i, j), N, K, case["p"]),
            _scales(_generator(seed, 11, i, j), N, 0.005, 0.05),
            _activations(_generator(seed, 12, i, j), case["M"], K))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "quantize":
        return {"case": case, "x": _activations(_generator(seed, 3), case["M"], case["K"])}
    if kind == "layers":
        linears = []
        for i in range(case["layers"]):
            for j in range(4):
                w, ws, x = _layer_inputs(case, seed, i, j)
                linears.append((x, apt.pack(w, case["p"]), ws))
        state = {"case": case, "linears": linears}
        # a serving program captures its decode step once and replays it per token
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _decode_step(state)
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            state["out"] = _decode_step(state)
        return state
    v = _gemm_inputs(case, seed)
    state = {"case": case, "w": apt.pack(v["w"], case["p"]), "ws": v["ws"]}
    if kind in ("packed", "affine"):
        state["a"] = apt.pack(v["x"], case["q"], activations=True)
    else:
        state["x"] = v["x"]
    for k in ("as", "wz", "az"):
        if k in v:
            state[k] = v[k]
    return state


def _decode_step(state):
    q = state["case"]["q"]
    return [apt.gemm_decode(x, q, w, out_int32=False, w_scale=ws, out_fp16=True)[1]
            for x, w, ws in state["linears"]]


# ---- one pass -------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "layers":
        state["graph"].replay()
        return state["out"]
    if kind == "quantize":
        packed, scale = apt.quantize_pack(state["x"], case["q"])
        return packed.data, packed.rowsum, scale
    if kind == "affine":
        return apt.gemm_affine(state["a"], state["w"], state["as"], state["az"], state["ws"],
                               state["wz"])[0]
    i32, f16 = case["out"] != "fp16", case["out"] != "int32"
    scales = {"a_scale": state.get("as"), "w_scale": state["ws"]} if f16 else {}
    if kind == "packed":
        out = apt.gemm(state["a"], state["w"], out_int32=i32, out_fp16=f16, **scales)
    elif kind == "decode":
        out = apt.gemm_decode(state["x"], case["q"], state["w"], out_int32=i32, out_fp16=f16, **scales)
    else:
        out = apt.gemm_act(state["x"], case["q"], state["w"], out_int32=i32, out_fp16=f16, **scales)
    return [t for t in out if t is not None]


# ---- what a pass cannot do without ------------------------------------------------

def _gemm_work(M, N, K, p, x_bytes, out_bytes):
    return {"bytes": x_bytes + N * K * p / 8 + out_bytes, "flops": 2.0 * M * N * K}


def work(case):
    kind, M = case["kind"], case["M"]
    if kind == "quantize":
        return {"bytes": M * case["K"] * (2 + case["q"] / 8) + 6 * M, "flops": 0}
    if kind == "layers":
        parts = [_gemm_work(M, N, K, case["p"], 2 * M * K, 2 * M * N) for N, K in _linears(case)]
        return {k: case["layers"] * sum(w[k] for w in parts) for k in ("bytes", "flops")}
    N, K = case["N"], case["K"]
    if kind in ("packed", "affine"):
        x = M * K * case["q"] / 8
    else:
        x = M * K * (2 if case["src"] == "fp16" else 1)
    out = {"int32": 4, "fp16": 2, "both": 6}[case.get("out", "fp16")] * M * N
    return _gemm_work(M, N, K, case["p"], x, out)


def tolerance(case):
    """The integer product and the packed bits are exact.  fp16 outputs are one rounding of an
    exact integer times its scales: against 64 bits the 2-norm is off by about 2e-4 and an element
    by up to 2^-11 of itself (with zero-points, of the sum of its terms' magnitudes)."""
    fp16 = case["kind"] in ("layers", "affine", "quantize") or case.get("out", "int32") != "int32"
    return {"rel": 8e-4, "max": 2e-3} if fp16 else "exact"


# ---- the same in 64 bits ----------------------------------------------------------

def _values(codes, bits):
    """Bipolar values 2x + 1 of signed codes."""
    return 2.0 * codes.double() + 1.0


def _quantized(x, q):
    """(bipolar values, fp16 scales) of fp16 rows: s = fp16(absmax / (2^q - 1)), and the odd
    level nearest x / s, ties upward, clamped."""
    top = (1 << q) - 1
    s = (x.float().abs().amax(dim=1) / top).half()
    t = torch.where(s[:, None] > 0, x.double() / s.double()[:, None], torch.zeros((), dtype=torch.float64, device="cuda"))
    return (2.0 * torch.floor(t / 2.0) + 1.0).clamp(-top, top), s


def _planes_rowsum(v):
    return v.sum(dim=1).to(torch.int64)


def exact(case, seed):
    kind, q = case["kind"], case["q"]
    if kind == "quantize":
        v, s = _quantized(prepare(case, seed)["x"], q)
        return None, _planes_rowsum(v), s.double()
    if kind == "layers":
        outs = []
        for i in range(case["layers"]):
            for j in range(4):
                w, ws, x = _layer_inputs(case, seed, i, j)
                v, s = _quantized(x, q)
                outs.append(v @ _values(w, case["p"]).t() * s.double()[:, None] * ws.double())
        return outs
    t = _gemm_inputs(case, seed)
    vw = _values(t["w"], case["p"])
    va, sa = _quantized(t["x"], q) if case.get("src") == "fp16" else (_values(t["x"], q), t["as"])
    if kind == "affine":
        a = va * sa.double()[:, None] + t["az"].double()[:, None]
        return a @ (vw * t["ws"].double()[:, None] + t["wz"].double()[:, None]).t()
    c = va @ vw.t()
    out = []
    if case["out"] != "fp16":
        out.append(c.to(torch.int64))
    if case["out"] != "int32":
        out.append(c * sa.double()[:, None] * t["ws"].double())
    if case.get("src") == "fp16":
        out.append(sa.double())
    return out
