"""What this library is used for, as cases that can be timed: fused blocks of convolutional networks, whole network
bodies through the graph layer, transformer feed-forward and attention subgraphs, and an encoder layer made of them.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare(case, seed)`` makes what a
program holds before the call (device tensors, workspaces, packed weights, launchers, captured graphs),
``run(state)`` is one pass through the public entry points, ``work(case)`` the bytes and operations the pass cannot
do without and ``tolerance(case)`` how far another correct implementation at the same precision may be off.
"""

import math

import torch

from paper_2212_01005_amd import binding as ago
from paper_2212_01005_amd import lowering

DEVICE = "cuda:0"

# The heaviest a drawn case may be; every bound lies below the largest listed case.
MAX_FLOPS = 2.0e11
MAX_BYTES = 1.0e9


def listed():
    return [
        # one inverted-residual block of a mobile network, batch 1, fp32 (the benchmark's first configuration):
        # a serving loop on fixed buffers, microseconds per call, launch and dependent latency count
        {"name": "block_f32_b1", "kind": "block", "N": 1, "H": 14, "W": 14, "Cin": 32, "Cexp": 192, "Cout": 32, "stride": 1,
         "ksize": 3, "residual": True, "bias": True, "dtype": "f32", "call": "prepared"},
        # the same kind of block at an early, large resolution and a throughput batch, bf16
        {"name": "block_bf16_b32", "kind": "block", "N": 32, "H": 56, "W": 56, "Cin": 24, "Cexp": 144, "Cout": 24, "stride": 1,
         "ksize": 3, "residual": True, "bias": True, "dtype": "bf16", "call": "prepared"},
        # a 5x5, stride-2 block (MNasNet-style) on an image size that divides nothing, small batch
        {"name": "block_k5_ragged", "kind": "block", "N": 8, "H": 29, "W": 27, "Cin": 40, "Cexp": 240, "Cout": 80, "stride": 2,
         "ksize": 5, "residual": False, "bias": True, "dtype": "bf16", "call": "direct"},
        # the 16 inverted-residual blocks of a MobileNetV2-style network at batch 1, partitioned and lowered by the
        # graph layer and replayed as a captured graph: latency of whole-network inference
        {"name": "body_b1", "kind": "body", "N": 1, "HW": 112, "mode": "graph"},
        # residual basic block of two 3x3 convolutions, 64 channels (the benchmark's third configuration)
        {"name": "chain_8x56", "kind": "chain", "N": 8, "H": 56, "W": 56, "residual": True, "call": "prepared"},
        # the same chain on detection-sized feature maps with ragged edges
        {"name": "chain_large_ragged", "kind": "chain", "N": 2, "H": 200, "W": 271, "residual": True, "call": "prepared"},
        # feed-forward of one 128-token sequence on weights packed once (batch-1 encoder inference)
        {"name": "ffn_128_packed", "kind": "ffn", "M": 128, "K": 768, "F": 3072, "act": "gelu_tanh", "weights": "packed",
         "call": "direct"},
        # feed-forward at 2048 tokens on row-major weights (the benchmark's fourth configuration)
        {"name": "ffn_2048", "kind": "ffn", "M": 2048, "K": 768, "F": 3072, "act": "gelu_tanh", "weights": "rows",
         "call": "prepared"},
        # attention of a base-size encoder at sequence length 384 (the benchmark's fifth configuration)
        {"name": "attn_384", "kind": "attn", "B": 8, "Hh": 12, "S": 384, "D": 64, "mask": "none", "call": "prepared"},
        # attention with a key-padding mask on sequences that fill no block
        {"name": "attn_masked_1000", "kind": "attn", "B": 4, "Hh": 12, "S": 1000, "D": 64, "mask": "batch", "call": "direct"},
        # long sequences, head dimension 128
        {"name": "attn_d128_long", "kind": "attn", "B": 2, "Hh": 32, "S": 2000, "D": 128, "mask": "none", "call": "prepared"},
        # one encoder layer of large-model width, 16 sequences of 512 tokens, called operator group by operator
        # group from Python: sibling projections, attention, output product with residual, feed-forward, add
        {"name": "layer_16x512", "kind": "layer", "B": 16, "S": 512, "Hh": 16, "D": 64, "F": 4096},
    ]


def _log_int(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread evenly over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999)))
    return max(lo, min(hi, int(v / step) * step))


def draw(rng):
    while True:
        case = _draw_one(rng)
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def _draw_one(rng):
    kind = rng.choice(["block", "block", "body", "chain", "ffn", "ffn", "attn", "attn", "layer"])
    call = rng.choice(["prepared", "direct"])
    if kind == "block":
        while True:
            cin = _log_int(rng, 16, 160, 8)
            cexp = (cin * rng.choice([3, 4, 6]) + 15) // 16 * 16
            stride = rng.choice([1, 1, 2])
            residual = stride == 1 and rng.random() < 0.6
            h = _log_int(rng, 7, 112)
            case = {"kind": "block", "N": _log_int(rng, 1, 32), "H": h, "W": h if rng.random() < 0.5 else _log_int(rng, 7, 112),
                    "Cin": cin, "Cexp": cexp, "Cout": cin if residual else _log_int(rng, 16, 320, 8), "stride": stride,
                    "ksize": rng.choice([3, 3, 5]), "residual": residual, "bias": rng.random() < 0.8,
                    "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "call": call}
            if case["N"] * case["H"] * case["W"] * cexp <= 20_000_000:
                return case
    if kind == "body":
        return {"kind": "body", "N": _log_int(rng, 1, 8), "HW": rng.randint(28, 112), "mode": rng.choice(["graph", "graph", "eager"])}
    if kind == "chain":
        while True:
            n, h, w = _log_int(rng, 1, 64), _log_int(rng, 7, 400), _log_int(rng, 7, 400)
            if n * h * w <= 150_000:
                return {"kind": "chain", "N": n, "H": h, "W": w, "residual": rng.random() < 0.7, "call": call}
    if kind == "ffn":
        k = _log_int(rng, 256, 1024, 64)
        return {"kind": "ffn", "M": _log_int(rng, 1, 16384), "K": k, "F": k * rng.choice([2, 3, 4]),
                "act": rng.choice(["gelu_tanh", "gelu_tanh", "relu"]), "weights": rng.choice(["rows", "packed"]), "call": call}
    if kind == "attn":
        return {"kind": "attn", "B": _log_int(rng, 1, 32), "Hh": rng.choice([4, 8, 12, 16, 32]), "S": _log_int(rng, 16, 4096),
                "D": rng.choice([64, 64, 128]), "mask": rng.choice(["none", "none", "batch", "head"]), "call": call}
    hh = rng.choice([4, 8, 12, 16])
    s = _log_int(rng, 16, 1024)
    return {"kind": "layer", "B": _log_int(rng, 1, max(1, 8192 // s)), "S": s, "Hh": hh, "D": 64, "F": 4 * hh * 64}


# ---- inputs ---------------------------------------------------------------------------------------------------

class _Maker:
    """Seeded device tensors: weights and activations in the storage type, biases fp32."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed))
        self.dtype = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(self, shape, std=1.0):
        return (torch.randn(shape, generator=self.gen, device=DEVICE) * std).to(self.dtype)

    def uniform(self, shape, lo, hi):
        return (torch.rand(shape, generator=self.gen, device=DEVICE) * (hi - lo) + lo).to(self.dtype)

    def bias(self, n):
        return torch.rand((n,), generator=self.gen, device=DEVICE) * 0.2 - 0.1

    def empty(self, shape):
        return torch.empty(shape, dtype=self.dtype, device=DEVICE)


def _workspace(op, dims, dt):
    n = ago.workspace_bytes(op, dims, dt)
    return torch.empty(n, dtype=torch.uint8, device=DEVICE) if n else None


def _launcher(case, entry, *args):
    """`prepared`: arguments marshalled once, as a serving loop on fixed buffers does; `direct`: the entry point itself."""
    if case["call"] == "prepared":
        return ago.prepare(entry, *args)
    return lambda: entry(*args)


def _out_hw(case):
    return (case["H"] - 1) // case["stride"] + 1, (case["W"] - 1) // case["stride"] + 1


def _prepare_block(case, seed):
    m = _Maker(seed, case["dtype"])
    N, H, W, ci, ce, co, ks, st = (case[k] for k in ("N", "H", "W", "Cin", "Cexp", "Cout", "ksize", "stride"))
    x = m.uniform((N, H, W, ci), -1.0, 1.0)
    w1, wd, w2 = m.normal((ci, ce), ci ** -0.5), m.normal((ks, ks, ce), 1.0 / ks), m.normal((ce, co), ce ** -0.5)
    b1, bd, b2 = (m.bias(n) if case["bias"] else None for n in (ce, ce, co))
    oh, ow = _out_hw(case)
    y = m.empty((N, oh, ow, co))
    ws = _workspace(ago.OP_FUSED_INVRES, [N, H, W, ci, ce, co, st, ks], ago.BF16 if case["dtype"] == "bf16" else ago.F32)
    entry = ago.ago_fused_invres if ks == 3 else ago.ago_fused_invres_k
    return {"call": _launcher(case, entry, x, w1, b1, wd, bd, w2, b2, y, st, case["residual"], ws), "out": y}


# (output channels, blocks, stride of the first) of the stages of a MobileNetV2-style body that starts at 16 channels
_BODY = ((24, 2, 2), (32, 3, 2), (64, 4, 2), (96, 3, 1), (160, 3, 2), (320, 1, 1))


def _body_blocks(case):
    hw, cin = case["HW"], 16
    for cout, reps, stride in _BODY:
        for r in range(reps):
            st = stride if r == 0 else 1
            yield hw, cin, 6 * cin, cout, st
            hw, cin = (hw - 1) // st + 1, cout


def _prepare_body(case, seed):
    m = _Maker(seed, "bf16")
    shape = (case["N"], case["HW"], case["HW"], 16)
    g = lowering.Graph([], {}, "bf16")
    cur = g.add("input", name="x", shape=shape)

    def param(name, tensor):
        g.params[name] = tensor
        return name

    for i, (_, ci, ce, co, st) in enumerate(_body_blocks(case)):
        src = cur
        cur = g.add("conv1x1", [cur], w=param("w1_%d" % i, m.normal((ci, ce), ci ** -0.5)))
        cur = g.add("bias", [cur], b=param("b1_%d" % i, m.bias(ce)))
        cur = g.add("relu6", [cur])
        cur = g.add("dwconv", [cur], w=param("wd_%d" % i, m.normal((3, 3, ce), 1.0 / 3)), stride=st)
        cur = g.add("bias", [cur], b=param("bd_%d" % i, m.bias(ce)))
        cur = g.add("relu6", [cur])
        cur = g.add("conv1x1", [cur], w=param("w2_%d" % i, m.normal((ce, co), ce ** -0.5)))
        cur = g.add("bias", [cur], b=param("b2_%d" % i, m.bias(co)))
        if st == 1 and ci == co:
            cur = g.add("add", [cur, src])
    x = m.uniform(shape, -1.0, 1.0)
    ex = lowering.Executor(g, lowering.lower(g, lowering.partition(g, ago)[0], ago), ago, torch)
    if case["mode"] == "eager":
        return {"executor": ex, "inputs": {"x": x}}
    replay, static_in, static_out = ex.capture({"x": x})
    return {"executor": ex, "x": x, "replay": replay, "in": static_in["x"], "out": static_out}


def _run_body(s):
    if "inputs" in s:
        return s["executor"].run(s["inputs"])
    s["in"].copy_(s["x"])            # this pass's image into the captured graph's input
    s["replay"]()
    return s["out"]


def _prepare_chain(case, seed):
    m = _Maker(seed, "bf16")
    N, H, W, C = case["N"], case["H"], case["W"], 64
    x = m.normal((N, H, W, C))
    std = (2.0 / (9 * C)) ** 0.5
    wa, wb, ba, bb = m.normal((3, 3, C, C), std), m.normal((3, 3, C, C), std), m.bias(C), m.bias(C)
    y = m.empty((N, H, W, C))
    ws = _workspace(ago.OP_FUSED_CONV_CHAIN, [N, H, W, C], ago.BF16)
    return {"call": _launcher(case, ago.ago_fused_conv_chain, x, wa, ba, wb, bb, y, case["residual"], ws), "out": y}


_ACTS = {"gelu_tanh": ago.ACT_GELU_TANH, "relu": ago.ACT_RELU}


def _pack(w):
    wp = torch.empty(ago.packed_weight_shape(*w.shape), dtype=w.dtype, device=DEVICE)
    ago.ago_pack_weight(w, wp)
    return wp


def _ffn_call(M, K, F, act, packed, x, w1, b1, w2, b2, y):
    """The feed-forward chain as the graph layer calls it: fused where the library says that pays, otherwise two products
    with fused epilogues; on packed weights where the caller packs and the library has a kernel for the size."""
    if ago.fused_ffn_pays(M, K, F, K):
        if packed and ago.fused_ffn_packed_supported(M, K, F, K):
            return ago.ago_fused_ffn_packed, (x, _pack(w1), b1, _pack(w2), b2, y, act,
                                              _workspace(ago.OP_FUSED_FFN_PACKED, [M, K, F, K], ago.BF16))
        return ago.ago_fused_ffn, (x, w1, b1, w2, b2, y, act, _workspace(ago.OP_FUSED_FFN, [M, K, F, K], ago.BF16))
    ws = _workspace(ago.OP_UNFUSED_FFN, [M, K, F, K], ago.BF16)
    if packed and ago.gemm_packed_supported(M, K, F) and ago.gemm_packed_supported(M, F, K):
        return ago.ago_unfused_ffn_packed, (x, _pack(w1), b1, _pack(w2), b2, y, act, ws)
    return ago.ago_unfused_ffn, (x, w1, b1, w2, b2, y, act, True, ws)


def _prepare_ffn(case, seed):
    m = _Maker(seed, "bf16")
    M, K, F = case["M"], case["K"], case["F"]
    x, w1, w2, b1, b2 = m.normal((M, K)), m.normal((K, F), 0.02), m.normal((F, K), 0.02), m.bias(F), m.bias(K)
    y = m.empty((M, K))
    entry, args = _ffn_call(M, K, F, _ACTS[case["act"]], case["weights"] == "packed", x, w1, b1, w2, b2, y)
    return {"call": _launcher(case, entry, *args), "out": y}


def _prepare_attn(case, seed):
    m = _Maker(seed, "bf16")
    B, Hh, S, D = case["B"], case["Hh"], case["S"], case["D"]
    q, k, v = m.normal((B, Hh, S, D)), m.normal((B, Hh, S, D)), m.normal((B, Hh, S, D))
    o = m.empty((B, Hh, S, D))
    scale = D ** -0.5
    if case["mask"] == "none":
        return {"call": _launcher(case, ago.ago_fused_attn, q, k, v, o, scale, None), "out": o}
    if case["mask"] == "head":          # a relative-position table shared by the batch
        bias = m.normal((1, Hh, S, S))
    else:                               # key padding: the last keys of every sequence are masked
        lens = torch.randint((S + 1) // 2, S + 1, (B, 1, 1, 1), generator=m.gen, device=DEVICE)
        keep = torch.arange(S, device=DEVICE).view(1, 1, 1, S) < lens
        bias = torch.where(keep, 0.0, -10000.0).expand(B, 1, S, S).to(torch.bfloat16).contiguous()
    return {"call": _launcher(case, ago.ago_fused_attn_bias, q, k, v, bias, o, scale, None), "out": o}


def _prepare_layer(case, seed):
    m = _Maker(seed, "bf16")
    B, S, Hh, D, F = (case[k] for k in ("B", "S", "Hh", "D", "F"))
    K, M = Hh * D, B * S
    s = {"x": m.normal((M, K))}
    for n in ("wq", "wk", "wv", "wo"):
        s[n] = m.normal((K, K), K ** -0.5)
    for n in ("bq", "bk", "bv", "bo"):
        s[n] = m.bias(K)
    s["q"], s["k"], s["v"], s["a"] = (m.empty((B, S, Hh, D)) for _ in range(4))
    s["h"], s["f"], s["y"] = (m.empty((M, K)) for _ in range(3))
    w1, w2, b1, b2 = m.normal((K, F), 0.02), m.normal((F, K), 0.02), m.bias(F), m.bias(K)
    s["ffn"] = _ffn_call(M, K, F, ago.ACT_GELU_TANH, False, s["h"], w1, b1, w2, b2, s["f"])
    s["scale"] = D ** -0.5
    return s


def _run_layer(s):
    ago.ago_fused_qkv(s["x"], s["wq"], s["wk"], s["wv"], s["bq"], s["bk"], s["bv"], s["q"], s["k"], s["v"], head_major=False)
    ago.ago_fused_attn_bshd(s["q"], s["k"], s["v"], s["a"], s["scale"])
    ago.ago_gemm(s["a"].view(s["x"].shape), s["wo"], s["bo"], s["x"], s["h"])
    entry, args = s["ffn"]
    entry(*args)
    ago.ago_add_act(s["h"], s["f"], s["y"])
    return {"h": s["h"], "y": s["y"]}


_PREPARE = {"block": _prepare_block, "body": _prepare_body, "chain": _prepare_chain, "ffn": _prepare_ffn,
            "attn": _prepare_attn, "layer": _prepare_layer}


def prepare(case, seed):
    s = _PREPARE[case["kind"]](case, seed)
    s["kind"] = case["kind"]
    return s


def run(state):
    if state["kind"] == "body":
        return _run_body(state)
    if state["kind"] == "layer":
        return _run_layer(state)
    state["call"]()
    return state["out"]


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def _block_work(N, H, W, ci, ce, co, st, ks):
    oh, ow = (H - 1) // st + 1, (W - 1) // st + 1
    flops = 2 * N * H * W * ci * ce + 2 * ks * ks * N * oh * ow * ce + 2 * N * oh * ow * ce * co
    return flops, N * H * W * ci, ci * ce + ks * ks * ce + ce * co, N * oh * ow * co


def work(case):
    kind = case["kind"]
    if kind == "block":
        flops, x, w, y = _block_work(*(case[k] for k in ("N", "H", "W", "Cin", "Cexp", "Cout", "stride", "ksize")))
        bias = 4 * (2 * case["Cexp"] + case["Cout"]) if case["bias"] else 0
        return {"bytes": (2 if case["dtype"] == "bf16" else 4) * (x + w + y) + bias, "flops": flops}
    if kind == "body":
        flops, moved, last = 0, 2 * case["N"] * case["HW"] ** 2 * 16, 0
        for hw, ci, ce, co, st in _body_blocks(case):
            f, _, w, y = _block_work(case["N"], hw, hw, ci, ce, co, st, 3)
            flops, moved, last = flops + f, moved + 2 * w + 4 * (2 * ce + co), 2 * y
        return {"bytes": moved + last, "flops": flops}
    if kind == "chain":
        p, C = case["N"] * case["H"] * case["W"], 64
        return {"bytes": 2 * (2 * p * C + 2 * 9 * C * C) + 8 * C, "flops": 4 * 9 * p * C * C}
    if kind == "ffn":
        M, K, F = case["M"], case["K"], case["F"]
        return {"bytes": 2 * (2 * M * K + 2 * K * F) + 4 * (F + K), "flops": 4 * M * K * F}
    if kind == "attn":
        B, Hh, S, D = case["B"], case["Hh"], case["S"], case["D"]
        mask = {"none": 0, "batch": B, "head": Hh}[case["mask"]] * S * S
        return {"bytes": 2 * (4 * B * Hh * S * D + mask), "flops": 4 * B * Hh * S * S * D}
    B, S, Hh, D, F = (case[k] for k in ("B", "S", "Hh", "D", "F"))
    M, K = B * S, Hh * D
    return {"bytes": 2 * (3 * M * K + 4 * K * K + 2 * K * F) + 4 * (5 * K + F),
            "flops": 2 * M * K * 4 * K + 4 * M * K * F + 4 * M * S * K}


def tolerance(case):
    if case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "body":          # sixteen blocks, each rounding its output to bf16
        return {"rel": 2e-2, "max": 0.2}
    return {"rel": 1e-2, "max": 0.1}
