"""Cases that the performance of this framework is measured on.

A program that serves a model whose linear layers are packed by this framework
calls it with a few rows (one token of one or several sequences), with some
tens of rows (a decode batch, a mixture-of-experts layer), and with hundreds
to thousands of rows (a prompt or a chunk of one).  It uses either execution
path (activations in the model dtype, or Dynamic-A8), any payload width from
one to eight bits and any group size from 32 to 512.  The listed cases are
such calls at the layer shapes of the benchmark and at generic ones; ``draw``
spreads over the same ranges.

Weights are quantized groups of Laplace-distributed values: every group has a
monotone cubic of its own, its scale follows the group's largest magnitude and
the codes are the nearest points of the curve.  Activations are normal with a
factor per token and a few large entries.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2608_06763_amd as cq

DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}

# The four linear layers of a decoder block of the benchmark's decode step.
BLOCK_LAYERS = ((4096, 6144), (4096, 4096), (4096, 28672), (14336, 4096))


def listed():
    def linear(name, op, bits, group, k, n, m, dtype="bf16"):
        return {"name": name, "op": op, "bits": bits, "group": group, "k": k, "n": n, "m": m, "dtype": dtype}

    return [
        # one token through one attention output projection: the smallest
        # call, where launches and latency count
        linear("decode_o_w4", "linear", 4, 128, 4096, 4096, 1),
        # one token through all the linear layers of a decoder block
        {"name": "decode_block_w4", "op": "block", "bits": 4, "group": 128, "m": 1, "dtype": "bf16"},
        # one token, Dynamic-A8 straight from FP16 activations, narrower payload
        linear("decode_a8_w3", "linear_a8_fused", 3, 64, 14336, 4096, 1, "fp16"),
        # eight sequences decoded together, eight-bit payload
        linear("batch_w8", "linear", 8, 128, 8192, 8192, 8),
        # an odd batch of sequences through an output head with an odd number of rows
        linear("batch_head_w4", "linear", 4, 128, 4096, 32003, 13),
        # 32 sequences decoded together over Dynamic-A8
        linear("batch_a8_w4", "linear_a8", 4, 128, 14336, 4096, 32),
        # 64 sequences over Dynamic-A8, five-bit payload, large groups
        linear("batch_a8_w5", "linear_a8", 5, 512, 3072, 3584, 64),
        # a chunk of a prompt of odd length, FP16, three-bit payload
        linear("chunk_w3_fp16", "linear", 3, 64, 5120, 13824, 300, "fp16"),
        # a chunk of a prompt, six-bit payload
        linear("chunk_w6", "linear", 6, 128, 4096, 14336, 512),
        # a prompt in the model dtype
        linear("prefill_w4", "linear", 4, 128, 8192, 10240, 2048),
        # several prompts over Dynamic-A8: the largest call
        linear("prefill_a8_w4", "linear_a8", 4, 128, 8192, 28672, 8192),
        # a decode batch through a mixture-of-experts layer, two experts a token
        {"name": "routed_w4", "op": "routed", "bits": 4, "group": 128, "k": 4096, "n": 28672, "m": 16, "experts": 8,
         "topk": 2, "dtype": "bf16"},
    ]


def _log_uniform(rng: random.Random, lo: float, hi: float) -> float:
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng: random.Random):
    """One more call of the ranges above: any width and group, K from 1024 to
    16384, N from 512 to 32768 (any integer), 1 to 8192 rows."""
    op = rng.choices(["linear", "linear_a8", "linear_a8_fused", "linear_a8_carriers", "routed"], [6, 4, 1, 1, 2])[0]
    bits = rng.choices([1, 2, 3, 4, 5, 6, 7, 8], [1, 2, 3, 5, 2, 2, 1, 3])[0]
    group = rng.choices([32, 64, 128, 256, 512], [1, 2, 4, 1, 1])[0]
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    step = max(group, 128 // math.gcd(bits, 128))
    k = max(1, round(_log_uniform(rng, 1024, 16384) / step)) * step
    n = int(_log_uniform(rng, 512, 32768))
    case = {"op": op, "bits": bits, "group": group, "k": k, "n": n, "dtype": dtype}
    if op == "routed":
        # the routed product takes payloads of up to five bits
        case["bits"] = min(bits, 5)
        case["experts"] = rng.choice([4, 8, 16])
        case["topk"] = rng.choice([1, 2, 3])
        case["n"] = int(_log_uniform(rng, 512, 8192))
        case["m"] = int(_log_uniform(rng, 1, 256.99))
        return case
    most = min(8192.0, 1.2e11 / (k * n))
    case["m"] = max(1, int(_log_uniform(rng, 1, most + 0.99)))
    return case


# ---------------------------------------------------------------- inputs


def _generator(seed: int):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _quantized(g, n: int, k: int, bits: int, group: int):
    """Codes int8 [n, k], scales FP32 and shapes (a, b) FP16 [n, k / group]."""
    ng = k // group
    mag = 1 if bits == 1 else (1 << (bits - 1)) - 1
    codes = torch.empty((n, ng, group), dtype=torch.int8, device="cuda")
    scale = torch.empty((n, ng), dtype=torch.float32, device="cuda")
    # monotone cubics a t + b t^2 + (1 - a - b) t^3, steep and flat at the origin
    a = (0.5 + 0.5 * torch.rand((n, ng), generator=g, device="cuda")).half()
    b = (-0.4 * torch.rand((n, ng), generator=g, device="cuda")).half()
    rows = max(1, (1 << 25) // k)
    for lo in range(0, n, rows):
        hi = min(n, lo + rows)
        u = torch.rand((hi - lo, ng, group), generator=g, device="cuda") - 0.5
        w = torch.log1p(-2.0 * u.abs().clamp_max(0.499999)).neg_()  # Laplace magnitudes
        s = 0.9 * w.amax(-1)
        scale[lo:hi] = s * 0.014
        if bits == 1:
            codes[lo:hi] = torch.where(u < 0, -1, 1).to(torch.int8)
            continue
        t = (w / s[..., None]).clamp_(max=1.0)
        af, bf = a[lo:hi, :, None].float(), b[lo:hi, :, None].float()
        cf = 1.0 - af - bf
        x = t.clone()
        for _ in range(8):  # invert the curve (fixed point of its Newton step, kept in [0, 1])
            q = x * (af + x * (bf + x * cf))
            dq = af + x * (2.0 * bf + 3.0 * cf * x)
            x = (x - (q - t) / dq.clamp_min(0.1)).clamp_(0.0, 1.0)
        c = torch.round(x * mag)
        codes[lo:hi] = torch.where(u < 0, -c, c).to(torch.int8)
    return codes.view(n, k), scale, a, b


def _pack(codes, bits: int):
    """The continuous little-endian bitstream of every row, uint8 [n, k bits / 8]."""
    n, k = codes.shape
    out = torch.empty((n, k // 32 * bits), dtype=torch.int32, device=codes.device)
    rows = max(1, (1 << 25) // k)
    for lo in range(0, n, rows):
        hi = min(n, lo + rows)
        f = codes[lo:hi].long()
        f = (f > 0).long() if bits == 1 else f & ((1 << bits) - 1)
        f = f.view(hi - lo, k // 32, 32)
        words = torch.zeros((hi - lo, k // 32, bits + 1), dtype=torch.int64, device=codes.device)
        for j in range(32):
            wd, sh = divmod(j * bits, 32)
            words[:, :, wd] |= (f[:, :, j] << sh) & 0xFFFFFFFF
            if sh + bits > 32:
                words[:, :, wd + 1] |= f[:, :, j] >> (32 - sh)
        w = words[:, :, :bits]
        out[lo:hi] = torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32).reshape(hi - lo, -1)
    return out.view(torch.uint8)


def _activations(g, m: int, k: int, dtype: str):
    x = torch.randn((m, k), generator=g, device="cuda")
    x *= 0.5 + 3.5 * torch.rand((m, 1), generator=g, device="cuda")
    x = torch.where(torch.rand((m, k), generator=g, device="cuda") < 0.005, 20.0 * x, x)
    return x.to(DTYPES[dtype])


def _routes(g, tokens: int, experts: int, topk: int):
    """Every token takes its topk experts, drawn uniformly, token-major."""
    picks = torch.rand((tokens, experts), generator=g, device="cuda").topk(topk, dim=1).indices
    token = torch.arange(tokens, device="cuda").repeat_interleave(topk)
    return token.to(torch.int32), picks.reshape(-1).to(torch.int32)


def _layers(case):
    return BLOCK_LAYERS if case["op"] == "block" else ((case["k"], case["n"]),)


def _seeded(seed: int, layer: int) -> int:
    return 16 * seed + layer


def _weight(case, k: int, n: int, g):
    codes, scale, a, b = _quantized(g, n * case.get("experts", 1), k, case["bits"], case["group"])
    return codes, scale, a, b


def prepare(case, seed):
    state = {"op": case["op"], "weights": [], "x": []}
    for i, (k, n) in enumerate(_layers(case)):
        g = _generator(_seeded(seed, i))
        codes, scale, a, b = _weight(case, k, n, g)
        w = cq.CQWeight(_pack(codes, case["bits"]), scale, a.view(torch.int16), b.view(torch.int16), case["bits"],
                        case["group"], codes.shape[0], k)
        del codes
        state["weights"].append(w)
        state["x"].append(_activations(g, case["m"], k, case["dtype"]))
        if case["op"] == "routed":
            state["experts"] = case["experts"]
            state["token"], state["expert"] = _routes(g, case["m"], case["experts"], case["topk"])
    if case["op"] == "linear_a8_carriers":
        state["carriers"] = cq.cq_build_carriers(state["weights"][0])
    return state


def run(state):
    op, w, x = state["op"], state["weights"][0], state["x"][0]
    if op == "linear":
        return cq.cq_gemm_model_dtype(w, x)
    if op == "block":
        return [cq.cq_gemm_model_dtype(wi, xi) for wi, xi in zip(state["weights"], state["x"])]
    if op == "linear_a8":
        x8, dx = cq.cq_quantize_act_a8(x)
        return [cq.cq_gemm_a8(w, x8, dx, y_dtype=x.dtype), x8, dx]
    if op == "linear_a8_fused":
        return list(cq.cq_gemm_a8_fused(w, x))
    if op == "linear_a8_carriers":
        x8, dx = cq.cq_quantize_act_a8(x)
        return [cq.cq_gemm_a8_carriers(w, state["carriers"], x8, dx, y_dtype=x.dtype), x8, dx]
    return cq.cq_gemm_routed_model_dtype(w, state["experts"], x, state["token"], state["expert"])


def work(case):
    """Packed codes and the metadata that the width needs (W1 and W2 have no
    shapes) read once, activations read once, outputs written once."""
    nbytes = flops = 0.0
    meta = 4 if case["bits"] <= 2 else 8
    for k, n in _layers(case):
        weight = n * k * (case["bits"] / 8 + meta / case["group"])
        rows = case["m"]
        if case["op"] == "routed":
            # experts that at least one token takes (expected number)
            e = case["experts"]
            weight *= e * (1.0 - (1.0 - case["topk"] / e) ** case["m"])
            rows = case["m"] * case["topk"]
        nbytes += weight + 2 * case["m"] * k + 2 * rows * n
        if case["op"].startswith("linear_a8"):
            nbytes += case["m"] * (k + 4)  # the quantized activations are outputs too
        flops += 2.0 * rows * n * k
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # one rounding to the output dtype, plus, in FP16, weights rounded to FP16
    # operands in the many-row GEMM
    if case["dtype"] == "fp16":
        return {"rel": 1e-3, "max": 4e-3}
    return {"rel": 6e-3, "max": 2e-2}


# ---------------------------------------------------------------- the same in 64 bits


def _levels(codes, scale, a, b, group: int, bits: int):
    """s sign(k) q(|k| / M) in FP64 for rows of codes."""
    mag = 1 if bits == 1 else (1 << (bits - 1)) - 1
    n, k = codes.shape
    c = codes.view(n, k // group, group)
    t = c.abs().double() / mag
    af, bf = a.double()[..., None], b.double()[..., None]
    q = t * (af + t * (bf + t * (1.0 - af - bf))) if bits > 1 else t
    return (torch.sign(c.double()) * q * scale.double()[..., None]).view(n, k)


def _carriers(codes, scale, a, b, group: int, bits: int):
    """s / 127 times the INT8 carrier RNE(127 q(|k| / M)), rounded in integers."""
    mag = 1 if bits == 1 else (1 << (bits - 1)) - 1
    n, k = codes.shape
    c = codes.view(n, k // group, group)
    i = c.abs().long()
    ai, bi = ((v.double() * 2.0**24).long()[..., None] for v in (a, b))
    ci = (1 << 24) - ai - bi
    num = 127 * i * (ai * mag * mag + i * (bi * mag + i * ci))
    den = mag**3 << 24
    r = torch.div(num, den, rounding_mode="floor")
    twice = 2 * (num - r * den)
    r = torch.where((twice > den) | ((twice == den) & (r % 2 == 1)), r + 1, r)
    if bits == 1:
        r = torch.full_like(r, 127)
    return (torch.sign(c.double()) * r.double() * (scale.double()[..., None] / 127.0)).view(n, k)


def _product(x, weight, bits: int, group: int, levels):
    codes, scale, a, b = weight
    n, k = codes.shape
    y = torch.empty((x.shape[0], n), dtype=torch.float64, device=x.device)
    rows = max(1, (1 << 25) // k)
    for lo in range(0, n, rows):
        hi = min(n, lo + rows)
        y[:, lo:hi] = x @ levels(codes[lo:hi], scale[lo:hi], a[lo:hi], b[lo:hi], group, bits).t()
    return y


def exact(case, seed):
    bits, group, outs = case["bits"], case["group"], []
    for i, (k, n) in enumerate(_layers(case)):
        g = _generator(_seeded(seed, i))
        weight = _weight(case, k, n, g)
        x = _activations(g, case["m"], k, case["dtype"])
        if case["op"] == "routed":
            token, expert = _routes(g, case["m"], case["experts"], case["topk"])
            y = torch.empty((token.numel(), n), dtype=torch.float64, device=x.device)
            for e in range(case["experts"]):
                sel = torch.nonzero(expert == e).flatten()
                if sel.numel():
                    part = [v[e * n:(e + 1) * n] for v in weight]
                    y[sel] = _product(x.double()[token[sel].long()], part, bits, group, _levels)
            return y
        if case["op"] in ("linear", "block"):
            outs.append(_product(x.double(), weight, bits, group, _levels))
            continue
        # d = fl32(max|x| / 127) and fl32(x / d): both quotients rounded once
        # from FP64 equal the FP32 divisions
        d = (x.double().abs().amax(1).clamp_min(float(torch.tensor(1e-10))) / 127.0).float()
        v = (x.double() / d.double()[:, None]).float().double()
        x8 = (torch.sign(v) * torch.floor(v.abs() + 0.5)).clamp(-127, 127)
        y = _product(x8, weight, bits, group, _carriers) * d.double()[:, None]
        return [y, x8, d.double()]
    return outs if case["op"] == "block" else outs[0]
