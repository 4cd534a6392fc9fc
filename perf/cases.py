"""The work that programs do with this library, as cases that can be timed: the expanded linear layer from one decoded
token to the largest prefill, in its three quantization settings, and the offline expansion of weight matrices.

Sizes are those of workloads.py (C2 .. C5) and of the expanded down and output projections of the paper's Tables 1-2
that bench.py times, plus token counts between them.  Activations have the structure of language-model activations that
workloads.py uses (Gaussian or Student-t rows with a few outlier channels); int4 weight codes are distributed as
round-to-nearest leaves Gaussian weights.
"""
from __future__ import annotations

import torch

import paper_2503_17513_amd as pme

# (d, d_e): every expansion of the workloads and of the paper's tables
PAIRS = ((2048, 2176), (8192, 8448), (8192, 8704), (8192, 8960), (8192, 9728), (8192, 10240), (8192, 12288),
         (14336, 15360), (14336, 18432), (14336, 19968), (14336, 22016))
# fp32 inputs: up to 18432 (the two largest expansions take them on the plain-ALU kernel, milliseconds a call)
FP32_PAIRS = PAIRS[:9]
MOST = 4096 * 15360 * 4096          # multiply-adds of the largest listed layer
MOST_WEIGHTS = 4096 * 15360         # outputs of the listed weight expansion


def _layer(name, fmt, T, d, d_e, N, x="bf16", tail="normal"):
    case = {"do": "layer", "format": fmt, "T": T, "d": d, "d_e": d_e, "N": N, "x": x, "tail": tail}
    return dict(case, name=name) if name else case


def _weights(name, fmt, N, d, d_e, x):
    case = {"do": "weights", "format": fmt, "N": N, "d": d, "d_e": d_e, "x": x}
    return dict(case, name=name) if name else case


def listed():
    return [
        # one user's next token through a 1B-shaped down projection: the smallest call, latency and launches
        _layer("decode 1 int4", "sym", 1, 8192, 8448, 2048),
        # the decode workload: eight sequences at once, bound by reading the weights
        _layer("decode 8 int4", "sym", 8, 8192, 8448, 2048),
        # the paper's own activation quantizer, a fuller decode batch, the 8B-shaped down projection
        _layer("decode 32 asymmetric", "asym", 32, 14336, 15360, 4096, tail="student"),
        # the same stage of a server that keeps MXFP4 weights
        _layer("decode 16 mxfp4", "mxfp4", 16, 8192, 8704, 2048),
        # one chunk of a chunked prefill: a ragged number of tokens, too few for the large tiles
        _layer("chunk 333 asymmetric", "asym", 333, 8192, 9728, 2048, tail="student"),
        # fp32 base precision (one of the paper's settings), a short prompt
        _layer("prompt 517 fp32", "sym", 517, 8192, 8704, 2048, x="f32"),
        # the prefill workloads
        _layer("qkv 2048 int4", "sym", 2048, 2048, 2176, 3072),
        _layer("down 1B 2048 int4", "sym", 2048, 8192, 8704, 2048, tail="student"),
        _layer("down 8B 4096 int4", "sym", 4096, 14336, 15360, 4096, tail="student"),
        # the paper's quantizer at its second expansion of the 8B-shaped model, an odd number of tokens
        _layer("down 8B 1999 asymmetric", "asym", 1999, 14336, 18432, 4096, tail="student"),
        # the paper's second setting at the largest workload
        _layer("down 8B 4096 mxfp4", "mxfp4", 4096, 14336, 15360, 4096, tail="student"),
        # loading a model: a weight matrix in fp32 (after rotations have been merged into it) is expanded and quantized
        _weights("expand weights fp32", "sym", 4096, 14336, 15360, "f32"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    weights = rng.random() < 0.15
    x = "f32" if rng.random() < (0.5 if weights else 0.12) else "bf16"
    d, d_e = rng.choice(FP32_PAIRS if x == "f32" else PAIRS)
    if weights:
        N = min(_log(rng, 256, 4096), MOST_WEIGHTS // d_e)
        return _weights(None, rng.choice(("sym", "mxfp4")), N, d, d_e, x)
    # output widths in use are multiples of 64; one in six is not
    N = _log(rng, 512, 6144)
    N = max(64, N // 64 * 64) if rng.random() < 5 / 6 else N
    # as many decode batches as prefills
    T = _log(rng, 1, 64) if rng.random() < 0.4 else _log(rng, 65, 4096)
    T = max(1, min(T, 2048 if x == "f32" else 4096, MOST // (d_e * N)))
    return _layer(None, rng.choice(("sym", "asym", "mxfp4")), T, d, d_e, N, x=x, tail=rng.choice(("normal", "student")))


_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _activations(case, gen):
    T, d = case["T"], case["d"]
    x = torch.randn((T, d), device="cuda", generator=gen)
    if case["tail"] == "student":          # Student-t with three degrees of freedom, 0.5 % of the channels x 100
        chi = torch.randn((T, d), device="cuda", generator=gen).square_()
        for _ in range(2):
            chi += torch.randn((T, d), device="cuda", generator=gen).square_()
        x /= (chi / 3).sqrt_()
        share, gain = 0.005, 100.0
    else:
        share, gain = 0.01, 50.0
    outliers = torch.randperm(d, device="cuda", generator=gen)[: max(1, int(share * d))]
    x[:, outliers] *= gain
    return x.to(_DTYPE[case["x"]])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    d, d_e, N = case["d"], case["d_e"], case["N"]
    if case["do"] == "weights":
        wt = torch.randn((N, d), device="cuda", generator=gen) / d ** 0.5
        return {"case": case, "wt": wt.to(_DTYPE[case["x"]])}
    T = case["T"]
    state = {"case": case, "x": _activations(case, gen),
             "y": torch.empty((T, N), dtype=torch.bfloat16, device="cuda"),
             "workspace": torch.empty((pme.workspace_bytes(T, d, d_e, N),), dtype=torch.uint8, device="cuda")}
    if case["format"] == "mxfp4":
        wt = torch.randn((N, d), device="cuda", generator=gen) / d ** 0.5
        state["qw"], state["ew"] = pme.hadamard_expand_quant_mxfp4(wt.to(torch.bfloat16), d_e)
    else:
        codes = torch.randn((N, d_e), device="cuda", generator=gen).mul_(1.8).round_().clamp_(-8, 7)
        state["qw"] = pme.pack_int4(codes.to(torch.int8))
        state["sw"] = torch.rand((N,), device="cuda", generator=gen) * 0.009 + 0.001
        if case["format"] == "asym":
            state["wsum"] = pme.weight_rowsum(state["qw"])
    return state


def run(state):
    s, case = state, state["case"]
    if case["do"] == "weights":
        if case["format"] == "mxfp4":
            return pme.hadamard_expand_quant_mxfp4(s["wt"], case["d_e"])
        return pme.expand_quantize_weights(s["wt"], case["d_e"])
    if case["format"] == "mxfp4":
        return pme.expanded_linear_mxfp4(s["x"], case["d_e"], s["qw"], s["ew"], s["y"], s["workspace"])
    if case["format"] == "asym":
        return pme.expanded_linear_asym(s["x"], case["d_e"], s["qw"], s["sw"], s["wsum"], s["y"], s["workspace"])
    return pme.expanded_linear(s["x"], case["d_e"], s["qw"], s["sw"], s["y"], s["workspace"])


def work(case):
    """Inputs and weights read once, outputs written once; two operations for each multiply-add of the expanded product
    and one for each addition of the rotation's butterflies."""
    d, d_e, N = case["d"], case["d_e"], case["N"]
    rows = case["N"] if case["do"] == "weights" else case["T"]
    size = 4 if case["x"] == "f32" else 2
    _, k = pme.factor_order(d_e)
    codes = N * d_e // 2 + (N * d_e // 32 if case["format"] == "mxfp4" else 4 * N)       # with their scales
    if case["do"] == "weights":
        return {"bytes": rows * d * size + codes, "flops": rows * d_e * k}
    return {"bytes": rows * d * size + codes + 2 * rows * N, "flops": 2 * rows * d_e * N + rows * d_e * k}


def _sylvester(n):
    H = torch.ones((1, 1), dtype=torch.float64, device="cuda")
    while H.shape[0] < n:
        H = torch.cat((torch.cat((H, H), 1), torch.cat((H, -H), 1)), 0)
    return H


def _paley(b):
    """I + [[0, 1], [-1, Q]] with Q[i][j] the quadratic character of i - j over GF(b - 1), b - 1 prime or 7^3 (polynomials
    over GF(7) modulo t^3 + t + 1, element number c0 + 7 c1 + 49 c2)."""
    if b == 1:
        return torch.ones((1, 1), dtype=torch.float64, device="cuda")
    q = b - 1
    i = torch.arange(q)
    if q == 343:
        digits = torch.stack((i % 7, i // 7 % 7, i // 49), 1)
        a0, a1, a2 = digits.unbind(1)
        p = [a0 * a0, 2 * a0 * a1, 2 * a0 * a2 + a1 * a1, 2 * a1 * a2, a2 * a2]
        p[2], p[1] = p[2] - p[4], p[1] - p[4]                # t^4 = -t^2 - t
        p[1], p[0] = p[1] - p[3], p[0] - p[3]                # t^3 = -t - 1
        square = p[0] % 7 + 7 * (p[1] % 7) + 49 * (p[2] % 7)
        minus = (digits[:, None] - digits[None]) % 7
        minus = minus[..., 0] + 7 * minus[..., 1] + 49 * minus[..., 2]
    else:
        square, minus = i * i % q, (i[:, None] - i[None]) % q
    chi = torch.full((q,), -1.0, dtype=torch.float64)
    chi[square] = 1.0
    chi[0] = 0.0
    P = torch.ones((b, b), dtype=torch.float64)
    P[1:, 0] = -1.0
    P[1:, 1:] = chi[minus] + torch.eye(q, dtype=torch.float64)
    return P.cuda()


def _rotate(x, d_e):
    """Zero padding to d_e and the orthonormal rotation P_b (x) S_n, in 64 bits."""
    for b in (1, 12, 20, 60, 68, 72, 132, 140, 152, 312, 344):
        n = d_e // b
        if n * b == d_e and n & (n - 1) == 0:
            break
    T, d = x.shape
    padded = torch.zeros((T, d_e), dtype=torch.float64, device="cuda")
    padded[:, :d] = x
    y = (padded.view(T * b, n) @ _sylvester(n)).view(T, b, n)
    y = (y.transpose(1, 2).reshape(T * n, b) @ _paley(b)).view(T, n, b).transpose(1, 2)
    return y.reshape(T, d_e) / d_e ** 0.5


def _nibbles(q):
    """The two codes of each byte, in order."""
    return torch.stack((q & 15, q >> 4), 2).view(q.shape[0], -1)


def _bytes(codes):
    codes = codes.to(torch.int64) & 15
    return (codes[:, ::2] | codes[:, 1::2] << 4).to(torch.uint8)


def _e2m1(u):
    table = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], dtype=torch.float64, device="cuda")
    return torch.where(u < 8, table[(u & 7).long()], -table[(u & 7).long()])


def _mxfp4(x):
    """Codes 0 .. 15 and the exponents of the blocks' scales (OCP microscaling: 2^(floor(log2 max) - 2), round half to
    even, saturating)."""
    blocks = x.view(x.shape[0], -1, 32)
    top = blocks.abs().amax(2)
    e = torch.frexp(top)[1].to(torch.int64) - 3
    e = torch.where(top > 0, e, -127).clamp(-127, 127)
    v = torch.ldexp(blocks, -e[:, :, None])
    m = v.abs()
    step = torch.where(m < 2, 0.5, torch.where(m < 4, 1.0, 2.0)).double()
    m = ((m / step).round() * step).clamp(max=6.0)
    code = torch.where(m <= 2, m * 2, torch.where(m <= 4, m + 2, m / 2 + 4)).long()
    return (code + torch.where(v < 0, 8, 0)).view(x.shape), e


def exact(case, seed):
    s = prepare(case, seed)
    d_e, fmt = case["d_e"], case["format"]
    x = _rotate(s["wt"] if case["do"] == "weights" else s["x"], d_e)
    if fmt == "mxfp4":
        code, e = _mxfp4(x)
        if case["do"] == "weights":
            return _bytes(code), (e + 127).to(torch.uint8)
        scaled = torch.ldexp(_e2m1(code).view(*e.shape, 32), e[:, :, None]).view(x.shape)
        ew = s["ew"].to(torch.int64) - 127
        w = torch.ldexp(_e2m1(_nibbles(s["qw"])).view(*ew.shape, 32), ew[:, :, None]).view(s["qw"].shape[0], d_e)
        return scaled @ w.t()
    if fmt == "asym":
        lo, hi = x.amin(1).clamp(max=0.0), x.amax(1).clamp(min=0.0)
        sx = (hi - lo) / 15
        z = (-lo / sx).round().clamp(0, 15)
        code = ((x / sx[:, None]).round() + z[:, None]).clamp(0, 15) - z[:, None]
    else:
        sx = x.abs().amax(1) / 7
        code = (x / sx[:, None]).round().clamp(-8, 7)
    if case["do"] == "weights":
        return _bytes(code), sx
    w = _nibbles(s["qw"]).to(torch.int64)
    w = torch.where(w < 8, w, w - 16).double()
    return (code @ w.t()) * sx[:, None] * s["sw"].double()


def tolerance(case):
    """Another correct implementation sums the rotation in another order, which moves a code by one where its value lies
    on a rounding boundary; layer outputs are then rounded to bf16.  Four times what the library's two sets of kernels
    differ by at up to 128 tokens: outputs 2-norm 6e-4, largest 1.8e-2; weight codes 1e-6 of the bytes, scales 2e-7.
    Where few tokens share an output, one moved code shows: it shifts its token by 1 / (code rms x sqrt(d_e)), with
    codes of rms 1.7 or more."""
    if case["do"] == "weights":
        return {"rel": 1e-6, "max": 2e-6, "differ": 1e-5}
    return {"rel": 2.4e-3 + 0.6 / (case["T"] * case["d_e"]) ** 0.5, "max": 7e-2}
