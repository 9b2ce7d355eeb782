"""The work this library does for its users, as cases that can be timed and checked one by one.

A case is a dict of plain values:
  entry   what is called: "inv" (chunk matrices built from keys and inverted), "inv_varlen" (the same on packed sequences),
          "tri" (given matrices inverted), "solve" / "solve2" (the inverse applied to one / two right-hand sides),
          "solve_varlen" (applied, packed sequences)
  B, T    sequences and tokens per sequence; packed sequences: their number and mean length (the lengths are drawn from `lens`)
  H, dk, dx, C          heads, key channels, right-hand-side columns, chunk size
  k, op, out            element types of the keys (entry "tri": of the given matrices), of the matrix-core operands and of the result
  gate    "scalar" (one decay per token and head), "channel" (one per key channel), "none"
  keys    "gaussian" (unit-norm Gaussian keys) or "rank4" (correlated keys: a rank-4 component shared by the sequence)
  method  inversion method
"""
import math
import random

import torch

import paper_2605_21325_amd as tri

_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_CODE = {"f32": tri.F32, "f16": tri.F16, "bf16": tri.BF16}
_GATE = {"scalar": tri.GATE_SCALAR, "channel": tri.GATE_PER_CHANNEL, "none": tri.GATE_NONE}
_METHOD = {"block": tri.BLOCK_RECURSIVE, "mixed": tri.MIXED, "direct": tri.BLOCK_DIRECT, "newton": tri.NEWTON_SCHULZ, "forward": tri.FWD_SUBST}
_DECAY = 0.05  # scale of a token's log-decay, softplus(N(0, 1)) times this


def _case(name, **kw):
    c = dict(entry="inv", B=1, T=4096, H=16, dk=128, dx=0, C=64, k="bf16", op="bf16", out="f32", gate="scalar", keys="gaussian",
             method="block", lens=0)
    c.update(kw)
    return dict(c, name=name)


def listed():
    return [
        # One short prompt in full fp32 (8 matrices): the smallest call, launch and argument handling.
        _case("tiny_fp32", T=256, H=2, dk=64, k="f32", op="f32"),
        # One layer's prefill of one 4096-token prompt, the plain entry point with its defaults.
        _case("prefill_1x4096"),
        # The same layer on a batch of long prompts: the throughput case.
        _case("batch_8x8192", B=8, T=8192),
        # Matrices another kernel has formed (fp32, single-layer size, an odd number of them), the standalone entry point.
        _case("given_fp32", entry="tri", B=1, T=4099 * 64, H=1, k="f32", op="f32"),
        # The same with everything kept in bf16 at the larger chunk size.
        _case("given_bf16_c128", entry="tri", B=1, T=8192 * 128, H=1, C=128, k="bf16", out="bf16"),
        # Per-channel decay over a batch of long prompts: the largest tensors.
        _case("kda_4x16384", B=4, T=16384, H=32, gate="channel"),
        # Large chunks, no decay, correlated keys: the numerically hard input, by the mixed recursion.
        _case("stress_c128", T=32768, H=32, C=128, gate="none", keys="rank4", method="mixed"),
        # What a layer does with the inverse: its key-side and value-side products in one call; prompts that end inside a chunk.
        _case("layer_pair_4x4000", entry="solve2", B=4, T=4000, dx=128),
        # Continuous batching on one shard of a tensor-parallel layer (4 heads): packed prompts of different lengths.
        _case("packed_4heads", entry="solve_varlen", B=48, T=1100, H=4, dx=128, lens=1),
        # The per-channel layer with large chunks, inverse applied.
        _case("kda_solve_c128", entry="solve", B=2, T=8192, C=128, gate="channel", dx=128),
        # Direct fp32 substitution with large chunks: the reference-accuracy setting.
        _case("forward_c128", T=8192, H=32, C=128, method="forward", op="f32"),
        # Newton-Schulz with fp32 operands, twelve iterations.
        _case("newton_fp32", B=4, T=8192, method="newton", op="f32"),
    ]


def draw(rng):
    """One more call of the same kinds: prompts of 1 to 32768 tokens, 1 to 32 heads, every chunk size, gate and data type."""
    pick = lambda pairs: rng.choices([p[0] for p in pairs], [p[1] for p in pairs])[0]
    entry = pick([("inv", 5), ("solve", 2), ("solve2", 2), ("tri", 2), ("inv_varlen", 1), ("solve_varlen", 2)])
    C = pick([(64, 6), (128, 4), (32, 1), (16, 1)])
    gate = pick([("scalar", 5), ("channel", 3), ("none", 2)])
    k = pick([("bf16", 7), ("f16", 1), ("f32", 2)])
    applied = entry.startswith("solve")
    dk = pick([(64, 3), (128, 8)] + ([] if applied and C == 128 and gate != "channel" else [(96, 1), (256, 1)]))
    method = pick([("block", 5), ("mixed", 3)] + ([] if applied else [("direct", 1), ("newton", 2), ("forward", 1)]))
    op = pick([("bf16", 5), ("f16", 2), ("f32", 3)])
    if method == "forward":
        op = "f32"
    composed = method in ("mixed", "newton") and C == 128 and entry != "tri" and (dk not in (64, 128) or (k == "f32" and dk == 128))
    out = "f32" if applied or composed or rng.random() < 0.7 else pick([("bf16", 3), ("f16", 1)])
    dx = pick([(64, 2), (128, 6), (256, 1), (72, 1)]) if applied else 0
    H = pick([(1, 1), (2, 1), (3, 1), (4, 3), (8, 3), (12, 1), (16, 4), (32, 2)])
    # token-head pairs, spread over the logarithm; the dearer settings end earlier
    top = 20.0
    if gate == "channel" or op == "f32" or method == "forward" or dk == 256 or dx == 256 or k == "f32":
        top = 19.0
    if method == "newton":
        top = 18.5 if op != "f32" else (18.5 if C <= 64 else 16.5)
    pairs = 2.0 ** rng.uniform(8.0, top)
    tokens = max(1, int(pairs / H))
    if entry.endswith("varlen"):
        B = rng.randint(2, max(2, min(64, tokens // 16)))
    else:
        B = rng.choice([1, 1, 2, 4, 8])
    T = max(1, tokens // B)
    if entry == "tri":
        B, T, H = 1, max(1, int(pairs / C)) * C, 1
    elif rng.random() < 0.5:
        T = max(C, T - T % C)  # half of the prompts end with a whole chunk
    c = _case("", entry=entry, B=B, T=T, H=H, dk=dk, dx=dx, C=C, k=k, op=op, out=out, gate=gate, method=method,
              lens=rng.randint(1, 10**6) if entry.endswith("varlen") else 0)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------------------------
def _seqlens(case):
    """Lengths of the packed sequences: log-uniform around the mean, as prompts in a serving batch are."""
    r = random.Random(case["lens"])
    return [max(1, int(case["T"] * 4.0 ** r.uniform(-1.0, 0.8))) for _ in range(case["B"])]


def _layout(case):
    """(sequences, tokens per sequence) as lists of lengths: what the chunks are cut from."""
    return _seqlens(case) if case["entry"].endswith("varlen") else [case["T"]] * case["B"]


def _chunk_cumsum(rate, C):
    """Running sum along dim 1 of [B, T, ...] that starts again at every chunk."""
    B, T = rate.shape[:2]
    pad = -T % C
    if pad:
        rate = torch.cat([rate, rate.new_zeros(B, pad, *rate.shape[2:])], 1)
    return rate.view(B, -1, C, *rate.shape[2:]).cumsum(2).view(B, T + pad, *rate.shape[2:])[:, :T].contiguous()


def _tokens(case, seed):
    """K, beta, g of the case: [B, T, H, ...], or [tokens, H, ...] for packed sequences."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    lens, H, dk, C = _layout(case), case["H"], case["dk"], case["C"]
    packed = case["entry"].endswith("varlen")
    B, T = (1, sum(lens)) if packed else (case["B"], case["T"])
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    K = rand(B, T, H, dk)
    if case["keys"] == "rank4":
        K.mul_(0.05).add_(torch.einsum("bthr,hrd->bthd", rand(B, T, H, 4), rand(H, 4, dk)))
        beta = 0.9 + 0.1 * torch.rand(B, T, H, generator=gen, device="cuda")
    else:
        beta = torch.sigmoid(rand(B, T, H))
    K = torch.nn.functional.normalize(K, dim=-1).to(_TORCH[case["k"]])
    g = None
    if case["gate"] != "none":
        rate = rand(B, T, H) if case["gate"] == "scalar" else rand(B, T, H, dk)
        rate = torch.nn.functional.softplus(rate).mul_(-_DECAY)
        g = torch.cat([_chunk_cumsum(r, C) for r in rate.split(lens, 1)], 1) if packed else _chunk_cumsum(rate, C)
    if packed:
        K, beta, g = K[0], beta[0], None if g is None else g[0]
    return K, beta, g, gen


def _given(case, seed):
    """Chunk matrices as a layer's own kernel would hand them over: scalar decay, stored in the type asked for."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    C, n, dk = case["C"], case["T"] // case["C"], case["dk"]
    A = torch.empty(n, C, C, device="cuda", dtype=_TORCH[case["k"]])
    for i in range(0, n, 2048):
        m = min(2048, n - i)
        K = torch.nn.functional.normalize(torch.randn(m, C, dk, generator=gen, device="cuda"), dim=-1)
        beta = torch.sigmoid(torch.randn(m, C, 1, generator=gen, device="cuda"))
        g = torch.nn.functional.softplus(torch.randn(m, C, generator=gen, device="cuda")).mul_(-_DECAY).cumsum(1)
        S = torch.bmm(K, K.transpose(1, 2).contiguous()) * beta
        A[i:i + m] = torch.tril(S * torch.exp(torch.tril(g[:, :, None] - g[:, None, :])), -1).to(A.dtype)
    return A


def prepare(case, seed):
    if case["entry"] == "tri":
        return {"case": case, "A": _given(case, seed)}
    K, beta, g, gen = _tokens(case, seed)
    s = {"case": case, "K": K, "beta": beta, "g": g}
    if case["entry"].endswith("varlen"):
        s["seqlens"] = _seqlens(case)
    if case["entry"].startswith("solve"):
        shape = tuple(K.shape[:-1])
        new = lambda: torch.randn(*shape, case["dx"], generator=gen, device="cuda").to(_TORCH[case["op"]])
        s["X"] = new()
        s["scale"] = beta
        if case["entry"] == "solve2":
            s["X2"] = new()
            s["scale2"] = beta * torch.exp(g) if case["gate"] == "scalar" else beta
    return s


# ---------------------------------------------------------------------------------------------------------------------
# The call
# ---------------------------------------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    method, gate, op, out = _METHOD[c["method"]], _GATE[c["gate"]], _CODE[c["op"]], _TORCH[c["out"]]
    if c["entry"] == "tri":
        if c["out"] == "f32" and c["op"] == c["k"]:
            return tri.tri_inv(s["A"], method=method)
        return tri.tri_inv_ex(s["A"], method=method, op_dtype=op, out_dtype=out)
    if c["entry"] == "inv":
        if (c["k"], c["op"], c["out"], c["gate"], c["method"]) == ("bf16", "bf16", "f32", "scalar", "block"):
            return tri.gdn_chunk_tri_inv(s["K"], s["beta"], s["g"], c["C"])
        return tri.gdn_chunk_tri_inv_ex(s["K"], s["beta"], s["g"], c["C"], gate_kind=gate, method=method, op_dtype=op, out_dtype=out)
    if c["entry"] == "inv_varlen":
        return tri.gdn_chunk_tri_inv_varlen(s["K"], s["beta"], s["g"], s["seqlens"], c["C"], gate_kind=gate, method=method, op_dtype=op,
                                            out_dtype=out)
    if c["entry"] == "solve":
        return tri.gdn_chunk_tri_solve(s["K"], s["beta"], s["g"], s["X"], c["C"], row_scale=s["scale"], gate_kind=gate, method=method)
    if c["entry"] == "solve_varlen":
        return tri.gdn_chunk_tri_solve_varlen(s["K"], s["beta"], s["g"], s["X"], s["seqlens"], c["C"], row_scale=s["scale"],
                                              gate_kind=gate, method=method)
    return tri.gdn_chunk_tri_solve_multi(s["K"], s["beta"], s["g"], [s["X"], s["X2"]], c["C"], row_scales=[s["scale"], s["scale2"]],
                                         gate_kind=gate, method=method)


# ---------------------------------------------------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def work(case):
    size = lambda t: 4 if t == "f32" else 2
    C, H, dk, dx = case["C"], case["H"], case["dk"], case["dx"]
    lens = _layout(case)
    n = sum(-(-x // C) for x in lens) * H
    inverse = C ** 3 / 3
    if case["entry"] == "tri":
        return {"bytes": n * (C * (C - 1) // 2 * size(case["k"]) + C * C * size(case["out"])), "flops": n * inverse}
    rows = sum(lens) * H
    read = rows * (dk * size(case["k"]) + 4 + {"scalar": 4, "channel": 4 * dk, "none": 0}[case["gate"]])
    flops = n * (inverse + C * C * dk)
    if not case["entry"].startswith("solve"):
        return {"bytes": read + n * C * C * size(case["out"]), "flops": flops}
    k = 2 if case["entry"] == "solve2" else 1
    return {"bytes": read + k * rows * (4 + 2 * dx * size(case["op"])), "flops": flops + k * n * C * C * dx}


def tolerance(case):
    """About four times the error against 64 bits that was measured for the coarsest of the operand and result types."""
    coarse = case["op"] if case["out"] == "f32" else case["out"] if case["op"] != "bf16" else "bf16"
    if coarse == "f32":
        return {"rel": 1e-6, "max": 4e-5}  # measured 1e-8 ... 5e-8 (the unit diagonal is exact and dominates the norm)
    if case["keys"] == "rank4":
        return {"rel": 3e-2, "max": 0.9}   # measured 9e-3: the inverse amplifies the rounding of correlated keys
    rel = 1e-2 if case["entry"].startswith("solve") else 4e-3  # measured 2.4e-3 and 3e-4 ... 6e-4 in bf16, an eighth in fp16
    if coarse == "f16":
        rel /= 8
    return {"rel": rel, "max": 40 * rel}


# ---------------------------------------------------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------------------------------
def _chunks(x, C, start, end):
    """Rows start .. end of [tokens, H, ...] as [chunks, H, C, ...] in 64 bits, zeros behind the last."""
    x = x[start:end].double()
    pad = -x.shape[0] % C
    if pad:
        x = torch.cat([x, x.new_zeros(pad, *x.shape[1:])])
    return x.view(-1, C, *x.shape[1:]).transpose(1, 2).contiguous()


def _matrices(K, beta, g, C, gate, start, end):
    """I + A of the chunks of one sequence (or whole chunks of it): [chunks * H, C, C]."""
    k, b = _chunks(K, C, start, end).flatten(0, 1), _chunks(beta, C, start, end).flatten(0, 1)
    if gate == "channel":
        d = _chunks(g, C, start, end).flatten(0, 1)
        d = d - d[:, :1] / 2 - d.amin(1, keepdim=True) / 2
        left, right = k * torch.exp(d), (k * torch.exp(-d))
    else:
        left, right = k, k
    A = torch.bmm(left, right.transpose(1, 2).contiguous()) * b[:, :, None]
    if gate == "scalar":
        d = _chunks(g, C, start, end).flatten(0, 1)
        A = A * torch.exp(torch.tril(d[:, :, None] - d[:, None, :]))
    return torch.tril(A, -1) + torch.eye(C, device=A.device, dtype=A.dtype)


def _unit_solve(M, rhs):
    return torch.linalg.solve_triangular(M, rhs, upper=False, unitriangular=True)


def exact(case, seed):
    s = prepare(case, seed)
    C, H = case["C"], case["H"]
    eye = torch.eye(C, device="cuda", dtype=torch.float64)
    if case["entry"] == "tri":
        A, parts = s["A"], []
        for i in range(0, A.shape[0], 2048):
            M = torch.tril(A[i:i + 2048].double(), -1) + eye
            parts.append(_unit_solve(M, eye.expand_as(M).contiguous()))
        return torch.cat(parts)
    flat = lambda x: None if x is None or case["entry"].endswith("varlen") else x.flatten(0, 1)
    K, beta, g = (s[n] if case["entry"].endswith("varlen") else flat(s[n]) for n in ("K", "beta", "g"))
    applied = case["entry"].startswith("solve")
    sides = [("X", "scale"), ("X2", "scale2")][:2 if case["entry"] == "solve2" else 1] if applied else []
    piece = max(1, 4096 // H) * C  # tokens at a time
    results = [torch.empty_like(s[x], dtype=torch.float64) for x, _ in sides]
    inverse, start = [], 0
    for n in _layout(case):
        for a in range(start, start + n, piece):
            e = min(a + piece, start + n)
            M = _matrices(K, beta, g, C, case["gate"], a, e)
            if not applied:
                inverse.append(_unit_solve(M, eye.expand_as(M).contiguous()))
            for (xn, sn), W in zip(sides, results):
                X, sc = (s[v] if case["entry"].endswith("varlen") else flat(s[v]) for v in (xn, sn))
                X = (_chunks(X, C, a, e) * _chunks(sc, C, a, e)[..., None]).flatten(0, 1)
                Y = _unit_solve(M, X).view(-1, H, C, X.shape[-1]).transpose(1, 2).reshape(-1, H, X.shape[-1])
                (W if case["entry"].endswith("varlen") else W.view(-1, H, X.shape[-1]))[a:e] = Y[:e - a]
        start += n
    if not applied:
        return torch.cat(inverse)
    return results if case["entry"] == "solve2" else results[0]
