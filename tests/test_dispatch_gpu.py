"""Rules that send a call to one kernel or launch shape rather than another: both sides of each line give the same result."""
import numpy as np
import pytest
import torch

import paper_2605_21325_amd as tri

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
GATES = [tri.GATE_SCALAR, tri.GATE_PER_CHANNEL, tri.GATE_NONE]


def make_inputs(T, H, d_k, gate, k_dtype=torch.bfloat16, seed=0, B=1):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rand = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    K = torch.nn.functional.normalize(rand(B, T, H, d_k), dim=-1).to(k_dtype)
    beta = torch.sigmoid(rand(B, T, H))
    shape = {tri.GATE_SCALAR: (B, T, H), tri.GATE_PER_CHANNEL: (B, T, H, d_k)}.get(gate)
    g = None if shape is None else -0.01 * (torch.arange(T, device=DEV) % 64).view(1, T, *[1] * (len(shape) - 2)) * torch.rand(
        1, 1, *shape[2:], generator=gen, device=DEV).expand(B, 1, *shape[2:])
    return K, beta, None if g is None else g.expand(*shape).contiguous()


# Up to 512 matrices a workgroup holds one wavefront, above four (with the per-channel gate: one matrix, formed by four of them): a matrix
# does not depend on the others of its call, so the same chunks give the same bits on either side.
@pytest.mark.parametrize("gate", GATES)
@pytest.mark.parametrize("H", [1, 3, 4, 8])
@pytest.mark.parametrize("C", [16, 32, 64])
def test_few_matrices_give_the_bits_of_a_larger_call(C, H, gate):
    most = 512 // H                                   # chunks of the largest call with one wavefront to a workgroup
    T = (most + 1) * C - 5                            # ends inside a chunk
    K, beta, g = make_inputs(T, H, 128 if gate == tri.GATE_PER_CHANNEL else 64, gate)
    X = torch.randn(1, T, H, 72, device=DEV).bfloat16()
    part = lambda x, n: None if x is None else x[:, :n * C].contiguous()
    many = [tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=gate, method=m) for m in (tri.BLOCK_RECURSIVE, tri.NEWTON_SCHULZ)]
    W = tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=beta, gate_kind=gate)
    for n in (1, 2, most):
        k, b, gg, x = part(K, n), part(beta, n), part(g, n), part(X, n)
        for m, T_many in zip((tri.BLOCK_RECURSIVE, tri.NEWTON_SCHULZ), many):
            few = tri.gdn_chunk_tri_inv_ex(k, b, gg, C, gate_kind=gate, method=m)
            assert few.shape[0] <= 512 < T_many.shape[0]
            assert torch.equal(few, T_many[:few.shape[0]])
        w = tri.gdn_chunk_tri_solve(k, b, gg, x, C, row_scale=b, gate_kind=gate)
        assert torch.equal(w, W[:, :n * C])
        w1, w2 = tri.gdn_chunk_tri_solve_multi(k, b, gg, [x, x], C, row_scales=[b, None], gate_kind=gate)
        assert torch.equal(w1, w)


# Plain calls are marshalled natively, all others in Python: same results, same exceptions, and the native route takes no call that the
# other refuses.
def _calls():
    K, beta, g = make_inputs(130, 4, 64, tri.GATE_SCALAR, B=2)
    X = torch.randn(2, 130, 4, 72, device=DEV).bfloat16()
    A = torch.tril(torch.randn(5, 64, 64, device=DEV), -1) * 0.05
    P, pb, pg, px = K[0].contiguous(), beta[0].contiguous(), g[0].contiguous(), X[0].contiguous()
    lens = [64, 1, 65]
    new = lambda *s, dt=torch.float32: torch.zeros(*s, device=DEV, dtype=dt)
    bf = torch.bfloat16
    calls = {
        "tri_inv": lambda: tri.tri_inv(A),
        "tri_inv into T": lambda: tri.tri_inv(A, new(5, 64, 64), method=tri.FWD_SUBST),
        "tri_inv_ex": lambda: tri.tri_inv_ex(A, op_dtype=tri.F16, out_dtype=torch.float16),
        "tri_inv_ex refined": lambda: tri.tri_inv_ex(A, flags=tri.FLAG_REFINE1),
        "no matrices": lambda: tri.tri_inv_ex(A[:0]),
        "short form": lambda: tri.gdn_chunk_tri_inv(K, beta, g, 64),
        "inv": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, g, 32, op_dtype=tri.F32),
        "inv into T": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, None, 128, T=new(16, 128, 128, dt=bf), gate_kind=tri.GATE_NONE, out_dtype=bf),
        "inv on a stream": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, g, 64, stream=torch.cuda.current_stream()),
        "solve": lambda: tri.gdn_chunk_tri_solve(K, beta, g, X, 64, row_scale=beta),
        "solve into W": lambda: tri.gdn_chunk_tri_solve(K, beta, g, X, 64, W=torch.empty_like(X), method=tri.MIXED),
        "two sides": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, [X, X * 2], 64, row_scales=[None, beta]),
        "two sides into W": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, (X, X * 2), 64, Ws=(torch.empty_like(X), torch.empty_like(X))),
        "packed": lambda: tri.gdn_chunk_tri_inv_varlen(P, pb, pg, lens, 64),
        "packed, lengths in a tensor": lambda: tri.gdn_chunk_tri_inv_varlen(P, pb, pg, torch.tensor(lens), 64),
        "packed solve": lambda: tri.gdn_chunk_tri_solve_varlen(P, pb, pg, px, lens, 64, row_scale=pb),
        "packed solve into W": lambda: tri.gdn_chunk_tri_solve_varlen(P, pb, pg, px, tuple(lens), 64, W=torch.empty_like(px)),
    }
    refused = {
        "chunk size": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, g, 48),
        "no gate": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, None, 64),
        "method": lambda: tri.tri_inv_ex(A, method=99),
        "flags": lambda: tri.tri_inv_ex(A, flags=1 << 20),
        "element type": lambda: tri.tri_inv_ex(A.double()),
        "keys of the short form": lambda: tri.gdn_chunk_tri_inv(K.float(), beta, g, 64),
        "16-bit T of the short forms": lambda: tri.tri_inv(A, T=new(5, 64, 64, dt=bf)),
        "16-bit T of the short forms, keys": lambda: tri.gdn_chunk_tri_inv(K, beta, g, 64, T=new(24, 64, 64, dt=torch.float16)),
        "operand type": lambda: tri.tri_inv_ex(A, op_dtype=-1),
        "operand type of keys": lambda: tri.gdn_chunk_tri_inv_ex(K, beta, g, 64, op_dtype=-7),
        "nested matrices": lambda: tri.tri_inv_ex(torch.nested.nested_tensor([A[0], A[1, :32, :32]])),
        "nested keys": lambda: tri.gdn_chunk_tri_inv_ex(torch.nested.nested_tensor([K[0], K[1, :70]]), beta, g, 64),
        "result type": lambda: tri.tri_inv_ex(A, T=new(5, 64, 64), out_dtype=bf),
        "result type unknown": lambda: tri.tri_inv_ex(A, out_dtype=torch.int32),
        "not contiguous": lambda: tri.gdn_chunk_tri_inv_ex(K.transpose(0, 1), beta, g, 64),
        "on the host": lambda: tri.gdn_chunk_tri_inv_ex(K, beta.cpu(), g, 64),
        "dimensions": lambda: tri.gdn_chunk_tri_inv_ex(K[0], beta, g, 64),
        "overlap": lambda: tri.tri_inv_ex(A, T=A),
        "X of another shape": lambda: tri.gdn_chunk_tri_solve(K, beta, g, X[:, 1:].contiguous(), 64),
        "d_x": lambda: tri.gdn_chunk_tri_solve(K, beta, g, X[..., :4].contiguous(), 64),
        "three sides": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, [X] * 3, 64),
        "no sides": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, [], 64),
        "sides of two types": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, [X, X.float()], 64),
        "scales missing": lambda: tri.gdn_chunk_tri_solve_multi(K, beta, g, [X, X], 64, row_scales=[beta]),
        "lengths too short": lambda: tri.gdn_chunk_tri_inv_varlen(P, pb, pg, [64, 1], 64),
        "negative length": lambda: tri.gdn_chunk_tri_inv_varlen(P, pb, pg, [64, -1, 67], 64),
        "length beyond 64 bits": lambda: tri.gdn_chunk_tri_solve_varlen(P, pb, pg, px, [1 << 70, 130], 64),
    }
    return calls, refused


@pytest.mark.filterwarnings("ignore:The PyTorch API of nested tensors")
def test_native_and_python_marshalling_agree(monkeypatch):
    calls, refused = _calls()
    tri.lib()
    assert tri.binding._fast is not None, "the native argument handling is not built"

    def outcome(f):
        try:
            r = f()
        except Exception as e:  # noqa: BLE001 (whatever it is, the other route has to raise it too)
            return type(e), str(e)
        torch.cuda.synchronize()
        return r

    for name, call in {**calls, **refused}.items():
        taken = []
        with monkeypatch.context() as m:
            m.setattr(tri.binding, "_fast", _Watch(tri.binding._fast, taken))
            native = outcome(call)
        with monkeypatch.context() as m:
            m.setattr(tri.binding, "_fast_lib", object())
            python = outcome(call)
        raised = isinstance(python, tuple) and isinstance(python[0], type)
        assert raised == (name in refused), name
        if raised:
            assert native == python and not any(taken), name
            continue
        assert type(native) is type(python), name
        for a, b in zip(*(x if isinstance(x, (list, tuple)) else [x] for x in (native, python))):
            assert a.dtype == b.dtype and torch.equal(a, b), name
            assert hasattr(a, "_triinv_keepalive") == hasattr(b, "_triinv_keepalive"), name
        assert any(taken) == (name not in ("inv on a stream", "packed, lengths in a tensor")), name


class _Watch:
    """The native module; `taken` collects whether it answered each call."""
    def __init__(self, module, taken):
        self.module, self.taken = module, taken

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.module, name)(*a)
            self.taken.append(r is not None)
            return r
        return call


def test_native_marshalling_runs_on_the_current_stream():
    K, beta, g = make_inputs(4096, 16, 128, tri.GATE_SCALAR)
    X = torch.randn(1, 4096, 16, 128, device=DEV).bfloat16()
    want = tri.gdn_chunk_tri_inv_ex(K, beta, g, 64)
    want_w = tri.gdn_chunk_tri_solve(K, beta, g, X, 64)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    K2, beta2, g2, X2 = (torch.zeros_like(x) for x in (K, beta, g, X))
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for dst, src in ((K2, K), (beta2, beta), (g2, g), (X2, X)):
            torch.cuda._sleep(200000)
            dst.copy_(src)
        T = tri.gdn_chunk_tri_inv_ex(K2, beta2, g2, 64)
        W = tri.gdn_chunk_tri_solve(K2, beta2, g2, X2, 64)
    s.synchronize()
    assert torch.equal(T, want) and torch.equal(W, want_w)


# With few matrices the channel loops (per-channel gate, head dimensions without a kernel of their own; fp32 keys of 128 channels at C = 64)
# share a matrix between four wavefronts.  Every method, whatever the number of k-steps (32 channels each) and the chunk's tokens,
# gives the bits of a larger call, where one wavefront forms it.
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("k_dtype", [torch.bfloat16, torch.float16, torch.float32], ids=str)
@pytest.mark.parametrize("d_k", [32, 64, 96, 128, 160, 256])
@pytest.mark.parametrize("C", [16, 32, 64])
def test_teams_of_wavefronts_in_the_channel_loops(C, d_k, k_dtype, op):
    H = 4
    many = 512 // H + 1
    x_type = {tri.F32: torch.float32, tri.F16: torch.float16, tri.BF16: torch.bfloat16}[op]
    for gate in GATES:
        K, beta, g = make_inputs(many * C - 3, H, d_k, gate, k_dtype)
        X = torch.randn(1, many * C - 3, H, 40, device=DEV).to(x_type)
        calls = {tri.METHOD_NAMES[m]: (lambda k, b, gg, x, m=m: tri.gdn_chunk_tri_inv_ex(k, b, gg, C, gate_kind=gate, method=m, op_dtype=op))
                 for m in tri.METHOD_NAMES if C > 16 or m != tri.MIXED_B32}
        if gate == tri.GATE_PER_CHANNEL:
            calls["refined"] = lambda k, b, gg, x: tri.gdn_chunk_tri_inv_ex(k, b, gg, C, gate_kind=gate, op_dtype=op, flags=tri.FLAG_REFINE1)
        calls["A"] = lambda k, b, gg, x: tri.gdn_chunk_build_A(k, b, gg, C, gate_kind=gate, op_dtype=op)
        for m in (tri.BLOCK_RECURSIVE, tri.MIXED):
            calls["applied " + tri.METHOD_NAMES[m]] = lambda k, b, gg, x, m=m: tri.gdn_chunk_tri_solve(k, b, gg, x, C, gate_kind=gate, method=m)
            calls["two sides " + tri.METHOD_NAMES[m]] = lambda k, b, gg, x, m=m: tri.gdn_chunk_tri_solve_multi(
                k, b, gg, [x, x], C, row_scales=[b, None], gate_kind=gate, method=m)[1]
        for name, call in calls.items():
            every = call(K, beta, g, X)
            for tokens in (C, C - 5, 2 * C + 1, 256 // H * C, 512 // H * C):
                few = call(*(None if x is None else x[:, :tokens].contiguous() for x in (K, beta, g, X)))
                if few.dim() == 4:  # applied
                    rows = tokens if tokens < C else tokens // C * C
                    same = torch.equal(few[:, :rows], every[:, :rows])
                else:
                    whole, v = max(1, tokens // C) * H, min(tokens, C)  # (a short chunk: the leading block of the whole one)
                    same = torch.equal(few[:whole, :v, :v], every[:whole, :v, :v])
                assert same, (name, gate, tokens)


# Beyond 8192 matrices some per-channel kernels no longer load gate rows a k-step ahead: the order of loads, not of sums.
@pytest.mark.parametrize("k_dtype", [torch.bfloat16, torch.float32], ids=str)
@pytest.mark.parametrize("C,op", [(32, tri.F32), (64, tri.BF16), (64, tri.F32)])
def test_more_than_8192_matrices_give_the_bits_of_a_smaller_call(C, op, k_dtype):
    H = 8
    K, beta, g = make_inputs(1030 * C, H, 64, tri.GATE_PER_CHANNEL, k_dtype)
    T = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, op_dtype=op)
    assert T.shape[0] > 8192
    for n in (40, 90, 1000):  # a team per matrix, a workgroup of four matrices, ahead
        part = tri.gdn_chunk_tri_inv_ex(*(x[:, :n * C].contiguous() for x in (K, beta, g)), C, gate_kind=tri.GATE_PER_CHANNEL, op_dtype=op)
        assert torch.equal(part, T[:n * H]), n


# Two right-hand sides at C = 128 with fp32 operands take turns on one set of published tiles: each side as if it were the only one.
@pytest.mark.parametrize("gate", GATES)
@pytest.mark.parametrize("k_dtype,d_k", [(torch.bfloat16, 128), (torch.float32, 64)])
@pytest.mark.parametrize("T,d_x", [(128, 64), (300, 128), (131, 200), (7, 8)])
def test_two_fp32_sides_at_c128(T, d_x, k_dtype, d_k, gate):
    K, beta, g = make_inputs(T, 3, d_k, gate, k_dtype)
    X1, X2 = (torch.randn(1, T, 3, w, device=DEV) for w in (d_x, 40))
    W1, W2 = tri.gdn_chunk_tri_solve_multi(K, beta, g, [X1, X2], 128, row_scales=[beta, None], gate_kind=gate)
    for X, s, W in ((X1, beta, W1), (X2, None, W2)):
        one = tri.gdn_chunk_tri_solve(K, beta, g, X, 128, row_scale=s, gate_kind=gate)
        assert (W - one).abs().max() <= 3e-6 * one.abs().max()  # the same fp32 products, summed tile by tile in another order


# The offsets of packed sequences travel as arguments of three sizes (up to 15, 63 and 229 sequences) and, beyond, of several launches.
@pytest.mark.parametrize("n_seq", [1, 15, 16, 63, 64, 229, 230, 500])
def test_offsets_of_packed_sequences_in_blocks(n_seq):
    lens = [1 + (7 * i) % 37 for i in range(n_seq)]
    K, beta, g = (x[0] for x in make_inputs(sum(lens), 2, 64, tri.GATE_SCALAR))
    T = tri.gdn_chunk_tri_inv_varlen(K, beta, g, lens, 16)
    start = chunk = 0
    for n in lens:
        part = [x[start:start + n][None].clone() for x in (K, beta, g)]  # (16-byte aligned)
        one = tri.gdn_chunk_tri_inv_ex(*part, 16)
        assert torch.equal(T[chunk:chunk + one.shape[0]], one)
        start, chunk = start + n, chunk + one.shape[0]
    assert chunk == T.shape[0]


# Packed sequences whose lengths travel as kernel arguments (the native route; 384 bits of them for inverses, 768 for the applied inverse) against
# the offsets in memory that the Python route uses: the same bits, whatever the kernel.
@pytest.mark.parametrize("C, gate, d_k, op", [(16, tri.GATE_SCALAR, 64, tri.BF16), (32, tri.GATE_PER_CHANNEL, 64, tri.BF16), (64, tri.GATE_SCALAR, 128, tri.F32),
                                              (64, tri.GATE_NONE, 96, tri.BF16), (128, tri.GATE_SCALAR, 128, tri.BF16), (128, tri.GATE_PER_CHANNEL, 64, tri.BF16)])
@pytest.mark.parametrize("n_seq, longest", [(1, 700), (2, 700), (17, 60000), (33, 2047), (33, 2048), (48, 65535), (64, 63), (64, 700), (65, 63)])
def test_packed_lengths_as_arguments_and_in_memory(monkeypatch, C, gate, d_k, op, n_seq, longest):
    H = 3
    r = np.random.default_rng(n_seq)
    lens = [min(int(x), longest) for x in r.choice([0, 1, C - 1, C, C + 1, 3 * C + 5], n_seq)]
    lens[n_seq // 2] = longest
    total = sum(lens)
    gen = torch.Generator(device=DEV).manual_seed(n_seq)
    K = torch.nn.functional.normalize(torch.randn(total, H, d_k, generator=gen, device=DEV), dim=-1).bfloat16()
    beta = torch.rand(total, H, generator=gen, device=DEV)
    g = None if gate == tri.GATE_NONE else -0.01 * torch.rand(total, H, *([d_k] if gate == tri.GATE_PER_CHANNEL else []), generator=gen, device=DEV)
    X = torch.randn(total, H, 72, generator=gen, device=DEV).to(torch.float32 if op == tri.F32 else torch.bfloat16)
    def calls():
        T = tri.gdn_chunk_tri_inv_varlen(K, beta, g, lens, C, gate_kind=gate, op_dtype=op)
        return T, tri.gdn_chunk_tri_solve_varlen(K, beta, g, X, lens, C, row_scale=beta, gate_kind=gate)
    native = calls()
    bits = longest.bit_length()
    assert tri.binding._fast is not None
    for r, words in zip(native, (12, 24)):
        assert (r._triinv_keepalive == ()) == (n_seq <= 64 and n_seq * max(bits, max(lens).bit_length()) <= 32 * words)
    monkeypatch.setattr(tri.binding, "_fast_lib", None)
    python = calls()
    assert len(python[0]._triinv_keepalive) == 1
    for a, b in zip(native, python):
        assert torch.equal(a, b)


# The same over the methods whose storing kernels take lengths, on both sides of the lines between few and many matrices.
@pytest.mark.parametrize("C, d_k", [(16, 64), (32, 96), (64, 64), (64, 96), (64, 128), (128, 64), (128, 96), (128, 128)])  # (96: channel loops; at C = 128 "mixed" and Newton-Schulz build A first)
@pytest.mark.parametrize("gate", [tri.GATE_SCALAR, tri.GATE_PER_CHANNEL])
@pytest.mark.parametrize("method, op", [(tri.FWD_SUBST, tri.F32), (tri.MIXED, tri.F32), (tri.MIXED, tri.F16), (tri.BLOCK_DIRECT, tri.BF16),
                                        (tri.NEWTON_SCHULZ, tri.F32), (tri.NEWTON_SCHULZ, tri.BF16)])
def test_packed_lengths_for_every_method(monkeypatch, method, op, gate, C, d_k):
    H = 5
    lines = {16: [512], 32: [512], 64: [256, 512, 768], 128: [256]}[C]
    for chunks in [3] + [m // H for m in lines] + [m // H + 1 for m in lines]:
        lens = [C + 1, 1, 0, C]                                  # four chunks, the second of one token
        lens += [(chunks - 4) * C - C // 2] if chunks > 4 else []
        K, beta, g = (x[0] for x in make_inputs(sum(lens), H, d_k, gate))
        call = lambda: tri.gdn_chunk_tri_inv_varlen(K, beta, g, lens, C, gate_kind=gate, method=method, op_dtype=op)
        with monkeypatch.context() as python_route:
            python_route.setattr(tri.binding, "_fast_lib", None)
            python = call()
        native = call()
        offsets = (C, gate, method) == (128, tri.GATE_PER_CHANNEL, tri.FWD_SUBST) or (  # kernels that are not given lengths
            (method == tri.NEWTON_SCHULZ and C <= 64 or method == tri.MIXED and (C <= 32 or C == 64 and chunks * H > 768)) and
            gate == tri.GATE_SCALAR and d_k != 96)
        assert (native._triinv_keepalive == ()) == (not offsets) and native.shape[0] == max(chunks, 4) * H
        assert len(python._triinv_keepalive) == 1 and torch.equal(native, python), chunks


# Rows of 2^31 bytes and more per chunk: at C = 128 with 16-bit operands a kernel that is not given lengths.
@pytest.mark.parametrize("d_x, native", [(504, True), (512, False)])
def test_packed_lengths_beside_wide_rows(monkeypatch, d_x, native):
    H, lens = 1 << 14, [2, 1]
    K, beta, g = (x[0] for x in make_inputs(3, H, 128, tri.GATE_SCALAR))
    X = torch.randn(3, H, d_x, device=DEV, dtype=torch.bfloat16)
    call = lambda: tri.gdn_chunk_tri_solve_varlen(K, beta, g, X, lens, 128, row_scale=beta)
    W = call()
    assert (W._triinv_keepalive == ()) == native
    want = (beta[..., None] * X.float())
    want[1] -= (beta[1] * (K[1].float() * K[0].float()).sum(-1) * torch.exp(g[1] - g[0]))[:, None] * want[0]
    assert (W.float() - want).norm() <= 1e-2 * want.norm()
    monkeypatch.setattr(tri.binding, "_fast_lib", None)
    assert torch.equal(call(), W)


# C = 128, head dimensions without a kernel of their own: up to 256 matrices four wavefronts form one (and its diagonal tiles once), above one wavefront:
# the same bits.  fp32 keys of 128 channels with fp32 operands go this way too; "mixed" builds A first.
@pytest.mark.parametrize("k_dtype, d_k", [(torch.float32, 128), (torch.float32, 256), (torch.bfloat16, 96), (torch.float16, 160)])
@pytest.mark.parametrize("method, op", [(tri.FWD_SUBST, tri.F32), (tri.BLOCK_RECURSIVE, tri.F32), (tri.BLOCK_DIRECT, tri.BF16), (tri.MIXED, tri.F32)])
def test_teams_of_large_chunks_give_the_bits_of_a_larger_call(method, op, k_dtype, d_k):
    C, H, most = 128, 4, 64
    T = (most + 1) * C - 5
    K, beta, g = make_inputs(T, H, d_k, tri.GATE_SCALAR, k_dtype)
    many = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, method=method, op_dtype=op)
    for tokens in (1, C, 3 * C + 17, most * C):
        k, b, gg = (x[:, :tokens].contiguous() for x in (K, beta, g))
        few = tri.gdn_chunk_tri_inv_ex(k, b, gg, C, method=method, op_dtype=op)
        whole = tokens // C * H
        assert torch.equal(few[:whole], many[:whole]), tokens
        if tokens % C:  # the short last chunk: the leading block of the whole one
            v = tokens % C
            assert torch.equal(few[whole:, :v, :v], many[whole:whole + H, :v, :v]), tokens


# Newton-Schulz at C = 128: up to 256 matrices eight wavefronts, of which two share a pair of tile rows by even and odd tile columns, above four with a
# pair each: the same bits, from keys and from given matrices.
@pytest.mark.parametrize("k_dtype, d_k", [(torch.bfloat16, 64), (torch.float16, 128), (torch.float32, 64)], ids=str)
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("gate", GATES)
def test_newton_schulz_by_eight_wavefronts_gives_the_bits_of_a_larger_call(gate, op, k_dtype, d_k):
    C, H, most = 128, 2, 128
    T = (most + 1) * C - 9
    K, beta, g = make_inputs(T, H, d_k, gate, k_dtype)
    part = lambda x, t: None if x is None else x[:, :t].contiguous()
    run = lambda t, o: tri.gdn_chunk_tri_inv_ex(part(K, t), part(beta, t), part(g, t), C, gate_kind=gate, method=tri.NEWTON_SCHULZ, op_dtype=op, out_dtype=o)
    for o in (torch.float32, torch.bfloat16):
        many = run(T, o)
        for t in (C, 3 * C, most * C):
            assert torch.equal(run(t, o), many[:t // C * H]), t
        last = [None if x is None else x[:, most * C:].contiguous() for x in (K, beta, g)]  # the short chunk by itself
        assert torch.equal(tri.gdn_chunk_tri_inv_ex(*last, C, gate_kind=gate, method=tri.NEWTON_SCHULZ, op_dtype=op, out_dtype=o), many[most * H:])
    A = torch.tril(torch.randn(257, C, C, device=DEV) * 0.03, -1).to(k_dtype)
    many = tri.tri_inv_ex(A, method=tri.NEWTON_SCHULZ, op_dtype=op)
    for n in (1, 5, 256):
        assert torch.equal(tri.tri_inv_ex(A[:n].contiguous(), method=tri.NEWTON_SCHULZ, op_dtype=op), many[:n]), n


# Methods without a kernel of their own for a head dimension at C = 128: A is written into T and inverted there, also where wavefronts store tile rows that
# others have fetched.  The bits of the same A inverted elsewhere.
@pytest.mark.parametrize("H", [1, 64, 257])
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("method, flags", [(tri.NEWTON_SCHULZ, 0), (tri.NEWTON_SCHULZ, tri.flag_iters(1)), (tri.NEUMANN, 0), (tri.MIXED, 0)])
@pytest.mark.parametrize("tokens", [1, 4 * 128])
def test_matrices_inverted_in_place(tokens, method, flags, op, H):
    K, beta, g = make_inputs(tokens, H, 96, tri.GATE_SCALAR, torch.float32)
    T = tri.gdn_chunk_tri_inv_ex(K, beta, g, 128, method=method, op_dtype=op, flags=flags)
    A = tri.gdn_chunk_build_A(K, beta, g, 128, op_dtype=op)
    assert torch.equal(T, tri.tri_inv_ex(A, method=method, op_dtype=op, flags=flags))


# C = 64, up to 768 matrices (direct leaves 256, applied 512): four wavefronts carry one matrix through the recursion and the store too; C = 128, up to 256:
# eight.  The bits of larger calls, on chunks that end anywhere in a tile; both element types of a result.
@pytest.mark.parametrize("C, most", [(64, 256), (128, 85)])  # chunks of the largest call by team, with three heads
@pytest.mark.parametrize("gate, k_dtype, d_k", [(g, k, d) for g in (tri.GATE_SCALAR, tri.GATE_NONE, tri.GATE_PER_CHANNEL)
                                                for k, d in ((torch.bfloat16, 64), (torch.float16, 128), (torch.float32, 64), (torch.float32, 128))]
                         + [(tri.GATE_PER_CHANNEL, torch.bfloat16, 32), (tri.GATE_PER_CHANNEL, torch.float32, 160), (tri.GATE_PER_CHANNEL, torch.float16, 256)], ids=str)
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_teams_through_the_recursion_give_the_bits_of_a_larger_call(op, k_dtype, d_k, gate, C, most):
    H = 3
    T = (most + 1) * C - 7
    K, beta, g = make_inputs(T, H, d_k, gate, k_dtype)
    part = lambda x, t: None if x is None else x[:, :t].contiguous()
    x_dtype = {tri.F32: torch.float32, tri.F16: torch.float16, tri.BF16: torch.bfloat16}[op]
    Xs = [torch.randn(1, T, H, d_x, device=DEV).to(x_dtype) for d_x in (72, 200)]
    def calls(t):
        k, b, gg, xs = part(K, t), part(beta, t), part(g, t), [part(x, t) for x in Xs]
        Ts = [tri.gdn_chunk_tri_inv_ex(k, b, gg, C, gate_kind=gate, method=m, op_dtype=op, out_dtype=o, flags=f)
              for m, o, f in ((tri.BLOCK_RECURSIVE, torch.float32, 0), (tri.MIXED, x_dtype, 0), (tri.MIXED, torch.float32, tri.flag_mxr_r(2)),
                              (tri.BLOCK_DIRECT, torch.float32, 0))]
        Ws = [tri.gdn_chunk_tri_solve(k, b, gg, xs[0], C, gate_kind=gate),
              *tri.gdn_chunk_tri_solve_multi(k, b, gg, xs, C, row_scales=[b, None], gate_kind=gate, method=tri.MIXED)]
        return Ts, Ws
    many, applied = calls(T)
    for t in (1, 16, 17, C - 1, C, C + 33, C + 100, 85 * C, 170 * C, most * C):
        if t > most * C: continue
        Ts, Ws = calls(t)
        whole, v = t // C * H, t % C
        for a, b in zip(Ts, many):
            assert torch.equal(a[:whole], b[:whole]), t
            if v:
                assert torch.equal(a[whole:, :v, :v], b[whole:whole + H, :v, :v]), t
                assert torch.equal(a[whole:, v:, v:], torch.eye(C - v, device=DEV).to(a.dtype).expand(H, -1, -1)) and not a[whole:, v:, :v].any(), t
        for a, b in zip(Ws, applied):
            assert torch.equal(a, b[:, :t]), t


# Applied to one side, fp16 keys of 64 channels at C = 64: the kernel of the larger calls has offsets in memory, the others lengths.
@pytest.mark.parametrize("method, k_dtype, chunks, offsets", [(tri.BLOCK_RECURSIVE, torch.float16, 128, False), (tri.BLOCK_RECURSIVE, torch.float16, 130, True),
                                                              (tri.MIXED, torch.float16, 130, False), (tri.BLOCK_RECURSIVE, torch.bfloat16, 130, False)])
def test_packed_applied_calls_of_fp16_keys(monkeypatch, method, k_dtype, chunks, offsets):
    H, lens = 4, [1, 65, (chunks - 4) * 64, 7]
    K, beta, g = (x[0] for x in make_inputs(sum(lens), H, 64, tri.GATE_SCALAR, k_dtype))
    X = torch.randn(sum(lens), H, 72, device=DEV).to(k_dtype)
    call = lambda: tri.gdn_chunk_tri_solve_varlen(K, beta, g, X, lens, 64, row_scale=beta, method=method)
    W = call()
    assert (W._triinv_keepalive == ()) == (not offsets)
    monkeypatch.setattr(tri.binding, "_fast_lib", None)
    assert torch.equal(W, call())


# Forward substitution at C = 64: fp32 keys of 64 channels have offsets in memory, of 128 and 16-bit ones lengths.
@pytest.mark.parametrize("k_dtype, d_k, offsets", [(torch.float32, 64, True), (torch.float32, 128, False), (torch.float16, 64, False)])
@pytest.mark.parametrize("chunks", [5, 150])
def test_packed_calls_of_forward_substitution(monkeypatch, chunks, k_dtype, d_k, offsets):
    H, lens = 4, [1, 65, (chunks - 4) * 64, 7]
    K, beta, g = (x[0] for x in make_inputs(sum(lens), H, d_k, tri.GATE_SCALAR, k_dtype))
    call = lambda: tri.gdn_chunk_tri_inv_varlen(K, beta, g, lens, 64, method=tri.FWD_SUBST, op_dtype=tri.F32)
    T = call()
    assert (T._triinv_keepalive == ()) == (not offsets)
    monkeypatch.setattr(tri.binding, "_fast_lib", None)
    assert torch.equal(T, call())
