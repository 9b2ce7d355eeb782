"""Parity of the HIP path against the fp64 CPU oracle, element by element, on the same seeded
inputs, through the C-ABI.  Tolerances (relative Frobenius error per matrix, maximum over the
batch): 1e-5 for the fp32 path (forward substitution, fp32 matrix-core operands), 2e-2 for
fp16 / bf16 operands.  The Neumann product is held to them on the benign workloads only; on the
stress workload the paper predicts it breaks, and its error is reported, not asserted."""
import math

import numpy as np
import pytest
import torch

import oracle
from oracle import metrics
import synth_inputs as si
import paper_2605_21325_amd as tri

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {tri.F32: 1e-5, tri.F16: 2e-2, tri.BF16: 2e-2}
MFMA_METHODS = [tri.BLOCK_RECURSIVE, tri.BLOCK_DIRECT, tri.MIXED, tri.NEUMANN]
_OPS = (tri.F32, tri.F16, tri.BF16)
ALL = [(tri.FWD_SUBST, tri.F32)] + [(m, o) for m in MFMA_METHODS for o in (tri.F32, tri.F16, tri.BF16)]


def ids(mo):
    return f"{tri.METHOD_NAMES[mo[0]]}-{tri.DTYPE_NAMES[mo[1]]}"


# Unit roundoff of the matrix-core operand types (round to nearest even).
UNIT = {tri.F32: 2.0 ** -24, tri.F16: 2.0 ** -11, tri.BF16: 2.0 ** -8}
SKIP = "skip"


def elementwise_bound(T_ref: np.ndarray, op: int, key_abs=None, ns_iters=None) -> np.ndarray:
    """First-order worst-case bound on every element of T_gpu - T for the blocked methods (and, with its C sequential
    fp32 multiply-adds per element, forward substitution).  One level of the 2 x 2 recursion forms -T22 (A21 T11): two
    chained products, both operands of each rounded to the operand type (unit roundoff u), so a level contributes at
    most 4u relative to the magnitudes it multiplies; log2 C levels; fp32 accumulation adds C 2^-24.  A right residual
    R = X(I + A) - I with |R| <= c |X| |I + A| gives |X - T| = |R T| <= c |T| |I + A| |T|:
        E = (4 log2(C) u + C 2^-24) |T| |I + A| |T| + 1e-6.
    key_abs (per-channel gate with 16-bit operands): the gated keys themselves are rounded, which perturbs A by at most
    2u beta_i sum_c |k_ic k_jc| exp(g_ic - g_jc) -- not proportional to |A_ij| when the dot product cancels -- and T by
    |T| dA |T|; key_abs is that sum (the oracle's build of A on |K|).
    ns_iters (Newton-Schulz, m iterations from X0 = I / C): the iterate is not the inverse but, in exact arithmetic,
    X_m = T (I - R0^(2^m)) with R0 = I - (I + A) / C (paper Eq. 8); that truncation |T R0^(2^m)| is added."""
    C = T_ref.shape[-1]
    Ta = np.abs(T_ref)
    M = np.abs(np.linalg.inv(T_ref))                      # |I + A|: unit lower triangular, kappa <= C^2, exact enough in fp64
    u = UNIT[op]
    E = (4 * np.log2(C) * u + C * 2.0 ** -24) * (Ta @ M @ Ta) + 1e-6
    if key_abs is not None:
        E = E + 2 * u * (Ta @ np.abs(key_abs) @ Ta)
    if ns_iters is not None:
        R = np.eye(C) - np.linalg.inv(T_ref) / C
        for _ in range(ns_iters):
            R = R @ R
        E = E + np.abs(T_ref @ R)
    return E


def key_abs_term(inp, gate_kind, C):
    """The matrix beta_i sum_c |k_ic k_jc| exp(g_ic - g_jc) for the per-channel gate (None for the other kinds)."""
    if gate_kind != tri.GATE_PER_CHANNEL:
        return None
    return oracle.build_A_ragged(inp["K"].abs(), inp["beta"], inp["g"], gate_kind, C)


def check(T_gpu: torch.Tensor, T_ref: np.ndarray, tol: float, what: str, op=None, key_abs=None, method=None):
    """Exact structure, the per-matrix relative Frobenius tolerance, and -- for the two standard tolerances -- the
    elementwise bound above (op: operand type; by default fp32 for the 1e-5 tolerance, bf16 for 2e-2).
    key_abs = SKIP leaves the elementwise bound out (per-channel gate with 16-bit operands where the caller has no
    inputs at hand to form the rounded-key term)."""
    torch.cuda.synchronize()
    Tg = T_gpu.cpu().numpy()
    assert metrics.structure_ok(Tg), f"{what}: not exactly unit lower triangular"
    Tg = Tg.astype(np.float64)
    err = metrics.forward_errors(T_ref, Tg)["rel_fro"]
    assert np.isfinite(err).all(), f"{what}: non-finite output"
    assert err.max() <= tol, f"{what}: rel_fro max {err.max():.3e} > {tol}"
    if tol in (1e-5, 2e-2) and key_abs is not SKIP:
        if op is None:
            op = tri.F32 if tol == 1e-5 else tri.BF16
        C = T_ref.shape[-1]
        ns_iters = 2 * int(np.log2(C)) if method == tri.NEWTON_SCHULZ else None      # the library's default count
        ratio = np.abs(Tg - T_ref) / elementwise_bound(T_ref, op, key_abs, ns_iters)
        worst = np.unravel_index(np.argmax(ratio), ratio.shape)
        assert ratio.max() <= 1.0, (f"{what}: element {worst} off by {abs(Tg[worst] - T_ref[worst]):.3e}, "
                                    f"{ratio.max():.2f} x its bound")
    return err.max()


@pytest.fixture(scope="module")
def cases():
    """Small instances of every workload recipe: inputs, fp64 A, fp64 T."""
    out = {}
    for idx, kw in [(0, {}), (1, dict(Tlen=1024)), (2, dict(B=2, Tlen=512, H=5)), (3, dict(B=2, Tlen=512, H=3)),
                    (4, dict(Tlen=512, H=3))]:
        inp = si.make_inputs(si.workload(idx, **kw))
        w = inp["workload"]
        A = oracle.build_A(inp["K"], inp["beta"], inp["g"], w.gate_kind, w.C)
        out[idx] = dict(inp=inp, w=w, A=A, T=oracle.tri_inv(A), key_abs=key_abs_term(inp, w.gate_kind, w.C))
    return out


# ------------------------------------------------------------------ standalone tri_inv
@pytest.mark.parametrize("mo", ALL, ids=ids)
@pytest.mark.parametrize("idx", [0, 1, 4])
def test_tri_inv_fp32_input(cases, idx, mo):
    method, op = mo
    c = cases[idx]
    if idx == 4 and method == tri.NEUMANN:
        pytest.skip("Neumann product on the stress input: reported, not asserted (see the last test)")
    A32 = torch.from_numpy(c["A"].astype(np.float32))
    T_ref = oracle.tri_inv(A32)                      # oracle on the values as stored
    T = tri.tri_inv_ex(A32.to(DEV), method=method, op_dtype=op)
    check(T, T_ref, TOL[op], f"cfg{idx} {ids(mo)}", op=op)


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("method", [tri.FWD_SUBST, tri.BLOCK_RECURSIVE, tri.NEUMANN, tri.MIXED, tri.BLOCK_DIRECT])
def test_tri_inv_16bit_input_short_form(cases, dt, method):
    # short form: operands in the input's own type; the oracle widens the stored values exactly
    A = torch.from_numpy(cases[1]["A"].astype(np.float32)).to(dt)
    T_ref = oracle.tri_inv(A)
    T = tri.tri_inv(A.to(DEV), method=method)
    check(T, T_ref, 1e-5 if method == tri.FWD_SUBST else 2e-2, f"short form {dt} {tri.METHOD_NAMES[method]}")
    # same stored values, fp32 operands: the fp32 tolerance holds against the same oracle result
    T = tri.tri_inv_ex(A.to(DEV), method=method, op_dtype=tri.F32)
    check(T, T_ref, 1e-5, f"{dt} input, f32 operands")


@pytest.mark.parametrize("C", [64, 128])
@pytest.mark.parametrize("mo", [(tri.FWD_SUBST, tri.F32), (tri.BLOCK_RECURSIVE, tri.F32), (tri.BLOCK_RECURSIVE, tri.BF16),
                                (tri.MIXED, tri.F16), (tri.NEUMANN, tri.F32), (tri.BLOCK_DIRECT, tri.F32),
                                (tri.BLOCK_DIRECT, tri.BF16)], ids=ids)
def test_entries_on_and_above_the_diagonal_are_ignored(C, mo):
    method, op = mo
    n = 37  # ragged: not a multiple of anything
    dirty = si.random_strict_lower(n, C, 0.5 / np.sqrt(C), seed=3, garbage_upper=True)
    clean = si.random_strict_lower(n, C, 0.5 / np.sqrt(C), seed=3, garbage_upper=False)
    assert torch.equal(torch.tril(dirty, -1), torch.tril(clean, -1))
    Td = tri.tri_inv_ex(dirty.to(DEV), method=method, op_dtype=op)
    Tc = tri.tri_inv_ex(clean.to(DEV), method=method, op_dtype=op)
    torch.cuda.synchronize()
    assert torch.equal(Td, Tc)                       # bit-identical: garbage never enters the arithmetic
    check(Tc, oracle.tri_inv(clean), TOL[op], f"random lower C={C} {ids(mo)}")


@pytest.mark.parametrize("n_mat", [0, 1, 3])
def test_tiny_batches(n_mat):
    A = si.random_strict_lower(max(n_mat, 1), 64, 0.05, seed=4, garbage_upper=False)[:n_mat].contiguous()
    guard = torch.full((n_mat + 1, 64, 64), 7.0, device=DEV)
    T = tri.tri_inv_ex(A.to(DEV), T=guard[:n_mat], method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)
    torch.cuda.synchronize()
    assert (guard[n_mat] == 7.0).all()               # nothing written past the batch
    if n_mat:
        check(T, oracle.tri_inv(A), 1e-5, f"n_mat={n_mat}")


def test_non_finite_values_stay_in_their_matrix():
    A = si.random_strict_lower(5, 64, 0.05, seed=5, garbage_upper=False)
    A[2, 40, 3] = float("nan")
    A[3, 10, 9] = float("inf")
    ref = oracle.tri_inv(A)
    for method, op in [(tri.FWD_SUBST, tri.F32), (tri.BLOCK_RECURSIVE, tri.BF16), (tri.NEUMANN, tri.F32),
                       (tri.BLOCK_DIRECT, tri.F32)]:
        T = tri.tri_inv_ex(A.to(DEV), method=method, op_dtype=op).cpu().numpy()
        for m in (0, 1, 4):
            e = metrics.forward_errors(ref[m][None], T[m][None].astype(np.float64))["rel_fro"][0]
            assert e <= TOL[op]
        assert not np.isfinite(T[2]).all() and not np.isfinite(T[3]).all()


def test_runs_on_the_callers_stream(cases):
    c = cases[1]
    A32 = torch.from_numpy(c["A"].astype(np.float32)).to(DEV)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        T = tri.tri_inv_ex(A32, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)          # picks the current stream
        T2 = tri.tri_inv_ex(A32, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32, stream=s)
    s.synchronize()
    assert torch.equal(T, T2)
    check(T, oracle.tri_inv(A32.cpu()), 1e-5, "side stream")


# ------------------------------------------------------------------ fused gdn_chunk_tri_inv
@pytest.mark.parametrize("mo", ALL, ids=ids)
@pytest.mark.parametrize("idx", [0, 1, 2, 3, 4])
def test_fused_matches_oracle(cases, idx, mo):
    method, op = mo
    c = cases[idx]
    w, inp = c["w"], c["inp"]
    if idx == 4 and method == tri.NEUMANN:
        pytest.skip("Neumann product on the stress input: reported, not asserted (see the last test)")
    g = None if inp["g"] is None else inp["g"].to(DEV)
    T = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, w.C, gate_kind=w.gate_kind,
                                 method=method, op_dtype=op)
    check(T, c["T"], TOL[op], f"fused cfg{idx} {ids(mo)}", op=op, key_abs=c["key_abs"])


def test_fused_short_form_and_f16_keys(cases):
    c = cases[1]
    w, inp = c["w"], c["inp"]
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    T = tri.gdn_chunk_tri_inv(K, beta, g, w.C)
    check(T, c["T"], 2e-2, "short form")
    T_ex = tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=tri.GATE_SCALAR, method=tri.BLOCK_RECURSIVE, op_dtype=tri.BF16)
    torch.cuda.synchronize()
    assert torch.equal(T, T_ex)
    # fp16 keys: the same recipe stored in fp16
    K16 = inp["K"].to(torch.float16)
    ref = oracle.gdn_chunk_tri_inv(K16, inp["beta"], inp["g"], w.gate_kind, w.C)
    T16 = tri.gdn_chunk_tri_inv_ex(K16.to(DEV), beta, g, w.C, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)
    check(T16, ref, 1e-5, "fp16 keys")


def test_fused_gate_kinds_agree(cases):
    # zero log-decay through the scalar-gate path == the no-gate path, bit for bit
    c = cases[1]
    w, inp = c["w"], c["inp"]
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    z = torch.zeros_like(inp["g"]).to(DEV)
    T0 = tri.gdn_chunk_tri_inv_ex(K, beta, None, w.C, gate_kind=tri.GATE_NONE, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)
    Tz = tri.gdn_chunk_tri_inv_ex(K, beta, z, w.C, gate_kind=tri.GATE_SCALAR, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)
    torch.cuda.synchronize()
    assert torch.equal(T0, Tz)


def test_per_channel_gate_reduces_to_scalar_gate(cases):
    # the same log-decay on every channel through the per-channel kernel == the scalar-gate kernel's matrix
    c = cases[2]
    w, inp = c["w"], c["inp"]
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g4 = inp["g"][..., None].expand(-1, -1, -1, w.d_k).contiguous().to(DEV)
    for method, op in [(tri.BLOCK_RECURSIVE, tri.F32), (tri.FWD_SUBST, tri.F32), (tri.NEUMANN, tri.F32), (tri.MIXED, tri.BF16),
                       (tri.BLOCK_DIRECT, tri.F32)]:
        T = tri.gdn_chunk_tri_inv_ex(K, beta, g4, w.C, gate_kind=tri.GATE_PER_CHANNEL, method=method, op_dtype=op)
        check(T, c["T"], TOL[op], f"per-channel == scalar {ids((method, op))}", op=op,
              key_abs=oracle.build_A(inp["K"].abs(), inp["beta"], inp["g"], w.gate_kind, w.C))


def test_per_channel_gate_fp32_and_fp16_keys(cases):
    c = cases[3]
    w, inp = c["w"], c["inp"]
    beta, g = inp["beta"].to(DEV), inp["g"].to(DEV)
    for dt in (torch.float32, torch.float16):
        Kd = inp["K"].to(dt)
        ref = oracle.gdn_chunk_tri_inv(Kd, inp["beta"], inp["g"], w.gate_kind, w.C)
        T = tri.gdn_chunk_tri_inv_ex(Kd.to(DEV), beta, g, w.C, gate_kind=tri.GATE_PER_CHANNEL,
                                     method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)
        check(T, ref, 1e-5, f"per-channel gate, keys {dt}")


@pytest.mark.parametrize("d_k", [32, 96, 256])
@pytest.mark.parametrize("C", [64, 128])
def test_other_head_dimensions(C, d_k):
    """Scalar and no-gate kinds at head dimensions without a specialised kernel (run-time channel loop)."""
    for k_dtype, gate in (("bf16", si.GATE_SCALAR), ("f32", si.GATE_NONE)):
        inp = si.make_inputs(si.workload(2, B=1, Tlen=3 * C, H=3, d_k=d_k, C=C, k_dtype=k_dtype, gate_kind=gate))
        w = inp["workload"]
        ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], gate, C)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        # (C = 64: one fused kernel per method; C = 128: the whole-matrix methods take the two-launch path)
        for method, op in [(tri.BLOCK_RECURSIVE, tri.BF16), (tri.BLOCK_RECURSIVE, tri.F32), (tri.BLOCK_DIRECT, tri.F32),
                           (tri.BLOCK_DIRECT, tri.F16), (tri.FWD_SUBST, tri.F32), (tri.MIXED, tri.BF16), (tri.MIXED_B32, tri.F16),
                           (tri.NEUMANN, tri.F32), (tri.NEWTON_SCHULZ, tri.BF16), (tri.NEWTON_SCHULZ, tri.F32)]:
            T = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate, method=method, op_dtype=op)
            check(T, ref, TOL[op], f"d_k={d_k} C={C} {k_dtype} {ids((method, op))}", op=op,
                  method=None if method == tri.NEUMANN else method)
        if C == 64:     # the fused kernels take a 16-bit result and the mixed recursion's refinement count
            T16 = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate, method=tri.MIXED, op_dtype=tri.BF16,
                                           out_dtype=torch.bfloat16)
            T32 = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate, method=tri.MIXED, op_dtype=tri.BF16)
            assert torch.equal(T16, T32.bfloat16())
            T0 = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate, method=tri.MIXED, op_dtype=tri.BF16,
                                          flags=tri.flag_mxr_r(0))
            assert not torch.equal(T0, T32), "the refinement count did not reach the kernel"


FP32_KEY_METHODS = [(tri.FWD_SUBST, tri.F32)] + [(m, o) for m in (tri.BLOCK_RECURSIVE, tri.BLOCK_DIRECT, tri.MIXED, tri.MIXED_B32,
                                                                  tri.NEUMANN, tri.NEWTON_SCHULZ) for o in _OPS]


@pytest.mark.parametrize("mo", FP32_KEY_METHODS, ids=ids)
@pytest.mark.parametrize("C", [64, 128])
def test_fp32_keys_with_128_channels(C, mo):
    """Keys stored in fp32 (paper Sec. 4.1: fp32 inputs) at d_k = 128, every method and operand type.  At C = 128 a
    chunk's keys alone are 256 registers per lane: that combination runs the channel-loop kernels (blocked, direct-leaf
    recursion, forward substitution) or the two-launch path (the others), never a kernel with scratch memory."""
    method, op = mo
    inp = si.make_inputs(si.workload(1, B=1, Tlen=3 * C + 17, H=3, C=C, d_k=128, k_dtype="f32"))
    assert inp["K"].dtype == torch.float32
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 0, C)
    n_mat = T_ref.shape[0]
    guard = torch.full((n_mat + 1, C, C), 7.0, device=DEV)
    tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), C, T=guard[:n_mat], method=method, op_dtype=op)
    check(guard[:n_mat], T_ref, TOL[op], f"fp32 keys d_k=128 C={C} {ids(mo)}", op=op, method=method)
    assert bool((guard[n_mat] == 7.0).all()), "wrote past the last matrix"


# The same calls with more matrices than the launch shapes and kernels for few of them take (512).
@pytest.mark.parametrize("mo", FP32_KEY_METHODS, ids=ids)
@pytest.mark.parametrize("gate,d_k,C,k_dtype", [("scalar", 128, 64, "f32"), ("scalar", 96, 64, "bf16"), ("scalar", 160, 32, "f32"), ("scalar", 96, 16, "bf16"),
                                                ("channel", 128, 64, "bf16"), ("channel", 96, 32, "f32"), ("channel", 64, 16, "bf16")])
def test_channel_loops_and_fp32_keys_in_larger_calls(gate, d_k, C, k_dtype, mo):
    method, op = mo
    if C == 16 and method == tri.MIXED_B32:
        pytest.skip("b0 = 32 needs C >= 32")
    w = si.workload(3 if gate == "channel" else 1, B=1, Tlen=173 * C + 7, H=3, C=C, d_k=d_k, k_dtype=k_dtype)
    inp = si.make_inputs(w)
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], w.gate_kind, C)
    n_mat = T_ref.shape[0]
    assert n_mat > 512
    guard = torch.full((n_mat + 1, C, C), 7.0, device=DEV)
    tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), C, T=guard[:n_mat], gate_kind=w.gate_kind, method=method, op_dtype=op)
    check(guard[:n_mat], T_ref, TOL[op], f"{gate} d_k={d_k} C={C} {ids(mo)}", op=op, method=method, key_abs=key_abs_term(inp, w.gate_kind, C))
    assert bool((guard[n_mat] == 7.0).all()), "wrote past the last matrix"


def test_group_counts_that_are_not_multiples_of_eight(cases):
    # 12 (batch, chunk) groups: 8 go through the XCD-aware map, 4 keep the plain order
    inp = si.make_inputs(si.workload(1, B=1, Tlen=768, H=4))
    w = inp["workload"]
    ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], w.gate_kind, w.C)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    for method, op in [(tri.BLOCK_RECURSIVE, tri.F32), (tri.FWD_SUBST, tri.F32), (tri.NEUMANN, tri.F32)]:
        check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, method=method, op_dtype=op), ref, 1e-5, f"12 groups {ids((method, op))}")
    g4 = inp["g"][..., None].expand(-1, -1, -1, w.d_k).contiguous().to(DEV)
    check(tri.gdn_chunk_tri_inv_ex(K, beta, g4, w.C, gate_kind=tri.GATE_PER_CHANNEL, method=tri.BLOCK_DIRECT, op_dtype=tri.F32),
          ref, 1e-5, "12 groups, per-channel kernel")


def test_refinement_step_recovers_digits(cases):
    """One step of iterative refinement (Alg. 6) after the mixed / blocked recursion.  The residual is
    formed with operands rounded to op_dtype like every other product, so the step cannot go below
    that rounding floor: on benign inputs it must stay within the tolerance and within 2.5x of the
    unrefined error; where the unrefined error is far above the floor (the stress recipe, next test)
    it must reduce it (paper Sec. 4.1: it brings the mixed recursion back on par)."""
    for idx in (1, 2):
        c = cases[idx]
        w, inp = c["w"], c["inp"]
        A32 = torch.from_numpy(c["A"].astype(np.float32))
        T_ref = oracle.tri_inv(A32)
        K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
        for method in (tri.MIXED, tri.BLOCK_RECURSIVE):
            for op in (tri.F32, tri.F16, tri.BF16):
                e0 = check(tri.tri_inv_ex(A32.to(DEV), method=method, op_dtype=op), T_ref, TOL[op], "unrefined")
                e1 = check(tri.tri_inv_ex(A32.to(DEV), method=method, op_dtype=op, flags=1), T_ref, TOL[op], "refined")
                f1 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=w.gate_kind, method=method, op_dtype=op, flags=1),
                           c["T"], TOL[op], "refined, fused")
                assert e1 <= 2.5 * e0 + 1e-7 and f1 <= 2.5 * e0 + 1e-7, (idx, method, op, e0, e1, f1)


def test_refinement_step_with_the_per_channel_gate(cases):
    c = cases[3]
    w, inp = c["w"], c["inp"]
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    for method in (tri.MIXED, tri.BLOCK_RECURSIVE):
        for op in (tri.F32, tri.F16, tri.BF16):
            e0 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=1, method=method, op_dtype=op), c["T"], TOL[op], "per-channel",
                       op=op, key_abs=c["key_abs"])
            e1 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=1, method=method, op_dtype=op, flags=1), c["T"], TOL[op],
                       "per-channel, refined", op=op, key_abs=c["key_abs"])
            assert e1 <= 2.5 * e0 + 1e-7, (method, op, e0, e1)


def test_refinement_on_the_stress_blocks():
    # C = 64 blocks of the stress recipe: mixed recursion with bf16 operands, before and after one step
    inp = si.make_inputs(si.workload(4, Tlen=512, H=3, C=64))
    A = oracle.build_A(inp["K"], inp["beta"], None, si.GATE_NONE, 64)
    T_ref = oracle.tri_inv(A)
    A32 = torch.from_numpy(A.astype(np.float32)).to(DEV)
    r0 = tri.flag_mxr_r(0)  # the mixed recursion without its refinement steps
    e0 = check(tri.tri_inv_ex(A32, method=tri.MIXED, op_dtype=tri.BF16, flags=r0), T_ref, 4e-2, "mixed bf16 stress C=64, r = 0")
    e1 = check(tri.tri_inv_ex(A32, method=tri.MIXED, op_dtype=tri.BF16, flags=r0 | 1), T_ref, 2e-2,
               "mixed bf16 stress C=64, r = 0, one step on the whole matrix")
    assert e1 < e0


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_refinement_step_c128(op):
    """Alg. 6 at C = 128 (a second pass over T, in place): inside the tolerance on benign and stress inputs,
    standalone and fused, with a short last chunk; it repairs the mixed recursion run without its own
    refinement of the diagonal blocks on the stress input; against the fp64 statement of the step applied
    to the unrefined GPU result it differs only by the operand rounding."""
    from oracle import methods
    inp = si.make_inputs(si.workload(1, Tlen=128 * 2 + 50, H=3, C=128))
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 0, 128)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    for method in (tri.BLOCK_RECURSIVE, tri.MIXED):
        check(tri.gdn_chunk_tri_inv_ex(K, beta, g, 128, method=method, op_dtype=op, flags=1), T_ref, TOL[op],
              f"refined C=128 fused {tri.METHOD_NAMES[method]}")
    st = si.make_inputs(si.workload(4, Tlen=512, H=3))
    A = oracle.build_A(st["K"], st["beta"], None, 2, 128)
    A32 = torch.from_numpy(A.astype(np.float32))
    T32 = oracle.tri_inv(A32)
    r0 = tri.flag_mxr_r(0)
    Y = tri.tri_inv_ex(A32.to(DEV), method=tri.MIXED, op_dtype=op, flags=r0)
    e0 = check(Y, T32, 2e-1, "mixed r=0 stress C=128")
    X = tri.tri_inv_ex(A32.to(DEV), method=tri.MIXED, op_dtype=op, flags=r0 | 1)
    e1 = check(X, T32, TOL[op], "mixed r=0 stress C=128 + whole-matrix step")
    assert e1 <= e0
    Kd, bd = st["K"].to(DEV), st["beta"].to(DEV)
    Xf = tri.gdn_chunk_tri_inv_ex(Kd, bd, None, 128, gate_kind=tri.GATE_NONE, method=tri.MIXED, op_dtype=op, flags=r0 | 1)
    check(Xf, oracle.tri_inv(A), TOL[op], "mixed r=0 stress C=128 + step, fused")
    # the step itself: fp64 statement of Alg. 6 applied to the unrefined GPU result
    Yh = Y.cpu().numpy().astype(np.float64)
    want = np.stack([methods.ir(Yh[m], A32[m].numpy().astype(np.float64)) for m in range(4)])
    got = X.cpu().numpy().astype(np.float64)[:4]
    rel = np.linalg.norm(got - want, axis=(1, 2)) / np.linalg.norm(want, axis=(1, 2))
    assert rel.max() <= {tri.F32: 1e-5, tri.F16: 5e-3, tri.BF16: 2e-2}[op], rel


def test_mixed_recursion_refines_its_diagonal_blocks():
    """Paper Alg. 2 / Sec. 4.1: without refinement the mixed recursion loses digits on the stress input;
    one step on the 16 x 16 blocks (the default) brings it to the accuracy of the blocked recursion."""
    inp = si.make_inputs(si.workload(4, Tlen=2048, H=4))
    T_ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], None, si.GATE_NONE, 128)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    err = {}
    for r in (0, 1, 2):
        T = tri.gdn_chunk_tri_inv_ex(K, beta, None, 128, gate_kind=tri.GATE_NONE, method=tri.MIXED, op_dtype=tri.BF16,
                                     flags=tri.flag_mxr_r(r))
        err[r] = check(T, T_ref, 2e-2 if r else 2e-1, f"mixed bf16 stress C=128 r={r}")
    T = tri.gdn_chunk_tri_inv_ex(K, beta, None, 128, gate_kind=tri.GATE_NONE, method=tri.MIXED, op_dtype=tri.BF16)
    assert check(T, T_ref, 2e-2, "mixed bf16 stress C=128 default") == err[1]
    e_block = check(tri.gdn_chunk_tri_inv_ex(K, beta, None, 128, gate_kind=tri.GATE_NONE, method=tri.BLOCK_RECURSIVE,
                                             op_dtype=tri.BF16), T_ref, 2e-2, "block bf16 stress C=128")
    assert err[1] < err[0] and err[1] <= 1.5 * e_block


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_newton_schulz(cases, op):
    """Alg. 3 with X0 = I / C: 12 iterations (the count the paper finds sufficient at C = 64) reach the
    tolerance on every C = 64 recipe, standalone and fused, including 64 x 64 blocks of the stress recipe."""
    for idx in (0, 1, 2, 3):
        c = cases[idx]
        w, inp = c["w"], c["inp"]
        A32 = torch.from_numpy(c["A"].astype(np.float32))
        check(tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=op), oracle.tri_inv(A32), TOL[op], f"NS cfg{idx}", op=op,
              method=tri.NEWTON_SCHULZ)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        Tf = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, w.C, gate_kind=w.gate_kind,
                                      method=tri.NEWTON_SCHULZ, op_dtype=op)
        check(Tf, c["T"], TOL[op], f"NS fused cfg{idx}", op=op, key_abs=c["key_abs"], method=tri.NEWTON_SCHULZ)
    inp = si.make_inputs(si.workload(4, Tlen=512, H=3, C=64))
    A = oracle.build_A(inp["K"], inp["beta"], None, si.GATE_NONE, 64)
    A32 = torch.from_numpy(A.astype(np.float32))
    check(tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=op), oracle.tri_inv(A32), TOL[op], "NS stress blocks", op=op,
          method=tri.NEWTON_SCHULZ)


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_newton_schulz_c128(op, capsys):
    """Alg. 3 at C = 128 (four wavefronts per matrix, X and Y in LDS): 14 = 2 log2 C iterations reach the
    tolerance on benign inputs, standalone, fused (scalar gate and none) and with a short last chunk; the
    iteration count flag is honoured; the stress workload is reported."""
    inp = si.make_inputs(si.workload(1, Tlen=128 * 3 + 40, H=3, C=128))
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 0, 128)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    check(tri.gdn_chunk_tri_inv_ex(K, beta, g, 128, method=tri.NEWTON_SCHULZ, op_dtype=op), T_ref, TOL[op], "NS C=128 fused", op=op,
          method=tri.NEWTON_SCHULZ)
    T_ref2 = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], None, 2, 128)
    check(tri.gdn_chunk_tri_inv_ex(K, beta, None, 128, gate_kind=tri.GATE_NONE, method=tri.NEWTON_SCHULZ, op_dtype=op), T_ref2,
          TOL[op], "NS C=128 fused, no gate")
    A = oracle.build_A_ragged(inp["K"], inp["beta"], inp["g"], 0, 128)
    A32 = torch.from_numpy(A.astype(np.float32))
    T32 = oracle.tri_inv(A32)
    check(tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=op), T32, TOL[op], "NS C=128 standalone", op=op,
          method=tri.NEWTON_SCHULZ)
    few = tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=op, flags=tri.flag_iters(5)).cpu().numpy()
    e_few = metrics.forward_errors(T32, few.astype(np.float64))["rel_fro"].max()
    assert e_few > 1e-1, "five iterations cannot have converged from X0 = I / 128"
    if op == tri.F32:
        from oracle import methods
        low = np.tril(np.ones((128, 128), dtype=bool), -1)
        want = np.stack([methods.ns(A32[i].numpy().astype(np.float64), m=5) for i in range(3)])
        assert np.allclose(few[:3][:, low], want[:, low], rtol=2e-4, atol=2e-6)
    # stress workload: reported, not asserted (X0 = I / C need not converge in 2 log2 C steps when ||A|| is large)
    st = si.make_inputs(si.workload(4, Tlen=512, H=3))
    Ts = oracle.gdn_chunk_tri_inv(st["K"], st["beta"], None, 2, 128)
    Tg = tri.gdn_chunk_tri_inv_ex(st["K"].to(DEV), st["beta"].to(DEV), None, 128, gate_kind=tri.GATE_NONE,
                                  method=tri.NEWTON_SCHULZ, op_dtype=op)
    torch.cuda.synchronize()
    e = metrics.forward_errors(Ts, Tg.cpu().numpy().astype(np.float64))["rel_fro"]
    with capsys.disabled():
        print(f"\nnewton_schulz {tri.DTYPE_NAMES[op]} on stress C=128, 14 iterations: rel_fro max {np.nanmax(e):.3e}")


def test_newton_schulz_iteration_count(cases):
    """Fewer iterations leave the iteration unconverged (paper Sec. 4.2: 6 iterations are markedly worse than
    12); the error after m iterations follows the fp64 statement of Alg. 3 in exact arithmetic."""
    from oracle import methods

    A32 = torch.from_numpy(cases[1]["A"][:8].astype(np.float32))
    T_ref = oracle.tri_inv(A32)
    errs = {}
    for m in (4, 8, 12, 16):
        T = tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=tri.F32, flags=tri.flag_iters(m)).cpu().numpy()
        errs[m] = metrics.forward_errors(T_ref, T.astype(np.float64))["rel_fro"].max()
        low = np.tril(np.ones((64, 64), dtype=bool), -1)
        want = np.stack([methods.ns(A32[i].numpy().astype(np.float64), m=m) for i in range(len(A32))])
        # the strictly-lower part of the unconverged iterate itself matches (diagonal is forced to 1 on store)
        assert np.allclose(T[:, low], want[:, low], rtol=2e-4, atol=2e-6), m
    assert errs[4] > 1e-1 and errs[8] > 10 * errs[12] and errs[12] <= 1e-5 and errs[16] <= 1e-5, errs
    default = tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=tri.F32)
    twelve = tri.tri_inv_ex(A32.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=tri.F32, flags=tri.flag_iters(12))
    torch.cuda.synchronize()
    assert torch.equal(default, twelve)


def test_unbuilt_combinations_report_unsupported(cases):
    c = cases[1]
    w, inp = c["w"], c["inp"]
    # head dimensions other than 64 / 128: the refinement flag is not built; at C = 128 the whole-matrix methods take the
    # composed path, which needs an fp32 result
    K96 = torch.zeros(1, 128, 2, 96, dtype=torch.bfloat16, device=DEV)
    b = torch.zeros(1, 128, 2, device=DEV)
    for C, kw in ((128, dict(out_dtype=torch.bfloat16)), (128, dict(flags=tri.FLAG_REFINE1)), (64, dict(flags=tri.FLAG_REFINE1))):
        with pytest.raises(tri.TriInvError) as e:
            tri.gdn_chunk_tri_inv_ex(K96, b, b, C, method=tri.MIXED, **kw)
        assert e.value.status == -9
    for kw in (dict(method=tri.BLOCK_RECURSIVE, flags=0x80), dict(method=tri.BLOCK_RECURSIVE, flags=8), dict(method=tri.FWD_SUBST, flags=1)):
        with pytest.raises(tri.TriInvError) as e:
            tri.tri_inv_ex(torch.zeros(2, 64, 64, device=DEV), op_dtype=tri.F32, **kw)
        assert e.value.status == -9
    with pytest.raises(tri.TriInvError) as e:   # refinement at C = 128 is a second pass over an fp32 result
        tri.tri_inv_ex(torch.zeros(2, 128, 128, device=DEV), method=tri.MIXED, op_dtype=tri.F32, flags=1, out_dtype=torch.bfloat16)
    assert e.value.status == -9
    # per-channel gate + refinement step at C = 128: a second pass over an fp32 result as well
    K = torch.zeros(1, 128, 2, 128, dtype=torch.bfloat16, device=DEV)
    g4 = torch.zeros(1, 128, 2, 128, device=DEV)
    with pytest.raises(tri.TriInvError) as e:
        tri.gdn_chunk_tri_inv_ex(K, torch.zeros(1, 128, 2, device=DEV), g4, 128, gate_kind=tri.GATE_PER_CHANNEL, method=tri.MIXED,
                                 flags=tri.FLAG_REFINE1, out_dtype=torch.bfloat16)
    assert e.value.status == -9


@pytest.mark.parametrize("k_dtype,d_k", [("bf16", 128), ("f32", 64), ("f16", 96)])
def test_per_channel_gate_c128_on_four_wavefronts(k_dtype, d_k):
    """Per-channel gate at C = 128 with the methods that run one matrix per workgroup of four wavefronts (the waves gate and
    exchange the keys 32 channels at a time): Newton-Schulz, the Neumann product, and the refinement pass behind any method.
    Short last chunk included; every operand type; a 16-bit result where the method writes it itself."""
    C = 128
    inp = si.make_inputs(si.workload(3, B=1, Tlen=2 * C + 41, H=3, C=C, d_k=d_k, k_dtype="f32" if k_dtype == "f16" else k_dtype))
    if k_dtype == "f16":
        inp["K"] = inp["K"].to(torch.float16)
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 1, C)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    n_mat = T_ref.shape[0]
    for op in _OPS:
        ka = None if op == tri.F32 else key_abs_term(inp, 1, C)
        for method in (tri.NEWTON_SCHULZ, tri.NEUMANN):
            guard = torch.full((n_mat + 1, C, C), 7.0, device=DEV)
            tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=guard[:n_mat], gate_kind=tri.GATE_PER_CHANNEL, method=method, op_dtype=op)
            check(guard[:n_mat], T_ref, TOL[op], f"per-channel C=128 {k_dtype} d_k={d_k} {ids((method, op))}", op=op, key_abs=ka,
                  method=method if method == tri.NEWTON_SCHULZ else None)
            assert bool((guard[n_mat] == 7.0).all()), "wrote past the last matrix"
        T16 = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, method=tri.NEWTON_SCHULZ, op_dtype=op,
                                       out_dtype=torch.bfloat16)
        T32 = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, method=tri.NEWTON_SCHULZ, op_dtype=op)
        assert torch.equal(T16, T32.bfloat16())
        floor = {tri.F32: 1e-6, tri.F16: 3e-4, tri.BF16: 2e-3}[op]
        for method in (tri.BLOCK_RECURSIVE, tri.MIXED, tri.NEWTON_SCHULZ, tri.NEUMANN):
            what = f"per-channel C=128 {k_dtype} d_k={d_k} {ids((method, op))}"
            e0 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, method=method, op_dtype=op), T_ref, TOL[op],
                       what, op=op, key_abs=ka, method=method if method != tri.NEUMANN else None)
            e1 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, method=method, op_dtype=op,
                                                flags=tri.FLAG_REFINE1), T_ref, TOL[op], what + " + refine", op=op, key_abs=ka,
                       method=method if method != tri.NEUMANN else None)
            assert e1 <= max(1.5 * e0, floor), (what, e0, e1)


# ------------------------------------------------------------------ full-size workloads, sampled
def _sample(n_mat, k=48, seed=0):
    rng = np.random.default_rng(seed)
    return np.unique(np.concatenate([[0, 1, n_mat - 1], rng.integers(0, n_mat, size=k)])).tolist()


# The precision matrix at full size (paper Sec. 4.1 protocol: every method in fp32, fp16 and bf16 operand modes):
# configs[2] x {forward substitution, blocked, direct-leaf, mixed recursion, Neumann product} and configs[4] (the stress
# workload) x {forward substitution, blocked, direct-leaf, mixed (b0 = 16 and 32) recursion, Newton-Schulz}, every operand
# type; configs[1] and configs[3] with the methods their kernels differ in.  The Neumann product on configs[4] is run and
# its error printed, not asserted (the paper predicts its failure there, Sec. 3.2 / 4.1).
FULL_MATRIX = ([(1, (tri.BLOCK_RECURSIVE, tri.BF16)), (1, (tri.FWD_SUBST, tri.F32))]
               + [(2, (tri.FWD_SUBST, tri.F32))]
               + [(2, (m, o)) for m in (tri.BLOCK_RECURSIVE, tri.BLOCK_DIRECT, tri.MIXED, tri.NEUMANN) for o in _OPS]
               + [(3, (tri.FWD_SUBST, tri.F32)), (3, (tri.BLOCK_DIRECT, tri.F32))]
               + [(3, (tri.BLOCK_RECURSIVE, o)) for o in _OPS]
               + [(4, (tri.FWD_SUBST, tri.F32))]
               + [(4, (m, o)) for m in (tri.BLOCK_RECURSIVE, tri.BLOCK_DIRECT, tri.MIXED, tri.MIXED_B32, tri.NEWTON_SCHULZ, tri.NEUMANN)
                  for o in _OPS])

_full_cache = {}


def full_size(idx):
    """Inputs of one full-size workload on the device, the sampled matrices and the oracle's results for them; one workload
    is kept at a time (configs[3] alone holds 1.6 GB of inputs)."""
    if _full_cache.get("idx") != idx:
        _full_cache.clear()
        w = si.WORKLOADS[idx]
        inp = si.make_inputs(w)
        sel = _sample(w.n_mat)
        T_ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], w.gate_kind, w.C, sel=sel)
        key_abs = None
        if w.gate_kind == tri.GATE_PER_CHANNEL:
            key_abs = oracle.build_A(inp["K"].abs(), inp["beta"], inp["g"], w.gate_kind, w.C, sel=sel)
        _full_cache.update(idx=idx, w=w, sel=sel, T_ref=T_ref, key_abs=key_abs, K=inp["K"].to(DEV), beta=inp["beta"].to(DEV),
                           g=None if inp["g"] is None else inp["g"].to(DEV))
    return _full_cache


@pytest.mark.parametrize("idx,mo", FULL_MATRIX, ids=lambda v: ids(v) if isinstance(v, tuple) else f"cfg{v}")
def test_full_size_workload_sampled(idx, mo, capsys):
    """The launch configuration the benchmark times, at the workload's full size; the oracle
    recomputes a sample of the output matrices one by one, and the structural property is
    checked on every matrix."""
    method, op = mo
    f = full_size(idx)
    w, sel = f["w"], f["sel"]
    T = tri.gdn_chunk_tri_inv_ex(f["K"], f["beta"], f["g"], w.C, gate_kind=w.gate_kind, method=method, op_dtype=op)
    torch.cuda.synchronize()
    diag = torch.diagonal(T, dim1=1, dim2=2)
    assert bool((diag == 1).all())
    above = torch.triu(T, 1) != 0
    if bool(above.any()):  # say where: a structural failure at this size is otherwise hard to trace
        at = above.nonzero()
        first = [(int(m), int(r), int(c), float(T[m, r, c])) for m, r, c in at[:8].cpu().numpy()]
        pytest.fail(f"full cfg{idx} {ids(mo)}: {len(at)} non-zeros above the diagonal in "
                    f"{len(torch.unique(at[:, 0]))} matrices, first (matrix, row, column, value): {first}")
    if idx == 4 and method == tri.NEUMANN:
        Ts = T[sel].cpu().numpy().astype(np.float64)
        with np.errstate(invalid="ignore"):
            e = metrics.forward_errors(f["T_ref"], Ts)["rel_fro"]
        bad = int((~np.isfinite(e)).sum())
        with capsys.disabled():
            print(f"\nneumann {tri.DTYPE_NAMES[op]} on configs[4] at full size: rel_fro max "
                  f"{np.nanmax(e) if bad < len(e) else float('nan'):.3e}, non-finite matrices {bad}/{len(e)} (reported, not asserted)")
        return
    check(T[sel], f["T_ref"], TOL[op], f"full cfg{idx} {ids(mo)}", op=op, key_abs=f["key_abs"], method=method)
    # every matrix: entries bounded by one (Cor. 2.1 and its source)
    assert float(T.abs().max()) <= 1.0 + (1e-4 if op == tri.F32 else 5e-2)


@pytest.mark.parametrize("idx", [2, 3, 4])
def test_full_size_workload_every_matrix_by_properties(idx):
    """Properties that hold at any size, checked on EVERY matrix of the full-size launch: the residual
    ||(I + A) T - I||_F (A written by gdn_chunk_build_A, which its own test pins to the oracle; products in fp64 on
    the device) and, for the scalar gate, the similarity T_gated = T_ungated * exp(g_i - g_j) (follows from
    A_gated = Gamma A Gamma^-1, paper Table 1)."""
    w = si.WORKLOADS[idx]
    inp = si.make_inputs(w)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    C = w.C
    A = tri.gdn_chunk_build_A(K, beta, g, C, gate_kind=w.gate_kind, op_dtype=tri.F32)
    eye = torch.eye(C, device=DEV, dtype=torch.float64)
    for method, op, tol in [(tri.BLOCK_DIRECT, tri.F32, 2e-6), (tri.BLOCK_RECURSIVE, tri.BF16, 2e-3)]:
        T = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=w.gate_kind, method=method, op_dtype=op)
        worst = 0.0
        for m0 in range(0, w.n_mat, 4096):        # in slabs, fp64 on the device
            Ts = T[m0:m0 + 4096].double()
            M = A[m0:m0 + 4096].double() + eye
            R = torch.bmm(M, Ts) - eye
            nrm = torch.linalg.matrix_norm(R) / (torch.linalg.matrix_norm(M) * torch.linalg.matrix_norm(Ts))
            assert bool(torch.isfinite(nrm).all())
            worst = max(worst, float(nrm.max()))
        assert worst <= tol, (idx, tri.METHOD_NAMES[method], worst)
    if w.gate_kind == tri.GATE_SCALAR:
        Tg = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_SCALAR, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
        Tu = tri.gdn_chunk_tri_inv_ex(K, beta, None, C, gate_kind=tri.GATE_NONE, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
        gg = g.reshape(w.B, w.Tlen // C, C, w.H).permute(0, 1, 3, 2).reshape(-1, C).double()
        sim = Tu.double() * torch.tril(torch.exp(gg[:, :, None] - gg[:, None, :]))
        assert float((Tg.double() - sim).abs().max()) <= 2e-6


def test_neumann_on_the_stress_input_is_reported_not_asserted(cases, capsys):
    """C = 64 sub-blocks of the stress recipe: large ||A||, the repeated squaring overflows or
    cancels (paper Sec. 3.2, Sec. 4.1).  The library must return whatever the algorithm yields."""
    inp = si.make_inputs(si.workload(4, Tlen=512, H=3, C=64))
    w = inp["workload"]
    A = oracle.build_A(inp["K"], inp["beta"], None, si.GATE_NONE, 64)
    T_ref = oracle.tri_inv(A)
    A32 = torch.from_numpy(A.astype(np.float32)).to(DEV)
    lines = []
    for op in (tri.F32, tri.F16, tri.BF16):
        T = tri.tri_inv_ex(A32, method=tri.NEUMANN, op_dtype=op).cpu().numpy().astype(np.float64)
        e = metrics.forward_errors(T_ref, T)["rel_fro"]
        lines.append(f"neumann {tri.DTYPE_NAMES[op]} on stress C=64: rel_fro max {np.nanmax(e):.3e}, "
                     f"non-finite matrices {int((~np.isfinite(e)).sum())}/{len(e)}")
        Tb = tri.tri_inv_ex(A32, method=tri.BLOCK_RECURSIVE, op_dtype=op)
        check(Tb, T_ref, TOL[op], "blocked recursion on the same input")
    with capsys.disabled():
        print("\n" + "\n".join(lines))


def test_neumann_c128_on_the_stress_input_is_reported(capsys):
    lines = []
    inp = si.make_inputs(si.workload(4, Tlen=512, H=3))
    A = oracle.build_A(inp["K"], inp["beta"], None, si.GATE_NONE, 128)
    T_ref = oracle.tri_inv(A)
    A32 = torch.from_numpy(A.astype(np.float32)).to(DEV)
    for op in (tri.F32, tri.F16, tri.BF16):
        T = tri.tri_inv_ex(A32, method=tri.NEUMANN, op_dtype=op).cpu().numpy().astype(np.float64)
        Tf = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), None, 128, gate_kind=tri.GATE_NONE,
                                      method=tri.NEUMANN, op_dtype=op).cpu().numpy().astype(np.float64)
        for tag, X in (("standalone", T), ("fused", Tf)):
            e = metrics.forward_errors(T_ref, X)["rel_fro"]
            lines.append(f"neumann {tri.DTYPE_NAMES[op]} on stress C=128 {tag}: rel_fro max {np.nanmax(e):.3e}, "
                         f"non-finite matrices {int((~np.isfinite(e)).sum())}/{len(e)}")
    with capsys.disabled():
        print("\n" + "\n".join(lines))


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_neumann_c128_on_benign_input(op):
    """The C = 128 Neumann kernel itself is held to the tolerance where the algorithm is
    accurate: small ||A|| (gated, strongly decayed keys)."""
    A = si.random_strict_lower(9, 128, 0.02, seed=11, garbage_upper=True)
    T = tri.tri_inv_ex(A.to(DEV), method=tri.NEUMANN, op_dtype=op)
    check(T, oracle.tri_inv(A), TOL[op], f"neumann C=128 benign {tri.DTYPE_NAMES[op]}")
    inp = si.make_inputs(si.workload(2, B=1, Tlen=256, H=3, C=128))
    w = inp["workload"]
    ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], w.gate_kind, 128)
    Tf = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), 128, gate_kind=w.gate_kind,
                                  method=tri.NEUMANN, op_dtype=op)
    check(Tf, ref, TOL[op], f"neumann C=128 fused benign {tri.DTYPE_NAMES[op]}")


# ------------------------------------------------------------------ short last chunks, packed sequences
RAGGED_METHODS = [(tri.FWD_SUBST, tri.F32), (tri.BLOCK_RECURSIVE, tri.BF16), (tri.BLOCK_DIRECT, tri.F32), (tri.MIXED, tri.F16),
                  (tri.NEUMANN, tri.F32)]


@pytest.mark.parametrize("mo", RAGGED_METHODS, ids=ids)
@pytest.mark.parametrize("gate_kind", [0, 1, 2])
@pytest.mark.parametrize("C,Tlen", [(64, 1), (64, 63), (64, 65), (64, 200), (128, 127), (128, 300)])
def test_sequence_lengths_that_are_not_multiples_of_the_chunk(C, Tlen, gate_kind, mo):
    method, op = mo
    idx = {0: 1, 1: 3, 2: 4}[gate_kind]
    inp = si.make_inputs(si.workload(idx, B=2, Tlen=Tlen, H=3, C=C, d_k=128, k_dtype="bf16"))
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    n_mat = 2 * ((Tlen + C - 1) // C) * 3
    guard = torch.full((n_mat + 1, C, C), 7.0, device=DEV)           # one matrix of slack behind the output
    tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=guard[:n_mat], gate_kind=gate_kind, method=method, op_dtype=op)
    torch.cuda.synchronize()
    assert bool((guard[n_mat] == 7.0).all()), "wrote past the last matrix"
    tol = TOL[op]
    if idx == 4 and method == tri.NEUMANN:
        return  # the Neumann product on the stress recipe is reported elsewhere, not asserted
    check(guard[:n_mat], T_ref, tol, f"ragged C={C} Tlen={Tlen} gate={gate_kind} {ids(mo)}", op=op, key_abs=key_abs_term(inp, gate_kind, C))


@pytest.mark.parametrize("d_k", [96, 128])
@pytest.mark.parametrize("gate_kind", [0, 1, 2])
@pytest.mark.parametrize("C", [64, 128])
def test_packed_variable_length_sequences(C, gate_kind, d_k):
    H = 3
    seqlens = [C, 1, 0, 2 * C + 5, C - 1, 3 * C, 0, 17]
    total = sum(seqlens)
    idx = {0: 1, 1: 3, 2: 4}[gate_kind]
    inp = si.make_inputs(si.workload(idx, B=1, Tlen=total, H=H, C=C, d_k=d_k, k_dtype="bf16"))
    K, beta = inp["K"][0].contiguous(), inp["beta"][0].contiguous()
    g = None
    if gate_kind != 2:
        # chunk-local cumulative log-decay, restarted at every chunk of every sequence
        gen = torch.Generator().manual_seed(11)
        shape = (total, H) if gate_kind == 0 else (total, H, d_k)
        rate = -0.05 * torch.nn.functional.softplus(torch.randn(*shape, generator=gen))
        g, t0 = torch.zeros(shape), 0
        for n in seqlens:
            for c0 in range(0, n, C):
                m = min(C, n - c0)
                g[t0 + c0:t0 + c0 + m] = torch.cumsum(rate[t0 + c0:t0 + c0 + m], 0)
            t0 += n
    T_ref = oracle.gdn_chunk_tri_inv_varlen(K, beta, g, seqlens, gate_kind, C)
    for method, op in [(tri.BLOCK_RECURSIVE, tri.BF16), (tri.FWD_SUBST, tri.F32), (tri.BLOCK_DIRECT, tri.F32)]:
        T = tri.gdn_chunk_tri_inv_varlen(K.to(DEV), beta.to(DEV), None if g is None else g.to(DEV), seqlens, C,
                                         gate_kind=gate_kind, method=method, op_dtype=op)
        assert T.shape[0] == T_ref.shape[0]
        check(T, T_ref, TOL[op], f"varlen C={C} gate={gate_kind} d_k={d_k} {ids((method, op))}", op=op,
              key_abs=SKIP if gate_kind == 1 and op != tri.F32 else None)


def test_packed_sequences_with_no_tokens_are_a_no_op():
    K = torch.zeros((0, 2, 128), dtype=torch.bfloat16, device=DEV)
    beta = torch.zeros((0, 2), device=DEV)
    T = tri.gdn_chunk_tri_inv_varlen(K, beta, None, [0, 0], 64, gate_kind=tri.GATE_NONE)
    assert T.shape == (0, 64, 64)


# ------------------------------------------------------------------ the small chunk sizes, C = 16 and 32
SMALL_C_METHODS = [(tri.FWD_SUBST, tri.F32)] + [(m, o) for m in (tri.BLOCK_RECURSIVE, tri.BLOCK_DIRECT, tri.MIXED, tri.NEUMANN,
                                                               tri.NEWTON_SCHULZ) for o in (tri.F32, tri.F16, tri.BF16)]


@pytest.mark.parametrize("mo", SMALL_C_METHODS, ids=ids)
@pytest.mark.parametrize("C", [16, 32])
def test_small_chunk_sizes_standalone(C, mo):
    method, op = mo
    A = si.random_strict_lower(37, C, 0.15, seed=3)
    T_ref = oracle.tri_inv(A)
    T = tri.tri_inv_ex(A.to(DEV), method=method, op_dtype=op)
    check(T, T_ref, TOL[op], f"standalone C={C} {ids(mo)}", op=op, method=method)


@pytest.mark.parametrize("mo", SMALL_C_METHODS, ids=ids)
@pytest.mark.parametrize("gate_kind", [0, 1, 2])
@pytest.mark.parametrize("C", [16, 32])
def test_small_chunk_sizes_fused(C, gate_kind, mo):
    method, op = mo
    idx = {0: 1, 1: 3, 2: 2}[gate_kind]
    inp = si.make_inputs(si.workload(idx, B=2, Tlen=5 * C + 3, H=5, C=C, d_k=128, k_dtype="bf16", gate_kind=gate_kind))
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    T = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate_kind, method=method, op_dtype=op)
    check(T, T_ref, TOL[op], f"fused C={C} gate={gate_kind} {ids(mo)}", op=op, key_abs=key_abs_term(inp, gate_kind, C), method=method)


@pytest.mark.parametrize("C", [16, 32])
def test_small_chunk_sizes_refinement_and_other_head_dimensions(C):
    inp = si.make_inputs(si.workload(1, B=1, Tlen=8 * C, H=3, C=C, d_k=96, k_dtype="f32"))
    T_ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], 0, C)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    T = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, method=tri.BLOCK_RECURSIVE, op_dtype=tri.F32)   # channel-loop kernel
    check(T, T_ref, 1e-5, f"C={C} d_k=96")
    inp = si.make_inputs(si.workload(1, B=1, Tlen=8 * C, H=4, C=C, d_k=64, k_dtype="bf16"))
    T_ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], 0, C)
    T = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), C, method=tri.MIXED, op_dtype=tri.BF16,
                                 flags=tri.FLAG_REFINE1)
    check(T, T_ref, 2e-2, f"C={C} mixed + refinement")


# ------------------------------------------------------------------ 16-bit result
OUT_U = {torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}   # unit roundoff of the result's type


@pytest.mark.parametrize("out", [torch.float16, torch.bfloat16], ids=["out_f16", "out_bf16"])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_sixteen_bit_result(C, out):
    """TRIINV_FLAG_OUT_*: the fp32 result rounded to nearest even on the way out; bit-exact against the
    fp32-output run of the same method rounded by torch; inside tolerance + one rounding against the oracle."""
    inp = si.make_inputs(si.workload(1, B=2, Tlen=3 * C + 7, H=5, C=C))
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 0, C)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    for method, op in [(tri.BLOCK_RECURSIVE, tri.BF16), (tri.MIXED, tri.F16), (tri.BLOCK_DIRECT, tri.F32), (tri.NEUMANN, tri.F32),
                       (tri.NEWTON_SCHULZ, tri.F32), (tri.FWD_SUBST, tri.F32)]:
        n_mat = T_ref.shape[0]
        guard = torch.full((n_mat + 1, C, C), 7.0, device=DEV, dtype=out)
        tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=guard[:n_mat], method=method, op_dtype=op)
        T32 = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, method=method, op_dtype=op)
        torch.cuda.synchronize()
        assert bool((guard[n_mat] == 7.0).all()), "wrote past the last matrix"
        assert torch.equal(guard[:n_mat], T32.to(out)), f"C={C} {ids((method, op))}: not the rounded fp32 result"
        check(guard[:n_mat].float(), T_ref, TOL[op] + OUT_U[out], f"16-bit out C={C} {ids((method, op))}")
    # standalone entry point and the per-channel gate
    A32 = torch.from_numpy(oracle.build_A_ragged(inp["K"], inp["beta"], inp["g"], 0, C).astype(np.float32)).to(DEV)
    for method in (tri.BLOCK_RECURSIVE, tri.FWD_SUBST):
        Ts = tri.tri_inv_ex(A32, method=method, op_dtype=tri.F32, out_dtype=out)
        assert Ts.dtype == out
        check(Ts.float(), oracle.tri_inv(A32.cpu()), 1e-5 + OUT_U[out], f"16-bit out standalone {tri.METHOD_NAMES[method]} C={C}")
    inp3 = si.make_inputs(si.workload(3, B=1, Tlen=2 * C + 5, H=3, C=C))
    T3 = tri.gdn_chunk_tri_inv_ex(inp3["K"].to(DEV), inp3["beta"].to(DEV), inp3["g"].to(DEV), C, gate_kind=tri.GATE_PER_CHANNEL,
                                  out_dtype=out)
    check(T3.float(), oracle.gdn_chunk_tri_inv_ragged(inp3["K"], inp3["beta"], inp3["g"], 1, C), 2e-2 + OUT_U[out],
          f"16-bit out per-channel C={C}")


def test_sixteen_bit_result_argument_errors():
    A = torch.zeros(2, 64, 64, device=DEV)
    with pytest.raises(tri.TriInvError) as e:     # the shuffle variant of forward substitution: fp32 result only
        tri.tri_inv_ex(A, method=tri.FWD_SUBST, out_dtype=torch.bfloat16, flags=tri.FLAG_FWD_SHUFFLE)
    assert e.value.status == -9
    with pytest.raises(tri.TriInvError) as e:     # both output types at once
        tri.lib()  # loaded
        T = torch.zeros(2, 64, 64, device=DEV)
        st = tri.lib().tri_inv_ex(A.data_ptr(), T.data_ptr(), 2, 64, 0, 1, 0, None, 0x2 | 0x4)
        raise tri.TriInvError(st, "both")
    assert e.value.status == -3


# ------------------------------------------------------------------ every Newton-Schulz iterate
@pytest.mark.parametrize("op", _OPS, ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_newton_schulz_iterates(C, op):
    """The m-th iterate, converged or not, against its closed form X_m = T (I - R0^(2^m)) in 64 bits (strictly lower part: the
    stored diagonal is exactly 1): m = 1 is the start that is written down directly, m = 2 the first full iteration.  The
    entries of A span eight orders of magnitude.  With fp32 operands every row is held to 5e-7 of its own norm (a norm over the matrix
    would be that of its large rows): products of fp32 accuracy give at most 2e-7; in an emulation of the split
    products, leaving out the third part of one operand gives 3.5e-6 and more from m = 2 on, of both 4.8e-6, and keeping three of
    the six products 4.8e-6 (C = 16, 32, 64)."""
    from oracle import methods
    A = si.random_strict_lower(5, C, 0.15, seed=23)
    A[1] *= 1e-4
    A[2, C // 2:] *= 1e-6
    for m in (1, 2, 3, 9):
        T = tri.tri_inv_ex(A.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=op, flags=tri.flag_iters(m))
        got = np.tril(T.cpu().numpy().astype(np.float64), -1)
        for k in range(A.shape[0]):
            want = np.tril(methods.newton_schulz_closed_form(np.tril(A[k].numpy().astype(np.float64), -1), m), -1)
            err = np.linalg.norm(got[k] - want) / np.linalg.norm(want)
            if op == tri.F32:
                rows = np.linalg.norm(got[k] - want, axis=1)[1:] / np.linalg.norm(want, axis=1)[1:]
                assert rows.max() <= 5e-7, (C, m, k, int(rows.argmax()) + 1, rows.max())
            # fp16: the start (I + A) / C^2 times entries of 1e-5 lies among the subnormal operands
            assert err <= (TOL[op] if op != tri.F16 or k != 1 else 1e-1), (C, m, k, err)


@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_newton_schulz_takes_entries_beyond_the_largest_bf16(C):
    """fp32 operands: entries between the largest bf16 (3.39e38) and the largest fp32 number, whose leading part alone would round to
    infinity.  A single one per matrix, the first two iterates (X0 A X0 = A / C^2, and 4 (1 - 3 / (2 C)) of it; later ones
    approach -A and overflow in 2 X)."""
    from oracle import methods
    pos = [(i, j) for i in (1, 9, C - 1) for j in (0, i - 1, i // 2)]
    A = torch.zeros(len(pos), C, C)
    for m, (i, j) in enumerate(pos):
        A[m, i, j] = (3.4028234e38, -3.395e38, 3.3953e38)[m % 3]
    for iters in (1, 2):
        T = tri.tri_inv_ex(A.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=tri.F32, flags=tri.flag_iters(iters)).cpu().double().numpy()
        for m, (i, j) in enumerate(pos):
            want = methods.newton_schulz_closed_form(A[m].double().numpy(), iters)[i, j]
            assert abs(T[m, i, j] / want - 1) < 1e-6, (C, iters, i, j, T[m, i, j], want)
            T[m, i, j] = 0
        assert np.array_equal(T, np.broadcast_to(np.eye(C), T.shape))


@pytest.mark.parametrize("n_mat", [1, 257])  # by eight wavefronts, by four
def test_newton_schulz_takes_iterates_beyond_the_largest_bf16(n_mat):
    """C = 128, fp32 operands: Y of the second iteration has one entry between the largest bf16 and the largest fp32 number,
    (A X1)_ij = -A_ik A_kj / C^2, and the iterate made of it is finite (about 4 / C of it)."""
    from oracle import methods
    C, pos = 128, [(2, 1, 0), (20, 17, 16), (100, 40, 39), (127, 126, 125), (127, 64, 3)]
    A = torch.zeros(max(n_mat, len(pos)), C, C)
    for m, (i, k, j) in enumerate(pos):
        A[m, i, k] = A[m, k, j] = math.sqrt(3.396e38) * C
    for first in range(0, len(pos), n_mat):
        part = A[first:first + n_mat]
        T = tri.tri_inv_ex(part.to(DEV), method=tri.NEWTON_SCHULZ, op_dtype=tri.F32, flags=tri.flag_iters(2)).cpu().double().numpy()
        assert np.isfinite(T).all()
        for m, (i, k, j) in enumerate(pos[first:first + n_mat]):
            want = methods.newton_schulz_closed_form(part[m].double().numpy(), 2)[i, j]
            assert abs(T[m, i, j] / want - 1) < 1e-6, (i, k, j, T[m, i, j], want)


# ------------------------------------------------------------------ packed sequences: the offsets' way to the device
@pytest.mark.parametrize("n_seq", [0, 1, 228, 229, 230, 459, 900])
def test_chunk_offsets_by_kernel_arguments(n_seq):
    """The offsets of n_seq sequences (empty ones among them) against the host lists, at the sizes where one launch's argument block
    (460 values) ends inside, at and behind an array."""
    import ctypes
    r = np.random.default_rng(n_seq)
    lens = [int(x) for x in r.integers(0, 300, n_seq)]
    dst = torch.full((2 * (n_seq + 1) + 2,), -7, dtype=torch.int64, device=DEV)
    chunks = ctypes.c_int64(-1)
    st = tri.lib().triinv_detail_chunk_offsets((ctypes.c_int64 * n_seq)(*lens), n_seq, 64, sum(lens), dst.data_ptr(), ctypes.byref(chunks), None)
    torch.cuda.synchronize()
    cu_s, cu_c = tri.varlen_chunk_offsets(lens, 64)
    assert st == 0 and chunks.value == cu_c[-1]
    assert dst.tolist() == cu_s + cu_c + [-7, -7]


def test_packed_sequences_by_either_route():
    """Lists, numpy integers, tensors and generators of lengths, a side stream, and more sequences than the kernel-argument route takes
    give the same result; a wrong sum is refused as before."""
    lens = [3] * 905 + [70, 130, 1]
    total, H, C = sum(lens), 2, 64
    g = torch.Generator().manual_seed(3)
    K = torch.nn.functional.normalize(torch.randn(total, H, 64, generator=g), dim=-1).bfloat16().to(DEV)
    beta = torch.rand(total, H, generator=g).to(DEV)
    every = tri.gdn_chunk_tri_inv_varlen(K, beta, None, lens, C, gate_kind=tri.GATE_NONE)      # copied
    few = [2715, 70, 130, 1]
    for way in (few, tuple(few), np.array(few), torch.tensor(few), iter(few)):
        T = tri.gdn_chunk_tri_inv_varlen(K, beta, None, way, C, gate_kind=tri.GATE_NONE)
        assert torch.equal(T[-5 * H:], every[-5 * H:]), type(way)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    S = tri.gdn_chunk_tri_inv_varlen(K, beta, None, few, C, gate_kind=tri.GATE_NONE, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(S, T)
    for wrong in (few + [1], [2716] + few[1:], [2715, 70, -1, 132], [1] * 905 + [-1, total - 904], [total + 2 ** 64]):
        with pytest.raises(ValueError):
            tri.gdn_chunk_tri_inv_varlen(K, beta, None, wrong, C, gate_kind=tri.GATE_NONE)
    with pytest.raises(tri.TriInvError) as e:
        tri.gdn_chunk_tri_inv_varlen(K, beta, None, few, 48, gate_kind=tri.GATE_NONE)
    assert e.value.status == -2


def test_packed_sequences_report_a_failing_offsets_launch(monkeypatch):
    """A launch of the offsets kernel that the runtime refuses is reported, not taken for a reason to copy them instead."""
    class Refused:
        def __getattr__(self, name):
            return (lambda *a: -8) if name == "triinv_detail_chunk_offsets" else getattr(lib, name)
    lib = tri.lib()
    monkeypatch.setattr(tri.binding, "_lib", Refused())
    K, beta = torch.zeros(128, 2, 64, dtype=torch.bfloat16, device=DEV), torch.zeros(128, 2, device=DEV)
    with pytest.raises(tri.TriInvError) as e:
        tri.gdn_chunk_tri_inv_varlen(K, beta, None, [100, 28], 64, gate_kind=tri.GATE_NONE)
    assert e.value.status == -8


def test_packed_sequences_replay_from_a_captured_graph():
    """The packed-sequence calls recorded into a graph with given results: the offsets' buffer comes from the graph's memory, so that
    replays are right after the result's own reference to it is gone (eager calls into the same results, and allocations in
    between, overwrite what was freed)."""
    C, H, lens = 64, 3, [70, 0, 1, 130, 64, 7]
    total = sum(lens)
    gen = torch.Generator().manual_seed(17)
    def inputs():
        K = torch.nn.functional.normalize(torch.randn(total, H, 64, generator=gen), dim=-1).bfloat16().to(DEV)
        return K, torch.rand(total, H, generator=gen).to(DEV), torch.randn(total, H, 72, generator=gen).bfloat16().to(DEV)
    ins = [inputs() for _ in range(3)]
    K, beta, X = (t.clone() for t in ins[0])
    inv = lambda T=None: tri.gdn_chunk_tri_inv_varlen(K, beta, None, lens, C, T=T, gate_kind=tri.GATE_NONE)
    solve = lambda W=None: tri.gdn_chunk_tri_solve_varlen(K, beta, None, X, lens, C, row_scale=beta, W=W, gate_kind=tri.GATE_NONE)
    T, W = inv(), solve()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        inv(T)
        solve(W)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        inv(T)
        solve(W)
    for rep in range(6):
        for dst, src in zip((K, beta, X), ins[rep % 3]):
            dst.copy_(src)
        inv(T)
        solve(W)
        junk = [torch.full((14,), -1 - i, dtype=torch.int64, device=DEV) for i in range(50)]
        T.fill_(7.0)
        W.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(T, inv()) and torch.equal(W, solve()), f"replay {rep} differs from the eager call"
        assert all(bool((j == -1 - i).all()) for i, j in enumerate(junk)), "a replay wrote memory that is not the graph's"


# ------------------------------------------------------------------ every element of a given A in its place
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16], ids=["f32", "f16", "bf16"])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_input_elements_in_place(C, dt):
    """Matrices with a single entry below the diagonal, where (I + A)^-1 = I - A exactly, the entry walking over every position
    of the tiles at the edges, of every level inside a leaf and over the element pairs whose lanes exchange data; NaN on and above
    the diagonal."""
    pos = [(i, j) for i in range(C) for j in range(i) if (i % 16 in (0, 1, 7, 15) or j // 16 == i // 16) and j % 4 in (0, 1, 3)]
    A = torch.full((len(pos), C, C), float("nan"))
    low = torch.tril(torch.ones(C, C, dtype=torch.bool), -1)
    A[:, low] = 0
    want = torch.eye(C).repeat(len(pos), 1, 1)
    for m, (i, j) in enumerate(pos):
        A[m, i, j] = 1 + j / 128 if dt != torch.float16 else 1 + (i * C + j) / 16384 // (1 / 1024) / 1024
        want[m, i, j] = -A[m, i, j]
    for method in (tri.BLOCK_RECURSIVE, tri.FWD_SUBST):
        T = tri.tri_inv_ex(A.to(dt).to(DEV), method=method, op_dtype={torch.float32: tri.F32, torch.float16: tri.F16, torch.bfloat16: tri.BF16}[dt])
        assert torch.equal(T.cpu(), want), (C, dt, tri.METHOD_NAMES[method])


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_smallest_input_elements(C, dt):
    """fp16 A with subnormal entries (bf16: the smallest normal ones), fp32 operands: a single entry below the diagonal,
    (I + A)^-1 = I - A exactly.  In one of the two orientations a tile is turned by a matrix product with the identity, which must
    not flush them."""
    bits = [1, 2, 3, 0x155, 0x2aa, 0x3ff] if dt == torch.float16 else [0x80, 0x81, 0x155]
    pos = [(i, j) for i in range(1, C) for j in (0, i // 2, i - 1)]
    A = torch.zeros(len(pos), C, C, dtype=dt)
    for m, (i, j) in enumerate(pos):
        A[m, i, j] = torch.tensor(bits[m % len(bits)] | (-0x8000 if m % 2 else 0), dtype=torch.int16).view(dt)
    want = torch.eye(C) - A.float()
    for method in (tri.BLOCK_RECURSIVE, tri.MIXED, tri.NEUMANN, tri.FWD_SUBST):
        T = tri.tri_inv_ex(A.to(DEV), method=method, op_dtype=tri.F32)
        assert torch.equal(T.cpu(), want), (C, dt, tri.METHOD_NAMES[method])


# ------------------------------------------------------------------ forward substitution, 16 rows at a time
@pytest.mark.parametrize("in_dt", [torch.float32, torch.bfloat16], ids=["A_f32", "A_bf16"])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_forward_substitution_by_tile_rows(C, in_dt):
    """Every element against the oracle within the elementwise bound, garbage on and above the diagonal, for one matrix and for an
    odd number of them; a matrix without off-diagonal tiles (block diagonal) and one with the diagonal tiles empty, where
    a tile row's two halves (the leaf, the products) each stand alone; the 16-bit result is the fp32 one rounded once."""
    A = si.random_strict_lower(7, C, 0.2, seed=31).to(in_dt)
    tile = torch.arange(C) // 16
    same = tile[:, None] == tile[None, :]
    A[1][~same] = 0
    A[2][same] = 0
    for n in (1, 7):
        T = tri.tri_inv_ex(A[:n].to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32)
        check(T, oracle.tri_inv(A[:n]), 1e-5, f"forward C={C} n={n}")
    for out in (torch.float16, torch.bfloat16):
        assert torch.equal(tri.tri_inv_ex(A.to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32, out_dtype=out), T.to(out))


def row_by_row_fp32(A: np.ndarray) -> np.ndarray:
    """(I + strict_lower(A))^-1 by substitution row by row in fp32, each element one chain of fused multiply-adds from the
    first row down (a multiply-add is formed in fp64, where the product is exact, and rounded once more to fp32)."""
    n, C, _ = A.shape
    T = np.zeros((n, C, C), np.float32)
    for i in range(C):
        acc = np.zeros((n, C), np.float32)
        for j in range(i):
            acc = (A[:, i, j, None].astype(np.float64) * T[:, j] + acc).astype(np.float32)
        T[:, i, :i] = -acc[:, :i]
        T[:, i, i] = 1
    return T


@pytest.mark.parametrize("keys", ["rank4", "gaussian"])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_forward_substitution_no_less_accurate_than_row_by_row(C, keys):
    """The error below the diagonal against 64 bits, over 192 matrices: no larger than that of fp32 substitution row by row on the
    same A.  Correlated keys without decay are the input where the order of the sums and the solve of the diagonal
    block show (sums down the tiles in one chain and a product with the block's inverse: 1.13 to 1.3 times row by row; the kernel's
    own order: 0.97 to 0.99 times; at C = 16 it is row by row)."""
    gen = torch.Generator().manual_seed(5)
    n, d = 192, 128
    K, beta = torch.randn(n, C, d, generator=gen), torch.sigmoid(torch.randn(n, C, 1, generator=gen))
    if keys == "rank4":
        K = 0.05 * K + torch.randn(n, C, 4, generator=gen) @ torch.randn(4, d, generator=gen)
        beta = 0.9 + 0.1 * torch.rand(n, C, 1, generator=gen)
    K = torch.nn.functional.normalize(K, dim=-1)
    A = torch.tril(K @ K.transpose(1, 2) * beta, -1)
    want = np.tril(oracle.tri_inv(A), -1)
    size = np.linalg.norm(want)
    ours = tri.tri_inv_ex(A.to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32).cpu().numpy()
    e = np.linalg.norm(np.tril(ours, -1) - want) / size
    e0 = np.linalg.norm(np.tril(row_by_row_fp32(A.numpy()), -1) - want) / size
    assert e <= (e0 if C > 16 else 1.001 * e0), (C, keys, e, e0)


# ------------------------------------------------------------------ what a non-finite entry reaches
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_non_finite_entry_reaches_only_the_rows_that_depend_on_it_forward(C):
    """Forward substitution, entry (i, j) infinite or NaN: the rows above i and the columns from i on do not depend on it."""
    A = torch.tril(torch.randn(1, C, C, generator=torch.Generator().manual_seed(9)) * 0.1, -1)
    clean = tri.tri_inv_ex(A.to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32)[0]
    pos = sorted({(i, j) for i in (1, 5, 15, 16, 22, C // 2, C // 2 + 9, C - 1) for j in (0, 3, i - 1, i - 2) if 0 <= j < i < C})
    for bad in (float("inf"), float("nan")):
        M = A.repeat(len(pos), 1, 1)
        for m, (i, j) in enumerate(pos):
            M[m, i, j] = bad
        T = tri.tri_inv_ex(M.to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32)
        for m, (i, j) in enumerate(pos):
            assert torch.equal(T[m, :i], clean[:i]), (C, i, j, bad)
            assert torch.equal(T[m, :, i:], clean[:, i:]), (C, i, j, bad)
            assert not torch.isfinite(T[m, i, j])


@pytest.mark.parametrize("op", _OPS, ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("C", [32, 64, 128])
def test_non_finite_entry_reaches_only_the_tiles_that_depend_on_it(C, op):
    """The matrix-product methods, an infinite or NaN entry below the diagonal in tile (I, J) of 16 x 16: tile rows above I and tile
    columns right of J of the result do not depend on it and are those of the matrix without it, bit for bit."""
    NB = C // 16
    A = torch.tril(torch.randn(1, C, C, generator=torch.Generator().manual_seed(11)) * 0.1, -1)
    tiles = [(I, J) for I in range(NB) for J in range(I + 1)]
    pos = [(16 * I + 9, 16 * J + 4) for I, J in tiles]
    M, Z = A.repeat(2 * len(pos), 1, 1), A.repeat(len(pos), 1, 1)
    for m, (i, j) in enumerate(pos):
        Z[m, i, j] = 0
        M[m, i, j], M[m + len(pos), i, j] = float("inf"), float("nan")
    for method in (tri.NEWTON_SCHULZ, tri.NEUMANN, tri.BLOCK_RECURSIVE, tri.MIXED, tri.MIXED_B32, tri.BLOCK_DIRECT):
        for in_dt in (torch.float32, torch.bfloat16):
            T = tri.tri_inv_ex(M.to(in_dt).to(DEV), method=method, op_dtype=op).cpu()
            want = tri.tri_inv_ex(Z.to(in_dt).to(DEV), method=method, op_dtype=op).cpu()
            for m in range(2 * len(pos)):
                (I, J), w = tiles[m % len(pos)], want[m % len(pos)]
                assert torch.equal(T[m, :16 * I], w[:16 * I]), (tri.METHOD_NAMES[method], in_dt, I, J, "rows above")
                assert torch.equal(T[m, :, 16 * J + 16:], w[:, 16 * J + 16:]), (tri.METHOD_NAMES[method], in_dt, I, J, "columns right")


# ------------------------------------------------------------------ forward substitution by wavefront shuffles
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
def test_forward_substitution_shuffle_variant(cases, dt):
    A = torch.from_numpy(cases[2]["A"].astype(np.float32)).to(dt)
    T_ref = oracle.tri_inv(A)
    T = tri.tri_inv_ex(A.to(DEV), method=tri.FWD_SUBST, op_dtype=tri.F32, flags=tri.FLAG_FWD_SHUFFLE)
    check(T, T_ref, 1e-5, f"fwd shuffle {dt}")
    junk = si.random_strict_lower(5, 64, 0.2, seed=9)                    # NaN / garbage on and above the diagonal
    check(tri.tri_inv_ex(junk.to(DEV), method=tri.FWD_SUBST, flags=tri.FLAG_FWD_SHUFFLE), oracle.tri_inv(junk), 1e-5, "fwd shuffle, junk upper")
    with pytest.raises(tri.TriInvError) as e:
        tri.tri_inv_ex(torch.zeros(2, 128, 128, device=DEV), method=tri.FWD_SUBST, flags=tri.FLAG_FWD_SHUFFLE)
    assert e.value.status == -9


# ------------------------------------------------------------------ HIP graph capture
def test_entry_points_replay_from_a_captured_graph():
    """The entry points neither allocate nor synchronise, so a launch-bound caller can record them into a HIP
    graph.  The graph is replayed several times with the program's own eager work and synchronisations in
    between, on new input values each time, and every replay is compared with the eager result."""
    C = 64
    inps = [si.make_inputs(si.workload(1, B=1, Tlen=4 * C + 9, H=6, C=C), seed_offset=k) for k in range(3)]
    A_in = [torch.from_numpy(oracle.build_A_ragged(i["K"], i["beta"], i["g"], 0, C).astype(np.float32)) for i in inps]
    K = inps[0]["K"].to(DEV).clone()
    beta, g = inps[0]["beta"].to(DEV).clone(), inps[0]["g"].to(DEV).clone()
    A = A_in[0].to(DEV).clone()
    n_mat = A.shape[0]
    T1 = torch.empty((n_mat, C, C), device=DEV)
    T2 = torch.empty((n_mat, C, C), device=DEV)
    rhs = [si.make_rhs(i["workload"], 64, torch.bfloat16, seed_offset=k) for k, i in enumerate(inps)]
    X, sc = rhs[0]["X"].to(DEV).clone(), rhs[0]["row_scale"].to(DEV).clone()
    W = torch.empty_like(X)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):      # warm-up on the side stream, as graph capture asks for
        tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=T1)
        tri.tri_inv_ex(A, T=T2, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
        tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=sc, W=W)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=T1)
        tri.tri_inv_ex(A, T=T2, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
        tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=sc, W=W)
    for rep in range(6):
        src = inps[rep % 3]
        K.copy_(src["K"].to(DEV))
        beta.copy_(src["beta"].to(DEV))
        g.copy_(src["g"].to(DEV))
        A.copy_(A_in[rep % 3].to(DEV))
        X.copy_(rhs[rep % 3]["X"].to(DEV))
        sc.copy_(rhs[rep % 3]["row_scale"].to(DEV))
        T1.fill_(7.0)
        T2.fill_(7.0)
        W.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        E1 = tri.gdn_chunk_tri_inv_ex(K, beta, g, C)
        E2 = tri.tri_inv_ex(A, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
        E3 = tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=sc)
        torch.cuda.synchronize()
        assert torch.equal(T1, E1) and torch.equal(T2, E2) and torch.equal(W, E3), f"replay {rep} differs from the eager launch"
        check_solve(W, oracle.gdn_chunk_tri_solve(src["K"], src["beta"], src["g"], rhs[rep % 3]["X"], rhs[rep % 3]["row_scale"], 0, C),
                    2e-2, f"graph replay {rep} (solve)", C=C)
        check(T1, oracle.gdn_chunk_tri_inv_ragged(src["K"], src["beta"], src["g"], 0, C), 2e-2, f"graph replay {rep}")


# ------------------------------------------------------------------ mixed recursion with b0 = 32
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("C", [32, 64, 128])
def test_mixed_recursion_b32(cases, C, op):
    """Alg. 2 with b0 = 32: inside the tolerance on benign inputs (standalone, every gate kind, short last chunk) and,
    with its default refinement step, on the stress recipe; against the numpy statement of Alg. 2 with the same b0,
    r and operand rounding the fp32-operand result agrees to fp32 rounding."""
    from oracle import methods
    for gate_kind, idx in ((0, 1), (1, 3), (2, 2)):
        inp = si.make_inputs(si.workload(idx, B=1, Tlen=3 * C + 9, H=5, C=C, d_k=128, k_dtype="bf16", gate_kind=gate_kind))
        T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        T = tri.gdn_chunk_tri_inv_ex(inp["K"].to(DEV), inp["beta"].to(DEV), g, C, gate_kind=gate_kind, method=tri.MIXED_B32,
                                     op_dtype=op)
        check(T, T_ref, TOL[op], f"mixed_b32 fused C={C} gate={gate_kind}", op=op, key_abs=key_abs_term(inp, gate_kind, C))
    A = si.random_strict_lower(21, C, 0.15, seed=5)
    T32 = oracle.tri_inv(A)
    for r in (0, 1, 2):
        T = tri.tri_inv_ex(A.to(DEV), method=tri.MIXED_B32, op_dtype=op, flags=tri.flag_mxr_r(r))
        check(T, T32, TOL[op], f"mixed_b32 standalone C={C} r={r}", op=op)
        if op == tri.F32:
            want = np.stack([methods.mxr(np.tril(A[m].numpy().astype(np.float64), -1), 32, r, "f32") for m in range(3)])
            got = T.cpu().numpy().astype(np.float64)[:3]
            assert np.abs(got - want).max() <= 2e-6, (C, r)
    if C >= 64:
        st = si.make_inputs(si.workload(4, Tlen=4 * C, H=3, C=C))
        T_ref = oracle.gdn_chunk_tri_inv(st["K"], st["beta"], None, 2, C)
        T = tri.gdn_chunk_tri_inv_ex(st["K"].to(DEV), st["beta"].to(DEV), None, C, gate_kind=tri.GATE_NONE, method=tri.MIXED_B32,
                                     op_dtype=op)
        check(T, T_ref, TOL[op], f"mixed_b32 stress C={C}", op=op)


def test_mixed_recursion_b32_needs_c32():
    with pytest.raises(tri.TriInvError) as e:
        tri.tri_inv_ex(torch.zeros(2, 16, 16, device=DEV), method=tri.MIXED_B32, op_dtype=tri.F32)
    assert e.value.status == -9
    with pytest.raises(tri.TriInvError) as e:      # also with the refinement flag
        tri.tri_inv_ex(torch.zeros(2, 16, 16, device=DEV), method=tri.MIXED_B32, op_dtype=tri.F32, flags=1)
    assert e.value.status == -9


# ------------------------------------------------------------------ per-channel gate with a strong decay
@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_per_channel_gate_with_a_strong_decay(C, op):
    """g falls by ~2.4 per token (~150 over a chunk of 64): exp(+-(g - one anchor per chunk)) would overflow
    fp32; with one anchor per 16 rows every exponent stays small and the result is inside the tolerance."""
    inp = si.make_inputs(si.workload(3, B=1, Tlen=4 * C + 5, H=3, C=C, rate_scale=3.0))
    g0 = inp["g"][0]
    half = max(float((g0[c0:c0 + C] - g0[min(c0 + C // 2, g0.shape[0] - 1)]).abs().max()) for c0 in range(0, g0.shape[0], C))
    in16 = max(float((g0[t0] - g0[t0:min(t0 + 16, (t0 // C + 1) * C)]).abs().max()) for t0 in range(0, g0.shape[0], 16))
    assert in16 < 85.0, in16                      # what the tile-row anchors need
    assert C < 64 or half > 89.0, half            # exp(g - g_mid) with one anchor per chunk overflows fp32 here
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], 1, C)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    # C = 128: the recursions (two wavefronts per chunk, tile-row anchors); forward substitution and the two-launch methods
    # build A with a single anchor per chunk there and are bound by the decay over the whole chunk
    methods = (tri.BLOCK_RECURSIVE, tri.FWD_SUBST, tri.MIXED_B32 if C >= 32 else tri.MIXED, tri.NEUMANN) if C < 128 else \
        (tri.BLOCK_RECURSIVE, tri.MIXED, tri.MIXED_B32, tri.BLOCK_DIRECT)
    for method in methods:
        T = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=tri.GATE_PER_CHANNEL, method=method, op_dtype=op)
        # fp32 operands: the gate's exponent g - a reaches ~80 here, and its fp32 rounding alone (80 x 1.44 x 2^-24) puts a
        # relative error of ~5e-6 on the gated keys -- above the elementwise model's fp32 term, so norms only in that mode
        check(T, T_ref, TOL[op] if method != tri.FWD_SUBST or op == tri.F32 else 2e-2, f"strong decay C={C} {tri.METHOD_NAMES[method]}",
              op=op, key_abs=SKIP if op == tri.F32 else key_abs_term(inp, 1, C))


# ------------------------------------------------------------------ the chunk matrices alone
@pytest.mark.parametrize("gate_kind", [0, 1, 2])
@pytest.mark.parametrize("C", [16, 32, 64, 128])
def test_build_A_alone(C, gate_kind):
    """gdn_chunk_build_A against the oracle's fp64 A (scalar / no gate: exact products of the stored keys, fp32
    accumulation and gate: 1e-6; per-channel gate: gated keys rounded to the operand type), exact zeros on and
    above the diagonal, and A -> tri_inv agrees with the fused entry point."""
    idx = {0: 1, 1: 3, 2: 2}[gate_kind]
    for d_k in (128, 96):
        inp = si.make_inputs(si.workload(idx, B=2, Tlen=3 * C + 11, H=3, C=C, d_k=d_k, k_dtype="bf16", gate_kind=gate_kind))
        A_ref = oracle.build_A_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C)
        K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        for op, tol in ((tri.F32, 1e-6), (tri.BF16, 1e-6 if gate_kind != 1 else 1e-2)):
            A = tri.gdn_chunk_build_A(K, beta, g, C, gate_kind=gate_kind, op_dtype=op)
            torch.cuda.synchronize()
            Ah = A.cpu().numpy().astype(np.float64)
            assert np.array_equal(np.triu(Ah), np.zeros_like(Ah)), "entries on or above the diagonal"
            num = np.linalg.norm(Ah - A_ref, axis=(1, 2))
            den = np.maximum(np.linalg.norm(A_ref, axis=(1, 2)), 1e-30)
            assert (num / den).max() <= tol, (C, gate_kind, d_k, op, (num / den).max())
        A16 = tri.gdn_chunk_build_A(K, beta, g, C, gate_kind=gate_kind, op_dtype=tri.F32, out_dtype=torch.bfloat16)
        A32 = tri.gdn_chunk_build_A(K, beta, g, C, gate_kind=gate_kind, op_dtype=tri.F32)
        torch.cuda.synchronize()
        assert torch.equal(A16, A32.to(torch.bfloat16))
        if d_k == 128:
            T_two = tri.tri_inv_ex(A32, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
            T_one = tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=gate_kind, method=tri.BLOCK_DIRECT, op_dtype=tri.F32)
            check(T_two, oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C), 1e-5, "A then tri_inv")
            torch.cuda.synchronize()
            assert float((T_two - T_one).abs().max()) <= 1e-5


# ------------------------------------------------------------------ the inverse applied: W = (I + A)^{-1} diag(s) X
XDT = {tri.F32: torch.float32, tri.F16: torch.float16, tri.BF16: torch.bfloat16}
# fp32: products and sums in fp32 throughout; 16-bit: the inverse's tolerance plus one rounding of the scaled inverse
# and one of W to the 16-bit type (2^-9 each for bf16) -- still inside 2e-2
SOLVE_TOL = {tri.F32: 1e-5, tri.F16: 2e-2, tri.BF16: 2e-2}


def check_solve(W_gpu, W_ref, tol, what, C=None, seqlens=None, ctx=None):
    """W_gpu, W_ref: [B, rows, H, d_x].  The relative Frobenius error is taken per chunk and head (C: chunk size; seqlens: row
    counts of the packed sequences, each chunked on its own; without C the rows passed are taken as one chunk per head),
    so that one bad row in a long sequence cannot hide in the norm.  ctx = dict(inp, rhs, gate_kind, op, [scale]) adds the
    elementwise bound: |dW| <= (E_T + 2u B)|s X| + u |W| + 1e-6, with E_T the elementwise bound of the inverse, B =
    |T||I + A||T| >= |T| (the scaled inverse is rounded to the operand type once more) and the last term the rounding of
    W to its storage type."""
    torch.cuda.synchronize()
    Wg = W_gpu.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(Wg).all(), f"{what}: non-finite output"
    B, rows, H, d_x = Wg.shape
    if C is None:
        starts = [0]
    else:
        starts, t0 = [], 0
        for n in (seqlens if seqlens is not None else [rows]):
            starts += [t0 + c0 for c0 in range(0, int(n), C)]
            t0 += int(n)
    if rows:
        num = np.sqrt(np.add.reduceat(((Wg - W_ref) ** 2).sum(axis=3), starts, axis=1))      # [B, chunks, H]
        den = np.sqrt(np.add.reduceat((W_ref ** 2).sum(axis=3), starts, axis=1))
        err = (num / den).max()
    else:
        err = 0.0
    assert err <= tol, f"{what}: rel_fro max {err:.3e} > {tol} (per chunk and head)"
    if ctx is not None and seqlens is None and C is not None:
        inp, rhs, gate_kind, op = ctx["inp"], ctx["rhs"], ctx["gate_kind"], ctx["op"]
        T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], gate_kind, C)        # [B * n_chunk * H, C, C]
        u = UNIT[op]
        Ta = np.abs(T_ref)
        E = elementwise_bound(T_ref, op, key_abs_term(inp, gate_kind, C)) + 2 * u * (Ta @ np.abs(np.linalg.inv(T_ref)) @ Ta)
        n_chunk = -(-rows // C)
        E = E.reshape(B, n_chunk, H, C, C)
        sX = rhs["X"].double().numpy()
        if ctx.get("scale", True) and rhs.get("row_scale") is not None:
            sX = sX * rhs["row_scale"].double().numpy()[..., None]
        pad = np.zeros((B, n_chunk * C, H, d_x))
        pad[:, :rows] = np.abs(sX)
        pad = pad.reshape(B, n_chunk, C, H, d_x).transpose(0, 1, 3, 2, 4)                              # [B, n_chunk, H, C, d_x]
        bound = (E @ pad).transpose(0, 1, 3, 2, 4).reshape(B, n_chunk * C, H, d_x)[:, :rows] + u * np.abs(W_ref) + 1e-6
        ratio = np.abs(Wg - W_ref) / bound
        worst = np.unravel_index(np.argmax(ratio), ratio.shape)
        assert ratio.max() <= 1.0, f"{what}: element {worst} off by {abs(Wg[worst] - W_ref[worst]):.3e}, {ratio.max():.2f} x its bound"
    return err


def solve_case(idx, d_x, op, **kw):
    w = si.workload(idx, **kw)
    inp = si.make_inputs(w)
    rhs = si.make_rhs(w, d_x, XDT[op])
    return w, inp, rhs


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("method", [tri.BLOCK_RECURSIVE, tri.MIXED], ids=lambda m: tri.METHOD_NAMES[m])
@pytest.mark.parametrize("idx,kw", [(0, {}), (1, dict(Tlen=512)), (2, dict(B=2, Tlen=256, H=5)), (3, dict(B=1, Tlen=256, H=3))])
def test_solve_matches_oracle(idx, kw, method, op):
    w, inp, rhs = solve_case(idx, 128, op, **kw)
    W_ref = oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], rhs["row_scale"], w.gate_kind, w.C)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    W = tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), g, rhs["X"].to(DEV), w.C,
                                row_scale=rhs["row_scale"].to(DEV), gate_kind=w.gate_kind, method=method)
    check_solve(W, W_ref, SOLVE_TOL[op], f"cfg{idx} {tri.METHOD_NAMES[method]} {tri.DTYPE_NAMES[op]}", C=w.C,
                ctx=dict(inp=inp, rhs=rhs, gate_kind=w.gate_kind, op=op))


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("method", [tri.BLOCK_RECURSIVE, tri.MIXED], ids=lambda m: tri.METHOD_NAMES[m])
@pytest.mark.parametrize("Tlen", [512, 300])
def test_solve_c128_stress_recipe(Tlen, method, op):
    # the C = 128 stress recipe (large growth in the inverse), full and short last chunk, scalar-gated variant included
    # and the per-channel gate (two wavefronts per chunk, the right-hand side requested after the recursion)
    for idx, kw in ((4, dict(Tlen=Tlen, H=3)), (1, dict(Tlen=Tlen, H=3, C=128)), (3, dict(B=1, Tlen=Tlen, H=3, C=128))):
        w, inp, rhs = solve_case(idx, 128, op, **kw)
        W_ref = oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], rhs["row_scale"], w.gate_kind, w.C)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        W = torch.full(rhs["X"].shape, float("nan"), dtype=XDT[op], device=DEV)
        tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), g, rhs["X"].to(DEV), w.C, row_scale=rhs["row_scale"].to(DEV),
                                W=W, gate_kind=w.gate_kind, method=method)
        check_solve(W, W_ref, SOLVE_TOL[op], f"C=128 cfg{idx} Tlen={Tlen} {tri.METHOD_NAMES[method]} {tri.DTYPE_NAMES[op]}", C=w.C,
                    ctx=dict(inp=inp, rhs=rhs, gate_kind=w.gate_kind, op=op))


@pytest.mark.parametrize("d_x", [8, 64, 72, 128, 200, 256, 512])
@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_solve_column_counts(d_x, op):
    # part of a 128-column group, exactly one, several, and a last group that is not full
    w, inp, rhs = solve_case(1, d_x, op, Tlen=192, H=4)
    W_ref = oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], None, w.gate_kind, w.C)
    W = torch.full(rhs["X"].shape, float("nan"), dtype=XDT[op], device=DEV)
    tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), rhs["X"].to(DEV), w.C, W=W)
    check_solve(W, W_ref, SOLVE_TOL[op], f"d_x={d_x}", C=w.C,   # every element written (no NaN left), none beyond
                ctx=dict(inp=inp, rhs=rhs, gate_kind=w.gate_kind, op=op, scale=False))


@pytest.mark.parametrize("d_x", [8, 72, 128, 200, 256, 512])
@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("idx,kw", [(1, {}), (3, dict(B=1)), (4, {}), (1, dict(k_dtype="f32"))], ids=["scalar", "channel", "nogate", "f32keys"])
def test_solve_column_counts_c128(idx, kw, d_x, op):
    # C = 128 on two wavefronts: part of a column group, exactly one, several (the waves meet again between groups), a
    # last group that is not full; the last chunk is short (300 = 2 * 128 + 44 tokens: a tile row cut in the middle)
    w, inp, rhs = solve_case(idx, d_x, op, Tlen=300, H=3, C=128, d_k=128, **kw)
    W_ref = oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], rhs["row_scale"], w.gate_kind, w.C)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    W = torch.full(rhs["X"].shape, float("nan"), dtype=XDT[op], device=DEV)
    tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), g, rhs["X"].to(DEV), w.C, row_scale=rhs["row_scale"].to(DEV), W=W,
                            gate_kind=w.gate_kind)
    check_solve(W, W_ref, SOLVE_TOL[op], f"C=128 cfg{idx} {kw} d_x={d_x}", C=w.C,   # every element written (no NaN left)
                ctx=dict(inp=inp, rhs=rhs, gate_kind=w.gate_kind, op=op))


@pytest.mark.parametrize("C", [16, 32, 64, 128])
@pytest.mark.parametrize("Tlen", [1, 50, 64, 150])
@pytest.mark.parametrize("gate_kind", [tri.GATE_SCALAR, tri.GATE_PER_CHANNEL, tri.GATE_NONE])
def test_solve_chunk_sizes_and_short_last_chunk(C, Tlen, gate_kind):
    idx = {tri.GATE_SCALAR: 1, tri.GATE_PER_CHANNEL: 3, tri.GATE_NONE: 4}[gate_kind]
    w, inp, rhs = solve_case(idx, 64, tri.BF16, B=2, Tlen=Tlen, H=3, C=C)
    W_ref = oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], rhs["row_scale"], gate_kind, C)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    # W sits inside a larger allocation filled with a sentinel: nothing outside [B, Tlen, H, d_x] may be touched
    pad = 4096
    buf = torch.full((pad + rhs["X"].numel() + pad,), -7.0, dtype=torch.bfloat16, device=DEV)
    W = buf[pad:pad + rhs["X"].numel()].view(rhs["X"].shape)
    tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), g, rhs["X"].to(DEV), C, row_scale=rhs["row_scale"].to(DEV),
                            W=W, gate_kind=gate_kind)
    check_solve(W, W_ref, 2e-2, f"C={C} Tlen={Tlen} gate={gate_kind}", C=C, ctx=dict(inp=inp, rhs=rhs, gate_kind=gate_kind, op=tri.BF16))
    assert (buf[:pad] == -7.0).all() and (buf[pad + rhs["X"].numel():] == -7.0).all()


def test_solve_agrees_with_the_stored_inverse_applied_in_fp32():
    # the same inverse, written out by gdn_chunk_tri_inv_ex and applied by torch in fp32: the two paths differ by
    # the rounding of the scaled inverse and of W only
    w, inp, rhs = solve_case(1, 128, tri.BF16, Tlen=256, H=4)
    K, beta, g, X, s = (inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), rhs["X"].to(DEV), rhs["row_scale"].to(DEV))
    W = tri.gdn_chunk_tri_solve(K, beta, g, X, w.C, row_scale=s).float()
    T = tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C).view(1, 4, 4, 64, 64)                 # [B, chunk, H, C, C]
    sX = (s[..., None] * X.float()).view(1, 4, 64, 4, 128)                               # [B, chunk, C, H, d_x]
    want = torch.einsum("bchij,bcjhx->bcihx", T, sX).reshape(W.shape)
    rel = ((W - want).norm() / want.norm()).item()
    assert rel < 6e-3, rel


def test_solve_rejects_what_it_does_not_build():
    w, inp, rhs = solve_case(1, 128, tri.BF16, Tlen=128, H=2)
    K, beta, g, X = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), rhs["X"].to(DEV)
    for kwargs in (dict(method=tri.NEUMANN), dict(method=tri.FWD_SUBST), dict(flags=tri.FLAG_REFINE1)):
        with pytest.raises(tri.TriInvError) as e:
            tri.gdn_chunk_tri_solve(K, beta, g, X, 64, **kwargs)
        assert e.value.status == -9
    with pytest.raises(tri.TriInvError) as e:                                           # in place
        tri.gdn_chunk_tri_solve(K, beta, g, X, 64, W=X)
    assert e.value.status == -7
    with pytest.raises(tri.TriInvError) as e:                                           # d_x not a multiple of 8
        tri.gdn_chunk_tri_solve(K, beta, g, X[..., :60].contiguous(), 64)
    assert e.value.status == -5


@pytest.mark.parametrize("gate_kind", [0, 1, 2])
@pytest.mark.parametrize("C", [32, 64, 128])
def test_solve_packed_variable_length_sequences(C, gate_kind):
    H, d_k, d_x = 3, 128, 72
    seqlens = [C, 1, 0, 2 * C + 5, C - 1, 3 * C, 0, 17]
    total = sum(seqlens)
    idx = {0: 1, 1: 3, 2: 4}[gate_kind]
    w = si.workload(idx, B=1, Tlen=total, H=H, C=C, d_k=d_k, k_dtype="bf16")
    inp = si.make_inputs(w)
    rhs = si.make_rhs(w, d_x, torch.bfloat16)
    K, beta, X, s = inp["K"][0].contiguous(), inp["beta"][0].contiguous(), rhs["X"][0].contiguous(), rhs["row_scale"][0].contiguous()
    g = None
    if gate_kind != 2:
        gen = torch.Generator().manual_seed(11)
        shape = (total, H) if gate_kind == 0 else (total, H, d_k)
        rate = -0.05 * torch.nn.functional.softplus(torch.randn(*shape, generator=gen))
        g, t0 = torch.zeros(shape), 0
        for n in seqlens:
            for c0 in range(0, n, C):
                m = min(C, n - c0)
                g[t0 + c0:t0 + c0 + m] = torch.cumsum(rate[t0 + c0:t0 + c0 + m], 0)
            t0 += n
    W_ref = oracle.gdn_chunk_tri_solve_varlen(K, beta, g, X, s, seqlens, gate_kind, C)
    W = torch.full(X.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    tri.gdn_chunk_tri_solve_varlen(K.to(DEV), beta.to(DEV), None if g is None else g.to(DEV), X.to(DEV), seqlens, C,
                                   row_scale=s.to(DEV), W=W, gate_kind=gate_kind)
    check_solve(W[None], W_ref[None], 2e-2, f"solve varlen C={C} gate={gate_kind}", C=C, seqlens=seqlens)


def test_solve_packed_sequences_with_no_tokens_are_a_no_op():
    K = torch.zeros((0, 2, 128), dtype=torch.bfloat16, device=DEV)
    X = torch.zeros((0, 2, 64), dtype=torch.bfloat16, device=DEV)
    W = tri.gdn_chunk_tri_solve_varlen(K, torch.zeros((0, 2), device=DEV), None, X, [0, 0], 64, gate_kind=tri.GATE_NONE)
    assert W.shape == X.shape


def test_forward_substitution_against_the_vendor_triangular_solve(cases):
    # an independent GPU-side check: the ROCm libraries' batched triangular solve of (I + A) T = I in fp32
    A32 = torch.from_numpy(cases[1]["A"].astype(np.float32)).to(DEV)
    C = A32.shape[-1]
    eye = torch.eye(C, device=DEV).expand(A32.shape[0], C, C).contiguous()
    Tv = torch.linalg.solve_triangular(torch.tril(A32, -1) + torch.eye(C, device=DEV), eye, upper=False, unitriangular=True)
    T = tri.tri_inv_ex(A32, method=tri.FWD_SUBST)
    torch.cuda.synchronize()
    rel = ((T - Tv).flatten(1).norm(dim=1) / Tv.flatten(1).norm(dim=1)).max().item()
    assert rel < 1e-6, rel


@pytest.mark.parametrize("idx", [2, 3, 4])
def test_repeated_full_size_launches_agree_bit_for_bit(idx):
    """Every kernel here is deterministic (no atomics, no launch-order dependence), so repeated launches on the same
    inputs give the same bits. A store that picked up a later value of its data registers once showed up as one matrix
    in about a million differing between launches; this keeps watch over the storing and the applied-inverse kernels at
    the size the benchmark runs."""
    w = si.WORKLOADS[idx]
    inp = si.make_inputs(w)
    rhs = si.make_rhs(w, 128, torch.bfloat16)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    X, s = rhs["X"].to(DEV), rhs["row_scale"].to(DEV)

    def launch():
        T = tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=w.gate_kind, method=tri.BLOCK_RECURSIVE, op_dtype=tri.BF16)
        T16 = tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=w.gate_kind, method=tri.BLOCK_RECURSIVE, op_dtype=tri.BF16,
                                       out_dtype=torch.bfloat16)
        W = tri.gdn_chunk_tri_solve(K, beta, g, X, w.C, row_scale=s, gate_kind=w.gate_kind)
        W2 = tri.gdn_chunk_tri_solve_multi(K, beta, g, [X, X], w.C, row_scales=[s, None], gate_kind=w.gate_kind)
        torch.cuda.synchronize()
        return [T.view(torch.int32), T16.view(torch.int16), W.view(torch.int16)] + [x.view(torch.int16) for x in W2]

    first = launch()
    for rep in range(1, 12):
        for name, a, b in zip(("T fp32", "T bf16", "W", "W pair 0", "W pair 1"), launch(), first):
            if not torch.equal(a, b):
                at = (a != b).nonzero()
                pytest.fail(f"cfg{idx} launch {rep}, {name}: {len(at)} elements differ from the first launch, first at {at[:6].cpu().numpy().tolist()}")


@pytest.mark.parametrize("idx", [2, 3, 4])
def test_solve_full_size_workload(idx):
    """gdn_chunk_tri_solve in the launch configuration the benchmark times (full-size workload, d_x = 128, bf16):
    the oracle recomputes sampled chunks, and the residual of (I + A) W = diag(s) X is checked for EVERY chunk (A
    written by gdn_chunk_build_A, products in fp64 on the device)."""
    w = si.WORKLOADS[idx]
    C, d_x = w.C, 128
    inp = si.make_inputs(w)
    rhs = si.make_rhs(w, d_x, torch.bfloat16)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    X, s = rhs["X"].to(DEV), rhs["row_scale"].to(DEV)
    W = tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=s, gate_kind=w.gate_kind)
    torch.cuda.synchronize()
    # (a) sampled chunks against the oracle: chunks are independent, so a slice of whole chunks is a workload of its own
    n_chunk = w.Tlen // C
    rng = np.random.default_rng(idx)
    for b, c in {(0, 0), (w.B - 1, n_chunk - 1)} | {(int(rng.integers(w.B)), int(rng.integers(n_chunk))) for _ in range(6)}:
        sl = (slice(b, b + 1), slice(c * C, (c + 1) * C))
        W_ref = oracle.gdn_chunk_tri_solve(inp["K"][sl], inp["beta"][sl], None if inp["g"] is None else inp["g"][sl],
                                           rhs["X"][sl], rhs["row_scale"][sl], w.gate_kind, C)
        check_solve(W[sl], W_ref, 2e-2, f"full cfg{idx} solve, batch {b} chunk {c}")
    # (b) every chunk: || (I + A) W - s X ||_F / (|| I + A ||_F || W ||_F)
    A = tri.gdn_chunk_build_A(K, beta, g, C, gate_kind=w.gate_kind, op_dtype=tri.F32)             # [B * n_chunk * H, C, C]
    eye = torch.eye(C, device=DEV, dtype=torch.float64)
    Wm = W.view(w.B, n_chunk, C, w.H, d_x).permute(0, 1, 3, 2, 4).reshape(-1, C, d_x)               # matrix order of A
    Rm = (s[..., None] * X.float()).view(w.B, n_chunk, C, w.H, d_x).permute(0, 1, 3, 2, 4).reshape(-1, C, d_x)
    worst = 0.0
    for m0 in range(0, w.n_mat, 4096):
        M = A[m0:m0 + 4096].double() + eye
        Wd = Wm[m0:m0 + 4096].double()
        R = torch.bmm(M, Wd) - Rm[m0:m0 + 4096].double()
        nrm = torch.linalg.matrix_norm(R) / (torch.linalg.matrix_norm(M) * torch.linalg.matrix_norm(Wd))
        assert bool(torch.isfinite(nrm).all())
        worst = max(worst, float(nrm.max()))
    assert worst <= 2e-3, (idx, worst)


@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("idx,kw", [(1, dict(Tlen=300, H=4)), (3, dict(B=2, Tlen=128, H=3)), (4, dict(Tlen=200, H=4, C=32)),
                                    (1, dict(Tlen=96, H=2, C=16)), (4, dict(Tlen=300, H=3)), (1, dict(Tlen=256, H=2, C=128, d_k=64)),
                                    (3, dict(B=1, Tlen=300, H=2, C=128))])
def test_solve_two_right_hand_sides_share_one_inversion(idx, kw, op):
    # two right-hand sides of different widths and scales in one launch: each result is what a launch of its own gives
    # (bit for bit at C <= 64: the same kernels' arithmetic), and matches the oracle
    w = si.workload(idx, **kw)
    inp = si.make_inputs(w)
    r1, r2 = si.make_rhs(w, 128, XDT[op]), si.make_rhs(w, 72, XDT[op], seed_offset=1)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    X1, X2, s2 = r1["X"].to(DEV), r2["X"].to(DEV), r2["row_scale"].to(DEV)
    for method in (tri.BLOCK_RECURSIVE, tri.MIXED):
        W1, W2 = tri.gdn_chunk_tri_solve_multi(K, beta, g, [X1, X2], w.C, row_scales=[None, s2], gate_kind=w.gate_kind, method=method)
        E1 = tri.gdn_chunk_tri_solve(K, beta, g, X1, w.C, gate_kind=w.gate_kind, method=method)
        E2 = tri.gdn_chunk_tri_solve(K, beta, g, X2, w.C, row_scale=s2, gate_kind=w.gate_kind, method=method)
        torch.cuda.synchronize()
        if w.C < 128 or w.gate_kind == tri.GATE_PER_CHANNEL:
            # (scalar / no gate at C = 128: the pair runs on two wavefronts per chunk, the single launch on one: same method, other kernel)
            assert torch.equal(W1, E1) and torch.equal(W2, E2)
        check_solve(W1, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r1["X"], None, w.gate_kind, w.C), SOLVE_TOL[op], "rhs 0", C=w.C)
        check_solve(W2, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r2["X"], r2["row_scale"], w.gate_kind, w.C),
                    SOLVE_TOL[op], "rhs 1", C=w.C)


@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
def test_solve_fp32_keys_with_128_channels_at_c128(op):
    """Keys stored in fp32 at d_k = 128, C = 128: a chunk's keys are 256 registers per lane on one wavefront, so this
    combination exists on two wavefronts per chunk only (each holds half the keys); one and two right-hand sides."""
    w = si.workload(1, B=1, Tlen=2 * 128 + 37, H=3, C=128, d_k=128, k_dtype="f32")
    inp = si.make_inputs(w)
    r1, r2 = si.make_rhs(w, 128, XDT[op]), si.make_rhs(w, 72, XDT[op], seed_offset=1)
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    for method in (tri.BLOCK_RECURSIVE, tri.MIXED):
        W = torch.full(r1["X"].shape, float("nan"), dtype=XDT[op], device=DEV)
        tri.gdn_chunk_tri_solve(K, beta, g, r1["X"].to(DEV), 128, row_scale=r1["row_scale"].to(DEV), W=W, method=method)
        check_solve(W, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r1["X"], r1["row_scale"], w.gate_kind, 128), SOLVE_TOL[op],
                    f"fp32 keys d_k=128 C=128 {tri.METHOD_NAMES[method]} {tri.DTYPE_NAMES[op]}", C=128,
                    ctx=dict(inp=inp, rhs=r1, gate_kind=w.gate_kind, op=op))
        W1, W2 = tri.gdn_chunk_tri_solve_multi(K, beta, g, [r1["X"].to(DEV), r2["X"].to(DEV)], 128,
                                               row_scales=[r1["row_scale"].to(DEV), None], method=method)
        assert torch.equal(W1, W)
        check_solve(W2, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r2["X"], None, w.gate_kind, 128), SOLVE_TOL[op],
                    "rhs 1", C=128)


def test_solve_multi_limits():
    w, inp, rhs = solve_case(4, 64, tri.BF16, Tlen=256, H=2)
    K, beta, X = inp["K"].to(DEV), inp["beta"].to(DEV), rhs["X"].to(DEV)
    with pytest.raises(tri.TriInvError) as e:                                 # three
        tri.gdn_chunk_tri_solve_multi(K, beta, None, [X, X.clone(), X.clone()], 64, gate_kind=tri.GATE_NONE)
    assert e.value.status == -5
    W = torch.empty_like(X)
    with pytest.raises(tri.TriInvError) as e:                                 # both results in one buffer
        tri.gdn_chunk_tri_solve_multi(K, beta, None, [X, X.clone()], 64, Ws=[W, W], gate_kind=tri.GATE_NONE)
    assert e.value.status == -7
    (W1,) = tri.gdn_chunk_tri_solve_multi(K, beta, None, [X], 128, gate_kind=tri.GATE_NONE)   # one is fine at C = 128
    assert torch.equal(W1, tri.gdn_chunk_tri_solve(K, beta, None, X, 128, gate_kind=tri.GATE_NONE))


# ------------------------------------------------------------------ combinations without a fused kernel: build A, invert in place
@pytest.mark.parametrize("op", [tri.F32, tri.F16, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("case", ["kda_c128_neumann", "kda_c128_ns", "f32keys_c128_neumann", "f32keys_c128_ns", "dk96_mixed", "dk96_ns",
                                  "dk256_c128_neumann", "dk32_c32_mixed_b32"])
def test_composed_combinations_match_oracle(case, op):
    """Method / gate / head-dimension combinations that have no fused kernel run as gdn_chunk_build_A into T followed by the
    standalone kernel in place; the result must be what tri_inv_ex gives on that A, bit for bit, and match the oracle."""
    idx, kw, method = {
        "kda_c128_neumann": (3, dict(B=1, Tlen=300, H=3, C=128), tri.NEUMANN),
        "kda_c128_ns": (3, dict(B=1, Tlen=256, H=3, C=128), tri.NEWTON_SCHULZ),
        "f32keys_c128_neumann": (1, dict(B=1, Tlen=256, H=3, C=128, k_dtype="f32"), tri.NEUMANN),
        "f32keys_c128_ns": (1, dict(B=1, Tlen=200, H=3, C=128, k_dtype="f32"), tri.NEWTON_SCHULZ),
        "dk96_mixed": (1, dict(B=2, Tlen=200, H=3, d_k=96), tri.MIXED),
        "dk96_ns": (1, dict(B=2, Tlen=128, H=3, d_k=96), tri.NEWTON_SCHULZ),
        "dk256_c128_neumann": (1, dict(B=1, Tlen=256, H=2, d_k=256, C=128), tri.NEUMANN),
        "dk32_c32_mixed_b32": (1, dict(B=2, Tlen=100, H=3, d_k=32, C=32), tri.MIXED_B32),
    }[case]
    w = si.workload(idx, **kw)
    inp = si.make_inputs(w)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    n_mat = w.B * ((w.Tlen + w.C - 1) // w.C) * w.H
    guard = torch.full((n_mat + 1, w.C, w.C), 7.0, device=DEV)
    T = tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, T=guard[:n_mat], gate_kind=w.gate_kind, method=method, op_dtype=op)
    A = tri.gdn_chunk_build_A(K, beta, g, w.C, gate_kind=w.gate_kind, op_dtype=op)
    E = tri.tri_inv_ex(A, method=method, op_dtype=op)
    torch.cuda.synchronize()
    assert torch.equal(T, E)
    assert bool((guard[n_mat] == 7.0).all())
    T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], w.gate_kind, w.C)
    check(T, T_ref, TOL[op], f"composed {case} {tri.DTYPE_NAMES[op]}", op=op, key_abs=key_abs_term(inp, w.gate_kind, w.C), method=method)


@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("d_k,C,Tlen", [(32, 16, 50), (96, 64, 200), (256, 64, 128), (192, 32, 96)])
def test_solve_other_head_dimensions(d_k, C, Tlen, op):
    # scalar and no-gate kinds with a d_k that has no specialised build: the channel-loop Gram, one and two right-hand sides
    for idx in (1, 4):
        w = si.workload(idx, B=2, Tlen=Tlen, H=3, d_k=d_k, C=C, k_dtype="bf16" if op != tri.F32 else "f32")
        inp = si.make_inputs(w)
        r1, r2 = si.make_rhs(w, 64, XDT[op]), si.make_rhs(w, 136, XDT[op], seed_offset=1)
        K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
        g = None if inp["g"] is None else inp["g"].to(DEV)
        for method in (tri.BLOCK_RECURSIVE, tri.MIXED):
            W = tri.gdn_chunk_tri_solve(K, beta, g, r1["X"].to(DEV), C, row_scale=r1["row_scale"].to(DEV), gate_kind=w.gate_kind,
                                        method=method)
            W1, W2 = tri.gdn_chunk_tri_solve_multi(K, beta, g, [r1["X"].to(DEV), r2["X"].to(DEV)], C,
                                                   row_scales=[r1["row_scale"].to(DEV), None], gate_kind=w.gate_kind, method=method)
            torch.cuda.synchronize()
            assert torch.equal(W, W1)
            check_solve(W, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r1["X"], r1["row_scale"], w.gate_kind, C),
                        SOLVE_TOL[op], f"d_k={d_k} C={C} cfg{idx} rhs 0", C=C)
            check_solve(W2, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], r2["X"], None, w.gate_kind, C),
                        SOLVE_TOL[op], f"d_k={d_k} C={C} cfg{idx} rhs 1", C=C)
    with pytest.raises(tri.TriInvError) as e:                               # C = 128 keeps to d_k = 64 / 128
        w = si.workload(1, B=1, Tlen=128, H=2, d_k=96, C=128)
        inp = si.make_inputs(w)
        tri.gdn_chunk_tri_solve(inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV), si.make_rhs(w, 64)["X"].to(DEV), 128)
    assert e.value.status == -9


# ------------------------------------------------------------------ the refinement step after every matrix-product method
REFINE_METHODS = [tri.BLOCK_RECURSIVE, tri.MIXED, tri.MIXED_B32, tri.BLOCK_DIRECT, tri.NEUMANN, tri.NEWTON_SCHULZ]


@pytest.mark.parametrize("op", [tri.F32, tri.BF16], ids=lambda o: tri.DTYPE_NAMES[o])
@pytest.mark.parametrize("method", REFINE_METHODS, ids=lambda m: tri.METHOD_NAMES[m])
@pytest.mark.parametrize("idx", [1, 3, 4])
def test_refinement_step_after_every_method(cases, idx, method, op):
    """TRIINV_FLAG_REFINE1 (Alg. 6) behind each matrix-product method, standalone and fused, at the workload's own C (64, 64 with
    the per-channel gate, 128): the result stays inside the tolerance and is not worse than without the step -- down to the
    rounding floor of the step's own operands (its residual is formed from operands rounded to op_dtype, so a result that was
    more accurate than that, like the Neumann product's on a benign input, comes back at the floor)."""
    floor = {tri.F32: 1e-6, tri.F16: 3e-4, tri.BF16: 2e-3}[op]
    c = cases[idx]
    w, inp = c["w"], c["inp"]
    if idx == 4 and method == tri.NEUMANN:
        pytest.skip("Neumann product on the stress input: reported, not asserted")
    A32 = torch.from_numpy(c["A"].astype(np.float32))
    T32 = oracle.tri_inv(A32)
    e0 = check(tri.tri_inv_ex(A32.to(DEV), method=method, op_dtype=op), T32, TOL[op], "standalone", op=op, method=method)
    e1 = check(tri.tri_inv_ex(A32.to(DEV), method=method, op_dtype=op, flags=tri.FLAG_REFINE1), T32, TOL[op], "standalone + refine", op=op, method=method)
    assert e1 <= max(1.5 * e0, floor), (e0, e1)
    K, beta = inp["K"].to(DEV), inp["beta"].to(DEV)
    g = None if inp["g"] is None else inp["g"].to(DEV)
    if w.gate_kind == tri.GATE_PER_CHANNEL and w.C == 128:
        return
    f0 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=w.gate_kind, method=method, op_dtype=op), c["T"], TOL[op], "fused",
               op=op, key_abs=c["key_abs"], method=method)
    f1 = check(tri.gdn_chunk_tri_inv_ex(K, beta, g, w.C, gate_kind=w.gate_kind, method=method, op_dtype=op, flags=tri.FLAG_REFINE1),
               c["T"], TOL[op], "fused + refine", op=op, key_abs=c["key_abs"], method=method)
    assert f1 <= max(1.5 * f0, floor), (f0, f1)


def test_refinement_repairs_an_unconverged_newton_schulz():
    # six iterations leave Newton-Schulz far from converged at C = 64 (Sec. 4.2); one refinement step squares the residual
    inp = si.make_inputs(si.workload(1, Tlen=256, H=4))
    K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
    T_ref = oracle.gdn_chunk_tri_inv(inp["K"], inp["beta"], inp["g"], 0, 64)
    def err(flags):
        T = tri.gdn_chunk_tri_inv_ex(K, beta, g, 64, method=tri.NEWTON_SCHULZ, op_dtype=tri.F32, flags=flags)
        torch.cuda.synchronize()
        return metrics.forward_errors(T_ref, T.cpu().numpy().astype(np.float64))["rel_fro"].max()
    e8, e8r, e9 = err(tri.flag_iters(8)), err(tri.flag_iters(8) | tri.FLAG_REFINE1), err(tri.flag_iters(9))
    assert e8r < 0.5 * e8
    # a refinement step and a Newton-Schulz iteration both square the residual: they land in the same place
    assert e8r < 3 * e9 + 1e-6 and e9 < 3 * e8r + 1e-6, (e8, e8r, e9)


# ------------------------------------------------------------------ few heads: the chunk-strided workgroup map and its tail
@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 7])
@pytest.mark.parametrize("n_chunk", [1, 3, 4, 7, 16, 19, 33])
def test_few_heads_and_few_matrices_cover_every_matrix_once(H, n_chunk):
    """Up to 512 matrices a workgroup has one of them, in plain order."""
    assert n_chunk * H <= 512
    every_matrix_once(H, n_chunk, 64)


@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 7, 9])
@pytest.mark.parametrize("beyond,C", [(0, 32), (1, 32), (3, 64), (7, 32), (16, 16)])
def test_few_heads_workgroup_map_covers_every_matrix_once(H, beyond, C):
    """More than 512 matrices: H < 8 runs the map in which a workgroup takes one head of four chunks a stride apart; chunk counts that
    are not a multiple of the group size end in a plain-order tail.  (H = 9: four matrices in a row, no multiple of the heads.)"""
    every_matrix_once(H, 512 // H + 1 + beyond, C)


def every_matrix_once(H, n_chunk, C):
    """Every matrix must be written, with the right chunk's result, for the storing kernels (scalar and per-channel gate), the applied
    inverse and the packed-sequence layout."""
    d_k = 64
    for idx in (1, 3):
        w = si.workload(idx, B=1, Tlen=n_chunk * C - 5, H=H, C=C, d_k=d_k)
        inp = si.make_inputs(w)
        K, beta, g = inp["K"].to(DEV), inp["beta"].to(DEV), inp["g"].to(DEV)
        T_ref = oracle.gdn_chunk_tri_inv_ragged(inp["K"], inp["beta"], inp["g"], w.gate_kind, C)
        T = torch.full((n_chunk * H + 1, C, C), 7.0, device=DEV)
        tri.gdn_chunk_tri_inv_ex(K, beta, g, C, T=T[:-1], gate_kind=w.gate_kind)
        check(T[:-1], T_ref, 2e-2, f"H={H} n_chunk={n_chunk} cfg{idx}", key_abs=key_abs_term(inp, w.gate_kind, C))
        assert bool((T[-1] == 7.0).all())
        rhs = si.make_rhs(w, 64, torch.bfloat16)
        W = torch.full(rhs["X"].shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        tri.gdn_chunk_tri_solve(K, beta, g, rhs["X"].to(DEV), C, W=W, gate_kind=w.gate_kind)
        check_solve(W, oracle.gdn_chunk_tri_solve(inp["K"], inp["beta"], inp["g"], rhs["X"], None, w.gate_kind, C), 2e-2,
                    f"solve H={H} n_chunk={n_chunk} cfg{idx}", C=C)
    # packed sequences: the same tensors read as two sequences (a chunk more where both end inside one)
    w = si.workload(1, B=1, Tlen=n_chunk * C - 5, H=H, C=C, d_k=d_k)
    inp = si.make_inputs(w)
    total = w.Tlen
    seqlens = [total // 3, total - total // 3]
    g = torch.zeros(total, H)
    gen = torch.Generator().manual_seed(3)
    t0 = 0
    for n in seqlens:
        for c0 in range(0, n, C):
            m = min(C, n - c0)
            g[t0 + c0:t0 + c0 + m] = torch.cumsum(-0.05 * torch.rand(m, H, generator=gen), 0)
        t0 += n
    Kp, bp = inp["K"][0].contiguous(), inp["beta"][0].contiguous()
    T = tri.gdn_chunk_tri_inv_varlen(Kp.to(DEV), bp.to(DEV), g.to(DEV), seqlens, C)
    check(T, oracle.gdn_chunk_tri_inv_varlen(Kp, bp, g, seqlens, 0, C), 2e-2, f"varlen H={H} n_chunk={n_chunk}")
    X = torch.randn(total, H, 40, generator=gen).bfloat16()
    W = torch.full(X.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    tri.gdn_chunk_tri_solve_varlen(Kp.to(DEV), bp.to(DEV), g.to(DEV), X.to(DEV), seqlens, C, W=W)
    check_solve(W[None], oracle.gdn_chunk_tri_solve_varlen(Kp, bp, g, X, None, seqlens, 0, C)[None], 2e-2, f"solve varlen H={H} n_chunk={n_chunk}",
                C=C, seqlens=seqlens)
