"""The binding's native argument handling (csrc/fastcall.cpp) without a GPU: host tensors (device -1) and a stand-in for the C-ABI that
records the calls it gets."""
import ctypes
import importlib.util
import os
import shutil
import sys
import types

import pytest
import torch

import paper_2605_21325_amd as tri
from paper_2605_21325_amd import build as tri_build

# as in csrc/fastcall.cpp, struct Abi
P, I, L, U = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_uint32
ABI = {
    "tri_inv_ex": (P, P, L, I, I, I, I, P, U),
    "inv_ex": (P, P, P, P, I, L, I, I, I, I, I, I, I, P, U),
    "inv_varlen": (P, P, P, P, P, P, I, L, L, I, I, I, I, I, I, I, P, U),
    "solve_multi": (P, P, P, I, P, P, P, P, I, L, I, I, I, I, I, I, I, P, U),
    "solve_varlen": (P, P, P, P, P, P, P, P, I, L, L, I, I, I, I, I, I, I, I, P, U),
    "offsets": (P, I, I, L, P, P, P),
}


class Native:
    """The module, connected to the stand-in.  calls: (function, arguments) as they arrive; status: what the stand-in answers."""
    def __init__(self, path):
        spec = importlib.util.spec_from_file_location("_fastcall", path)
        self.module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.module)
        self.calls, self.status, self.keep = [], 0, []
        for name, types in ABI.items():
            self.keep.append(ctypes.CFUNCTYPE(I, *types)(lambda *a, name=name: self.answer(name, a)))
        self.module.connect(*(ctypes.cast(f, P).value for f in self.keep))

    def answer(self, name, args):
        self.calls.append((name, args))
        if name == "offsets":
            lens, n, C, total, _, n_chunk, _ = args
            lens = ctypes.cast(lens, ctypes.POINTER(L))[:n]
            if sum(lens) != total:
                return -5
            ctypes.cast(n_chunk, ctypes.POINTER(L))[0] = sum(-(-x // C) for x in lens)
            return 0
        return self.status


@pytest.fixture
def native(tmp_path):
    if not tri_build._fastcall_current():
        tri_build.build_fastcall()
    copy = str(tmp_path / "_fastcall.so")  # a copy: the module a process has connected to the library stays as it is
    shutil.copy(tri_build.FASTCALL, copy)
    return Native(copy)


def tri_inv(n, A, T=None, method=1, op=None, flags=0, out=None):
    return n.module.tri_inv(-1, 0, A, T, method, op, flags, out)


def gdn_inv(n, K, beta, g, C=64, T=None):
    return n.module.gdn_inv(-1, 0, K, beta, g, C, T, tri.GATE_SCALAR, 1, tri.BF16, 0, None)


def keys(*shape):
    return torch.randn(*shape).bfloat16(), torch.rand(shape[:-1]), -torch.rand(shape[:-1])


def nested(*shapes, dtype=torch.float32):
    return torch.nested.nested_tensor([torch.randn(s, dtype=dtype) for s in shapes])


def test_plain_calls_reach_the_library(native):
    A = torch.randn(3, 64, 64)
    T = tri_inv(native, A, op=tri.F32)
    assert T.shape == A.shape and T.dtype == torch.float32
    (name, a), = native.calls
    assert (name, a[0], a[1], a[2:7]) == ("tri_inv_ex", A.data_ptr(), T.data_ptr(), (3, 64, tri.F32, 1, tri.F32))
    K, beta, g = keys(2, 130, 4, 64)
    assert gdn_inv(native, K, beta, g).shape == (24, 64, 64)
    native.status = -9  # refused: None, and the Python route reports it
    assert tri_inv(native, A, op=tri.F32) is None


# libtorch throws when a nested tensor is asked for a size: nothing of that may reach the interpreter as a C++ exception (it ends the
# process), and no nested tensor is taken, whatever its parts' shapes.
@pytest.mark.filterwarnings("ignore:The PyTorch API of nested tensors")
@pytest.mark.parametrize("shapes", [((64, 64), (32, 32)), ((64, 64), (64, 64))], ids=["ragged", "uniform"])
def test_nested_tensors_are_left_to_the_python_route(native, shapes):
    assert tri_inv(native, nested(*shapes), op=tri.F32) is None
    assert tri_inv(native, torch.randn(2, 64, 64), T=nested(*shapes), op=tri.F32) is None
    K, beta, g = keys(2, 130, 4, 64)
    ragged = nested((130, 4, 64), (shapes[1][0] + 66, 4, 64), dtype=torch.bfloat16)
    assert gdn_inv(native, ragged, beta, g) is None
    solve = lambda K, X, W=None: native.module.gdn_solve(-1, 0, K, beta, g, (X,), 64, None, None if W is None else (W,), 0, 1, 0)
    assert solve(K, ragged) is None and solve(ragged, K) is None and solve(K, K, ragged) is None
    packed = nested((100, 64), (shapes[1][0] + 36, 64), dtype=torch.bfloat16)
    assert native.module.gdn_inv_varlen(-1, 0, packed, beta, g, [200], 64, None, 0, 1, 2, 0, None) is None
    P, b = torch.randn(200, 4, 64).bfloat16(), torch.rand(200, 4)
    assert native.module.gdn_solve_varlen(-1, 0, P, b, b, packed, [200], 64, None, None, 0, 1, 0) is None
    assert native.module.gdn_solve_varlen(-1, 0, P, b, b, P, [200], 64, None, packed, 0, 1, 0) is None
    assert not native.calls


@pytest.mark.filterwarnings("ignore")
def test_tensors_of_a_functional_transform_are_left_to_the_python_route(native):
    A, seen = torch.randn(2, 3, 64, 64), []
    torch.func.vmap(lambda a: (seen.append(tri_inv(native, a, op=tri.F32)), a)[1])(A)
    torch.func.jvp(lambda a: (seen.append(tri_inv(native, a, op=tri.F32)), a)[1], (A[0],), (A[0],))
    assert seen == [None, None] and not native.calls


# Only None asks for the matrices' own type; every number goes to the library, which refuses those that name no type.
def test_operand_type_of_given_matrices(native):
    A = torch.randn(2, 64, 64).bfloat16()
    for op, want in ((None, tri.BF16), (tri.F32, tri.F32), (-1, -1), (-7, -7), (3, 3)):
        native.calls.clear()
        tri_inv(native, A, op=op)
        assert native.calls[0][1][6] == want


# The short forms write fp32, so neither route takes a T of 16-bit elements (the Python route would write past its end).
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_short_forms_refuse_a_result_of_16_bits(monkeypatch, native, dtype):
    A = torch.randn(2, 64, 64)
    K, beta, g = keys(1, 128, 2, 64)
    T = torch.zeros(4, 64, 64, dtype=dtype)
    answers = []

    class Watch:  # as the binding calls it, for host tensors
        def __getattr__(self, name):
            def call(dev, stream, *a):
                answers.append(getattr(native.module, name)(-1, 0, *a))
                return answers[-1]
            return call

    monkeypatch.setattr(tri.binding, "_fast", Watch())
    monkeypatch.setattr(tri.binding, "_fast_lib", tri.binding._lib)
    monkeypatch.setattr(tri.binding, "_device_index", lambda: 0)
    monkeypatch.setattr(torch.Tensor, "is_cuda", property(lambda t: True))
    for call in (lambda: tri.tri_inv(A, T=T[:2]), lambda: tri.gdn_chunk_tri_inv(K, beta, g, 64, T=T)):
        with pytest.raises(TypeError, match="writes fp32"):
            call()
    assert answers == [None, None] and not native.calls


# The library does not need the native argument handling: where that does not compile, the build says so and links the library.
def test_the_library_is_built_without_the_native_argument_handling(monkeypatch, tmp_path):
    done = []
    monkeypatch.setattr(tri_build, "FASTCALL", str(tmp_path / "_fastcall.so"))
    open(tri_build.FASTCALL, "w").close()
    os.utime(tri_build.FASTCALL, (0, 0))
    monkeypatch.setattr(tri_build, "LIB", str(tmp_path / "libtriinv.so"))
    monkeypatch.setattr(tri_build, "RESOURCES", str(tmp_path / "resources.json"))
    monkeypatch.setattr(tri_build, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(tri_build, "HIPCC", "true")  # the link
    monkeypatch.setattr(tri_build, "_compile", lambda unit: (done.append(unit), (str(tmp_path / "unit.o"), {}))[1])
    monkeypatch.setenv("CXX", "false")
    with pytest.warns(UserWarning, match="native argument handling is not built"):
        assert tri_build.build() == tri_build.LIB
    assert len(done) == len(tri_build.UNITS) and not os.path.exists(tri_build.FASTCALL)  # (one of older sources is not left either)
    open(tri_build.LIB, "w").close()
    with pytest.warns(UserWarning, match="native argument handling is not built"):
        tri_build.build()
    assert len(done) == len(tri_build.UNITS)  # the library is current: it is not compiled again


# The module reads Python's and torch's objects as their headers lay them out: one of another build is neither connected nor kept.
def test_a_module_built_for_another_torch_is_not_used(monkeypatch, native):
    module = types.ModuleType("paper_2605_21325_amd._fastcall")
    module.connect = lambda *a: connected.append(a)
    connected = []
    monkeypatch.setattr(tri, "_fastcall", module, raising=False)
    monkeypatch.setitem(sys.modules, module.__name__, module)
    for name, value in (("_raw_stream", int), ("_device_index", int), ("_fast", None), ("_fast_lib", None)):
        monkeypatch.setattr(tri.binding, name, value)
    for stamp, taken in ((None, False), (tri_build.fastcall_stamp() + "1", False), (native.module.BUILT_FOR, True)):
        module.BUILT_FOR = stamp
        tri.binding._connect(tri.lib())
        assert bool(connected) == taken and (tri.binding._fast is module) == taken, stamp
    assert tri_build._fastcall_current()
    monkeypatch.setattr(torch.version, "git_version", "another")
    assert not tri_build._fastcall_current()


# Up to 64 sequences are offered to the library by their lengths; what it does not take, and everything else, goes by offsets.
@pytest.mark.parametrize("lens, taken, as_lengths", [([130, 0, 70], True, True), ([1] * 64, True, True), ([1] * 65, True, False), ([65536], False, False),
                                                     ([100, 101], True, None)])
def test_packed_sequences_by_lengths_or_offsets(native, lens, taken, as_lengths):
    extra = {"inv_packed": (P, P, P, P, P, I, L, I, I, I, I, I, I, I, P, U), "solve_packed": (P, P, P, P, P, P, P, I, L, I, I, I, I, I, I, I, I, P, U)}
    def answer(name, a):
        native.calls.append((name, a))
        return 0 if taken else -5
    for name, types in extra.items():
        native.keep.append(ctypes.CFUNCTYPE(I, *types)(lambda *a, name=name: answer(name, a)))
    native.module.connect(*(ctypes.cast(f, P).value for f in native.keep))
    total = 200 if as_lengths is None else sum(lens)
    K, beta, _ = keys(total, 1, 32)
    X = torch.randn(total, 1, 8).bfloat16()
    T = native.module.gdn_inv_varlen(-1, 0, K, beta, None, lens, 64, None, tri.GATE_NONE, 1, tri.BF16, 0, None)
    W = native.module.gdn_solve_varlen(-1, 0, K, beta, None, X, lens, 64, None, None, tri.GATE_NONE, 1, 0)
    if as_lengths is None:
        assert T is None and W is None
        return
    assert T.shape == (sum(-(-n // 64) for n in lens), 64, 64) and W.shape == X.shape
    assert hasattr(T, "_triinv_keepalive") and hasattr(W, "_triinv_keepalive")
    offered = len(lens) <= 64
    want = (["inv_packed"] * offered + ([] if as_lengths else ["offsets", "inv_varlen"]) + ["solve_packed"] * offered
            + ([] if as_lengths else ["offsets", "solve_varlen"]))
    assert [name for name, _ in native.calls] == want
    if as_lengths:
        (_, a), (_, b) = native.calls
        assert a[5:9] == (len(lens), total, 1, 32) and b[7:11] == (len(lens), total, 1, 32) and b[11:13] == (8, 64)
        assert (a[0], b[0], b[3], b[5]) == (K.data_ptr(), K.data_ptr(), X.data_ptr(), W.data_ptr())
