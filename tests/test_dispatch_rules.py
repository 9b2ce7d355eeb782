"""The launch rules on the host: csrc/dispatch.hpp compiled with plain g++, nothing launched."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2605_21325_amd as tri

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
LAUNCHED, NOT_BUILT = 0, 1


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("dispatch") / "dispatch_host.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    os.path.join(HERE, "host", "dispatch_host.cpp"), "-o", so, f"-L{ROCM}/lib", "-lamdhip64"], check=True)
    lib = ctypes.CDLL(so)
    lib.dispatch_launched.argtypes = [ctypes.c_int, ctypes.c_bool, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_int64]
    lib.dispatch_lengths_in_arguments.argtypes = [ctypes.c_int, ctypes.c_bool]
    lib.dispatch_lengths_in_arguments.restype = ctypes.c_bool
    return lib


# words: 0 the kernels with offset arrays in memory, 12 the storing kernels, 24 those that apply the inverse to one right-hand side
@pytest.mark.parametrize("lens, fits", [([5, 70], (12, 24)), ([(1 << 24) - 1] * 16, (12, 24)), ([(1 << 24) - 1] * 17, (24,)),
                                        ([700] * 64, (24,)), ([(1 << 24) - 1] * 33, ()), ([1] * 65, ()), ([1 << 24], ())])
@pytest.mark.parametrize("words", [0, 12, 24])
def test_a_kernel_that_cannot_be_given_the_lengths_is_not_launched(rules, words, lens, fits):
    a = np.array(lens, dtype=np.int64)
    assert rules.dispatch_launched(words, True, a.ctypes.data, len(lens), int(a.sum())) == (LAUNCHED if words in fits else NOT_BUILT)
    assert rules.dispatch_launched(words, False, a.ctypes.data, len(lens), int(a.sum())) == LAUNCHED  # (offset arrays go with every kernel)


def test_methods_whose_kernels_take_offsets_alone(rules):
    for method in range(7):
        assert rules.dispatch_lengths_in_arguments(method, False) == (method not in (tri.NEUMANN, tri.MIXED_B32))
        assert not rules.dispatch_lengths_in_arguments(method, True)
