"""The chunk map (which tokens a chunk id stands for) on the host: csrc/chunk_map.hpp compiled with plain g++.
Paper Sec. 1: a sequence of L tokens is cut into ceil(L / C) chunks of at most C tokens."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def locate(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("chunk_map") / "chunk_map_host.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "host", "chunk_map_host.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.chunk_map_locate.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_void_p,
                                     ctypes.c_void_p, ctypes.c_uint32, ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int)]
    lib.chunk_map_locate_argument.argtypes = lib.chunk_map_locate.argtypes
    lib.chunk_map_locate_packed.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_uint32,
                                            ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int)]
    lib.chunk_map_locate_packed.restype = ctypes.c_bool

    def packed(words, C, lens, bc):
        tok0, valid = ctypes.c_int64(), ctypes.c_int()
        arr = np.ascontiguousarray(lens, dtype=np.int64)
        if not lib.chunk_map_locate_packed(words, C, sum(lens), len(lens), arr.ctypes.data, bc, ctypes.byref(tok0), ctypes.byref(valid)):
            return None
        return tok0.value, valid.value

    def call(C, total, cps, seqlens, chunks, bc):
        tok0, valid = ctypes.c_int64(), ctypes.c_int()
        if seqlens is None:
            lib.chunk_map_locate(C, total, cps, 0, None, None, bc, ctypes.byref(tok0), ctypes.byref(valid))
        else:
            s = np.ascontiguousarray(seqlens, dtype=np.int64)
            c = np.ascontiguousarray(chunks, dtype=np.int64)
            lib.chunk_map_locate(C, total, 0, len(s) - 1, s.ctypes.data, c.ctypes.data, bc, ctypes.byref(tok0), ctypes.byref(valid))
        return tok0.value, valid.value

    call.packed, call.argument = packed, lib.chunk_map_locate_argument
    return call


@pytest.mark.parametrize("C", [16, 32, 64, 128])
@pytest.mark.parametrize("Tlen", [1, 63, 64, 65, 300])
def test_fixed_layout(locate, C, Tlen):
    cps = -(-Tlen // C)
    for b in range(3):
        for k in range(cps):
            tok0, valid = locate(C, Tlen, cps, None, None, b * cps + k)
            assert tok0 == b * Tlen + k * C
            assert valid == min(C, Tlen - k * C)


@pytest.mark.parametrize("C", [32, 64, 128])
def test_packed_sequences_chunk_by_chunk(locate, C):
    lens = [5, 0, 200, C, 0, 0, 2 * C + 1, 1]
    seqlens = np.concatenate([[0], np.cumsum(lens)])
    chunks = np.concatenate([[0], np.cumsum([-(-n // C) for n in lens])])
    total = int(seqlens[-1])
    bc = 0
    for s, n in enumerate(lens):                      # walk the sequences the plain way
        for k in range(-(-n // C)):
            tok0, valid = locate(C, total, 0, seqlens, chunks, bc)
            assert tok0 == seqlens[s] + k * C and valid == min(C, n - k * C), (s, k)
            bc += 1
    assert bc == chunks[-1]


# 12 words: 384 bits.  The widest lengths that n_seq sequences may have, and the sizes around chunks.
@pytest.mark.parametrize("C", [16, 32, 64, 128])
@pytest.mark.parametrize("words, n_seq, bits", [(12, 1, 24), (12, 2, 24), (12, 16, 24), (12, 17, 22), (12, 24, 16), (12, 32, 12), (12, 33, 11), (12, 64, 6),
                                                (24, 32, 24), (24, 33, 23), (24, 48, 16), (24, 63, 12), (24, 64, 12)])
def test_lengths_in_the_arguments_give_the_chunks_of_the_offset_arrays(locate, C, words, n_seq, bits):
    rng = np.random.default_rng(n_seq * C)
    lens = [min(int(x), 2 ** bits - 1) for x in rng.choice([0, 1, C - 1, C, C + 1, 700], n_seq)]
    lens[n_seq // 2] = 2 ** bits - 1
    seqlens = np.concatenate([[0], np.cumsum(lens)])
    chunks = np.concatenate([[0], np.cumsum([-(-n // C) for n in lens])])
    last = int(chunks[-1]) - 1
    for bc in sorted({int(c) + d for c in chunks for d in (-1, 0, 1) if 0 <= c + d <= last} | {last // 3}):
        assert locate.packed(words, C, lens, bc) == locate(C, sum(lens), 0, seqlens, chunks, bc), bc
    for bc in (last + 1, 2 ** 31 - 1):                 # beyond the last: inside the buffers all the same
        tok0, valid = locate.packed(words, C, lens, bc)
        assert 0 <= tok0 and tok0 + valid <= sum(lens) and valid >= 1
    wider = lens[:-1] + [2 ** bits]
    assert (locate.packed(words, C, wider, 0) is None) == (bits == 24 or n_seq * (bits + 1) > 32 * words)
    assert locate.packed(words, C, [1] * 65, 0) is None and locate.packed(words, C, [5, -1], 0) is None and locate.packed(words, C, [], 0) is None


def test_the_other_layouts_as_kernel_arguments(locate):
    """More sequences than 16 bits count, a fixed layout, and addresses beyond 32 bits go through the argument's words unchanged."""
    n_seq = 70000
    seqlens = np.arange(n_seq + 1, dtype=np.int64) * 3
    chunks = np.arange(n_seq + 1, dtype=np.int64)
    tok0, valid = ctypes.c_int64(), ctypes.c_int()
    for bc in (0, 1, 65535, 65536, n_seq - 1):
        locate.argument(64, 3 * n_seq, 0, n_seq, seqlens.ctypes.data, chunks.ctypes.data, bc, ctypes.byref(tok0), ctypes.byref(valid))
        assert (tok0.value, valid.value) == (3 * bc, 3)
    for T, bc in ((2 ** 33 + 5, 3), (100, 5), (1, 0)):
        cps = -(-T // 128)
        locate.argument(128, T, cps, 0, None, None, bc, ctypes.byref(tok0), ctypes.byref(valid))
        assert (tok0.value, valid.value) == locate(128, T, cps, None, None, bc)


@pytest.mark.parametrize("C", [64, 128])
def test_surplus_chunk_ids_and_bad_offsets_stay_inside_the_buffers(locate, C):
    """Chunk ids at or beyond the last one, trailing empty sequences and offset arrays that disagree with each other must
    still give rows inside [0, total): the kernels read rows tok0 .. tok0 + valid - 1 without any further check."""
    lens = [70, 0, 3, 0, 0]
    seqlens = np.concatenate([[0], np.cumsum(lens)])
    chunks = np.concatenate([[0], np.cumsum([-(-n // C) for n in lens])])
    total = int(seqlens[-1])
    for bc in list(range(int(chunks[-1]), int(chunks[-1]) + 5)) + [10 ** 6, 2 ** 31 - 1]:
        tok0, valid = locate(C, total, 0, seqlens, chunks, bc)
        assert 0 <= tok0 and tok0 + valid <= total and 1 <= valid <= C, (bc, tok0, valid)
    rng = np.random.default_rng(7)
    for _ in range(500):                             # garbage offsets of every kind
        n_seq = int(rng.integers(1, 6))
        bad_s = rng.integers(-500, 500, size=n_seq + 1)
        bad_c = rng.integers(-5, 10, size=n_seq + 1)
        tot = int(rng.integers(1, 300))
        bc = int(rng.integers(0, 12))
        tok0, valid = locate(C, tot, 0, bad_s, bad_c, bc)
        assert 0 <= tok0 and tok0 + valid <= tot and 1 <= valid <= C, (bad_s, bad_c, tot, bc, tok0, valid)
