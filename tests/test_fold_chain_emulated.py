"""The fold chains (all harmonic folds in one launch, single plane and batch)
in the CPU emulation, against the FP32 oracle in its summation order: lengths
around the chunk of 256 columns and its octaves, and row counts around the
batch's groups of four rows; every output inside sentinel guards."""
import ctypes

import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh

GUARD = 4096


@pytest.fixture(scope="module")
def emu():
    from tests.emu import build_emu
    L = ctypes.CDLL(build_emu.build())
    L.fdas_harmonic_sums_batched_workspace_bytes.restype = ctypes.c_size_t
    return L


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _guarded(n):
    buf = np.full(n + 2 * GUARD, -12345.0, dtype=np.float32)
    buf[GUARD:GUARD + n] = np.nan
    return buf, buf[GUARD:GUARD + n]


def _intact(buf, n):
    return np.all(buf[:GUARD] == -12345.0) and np.all(buf[GUARD + n:] == -12345.0)


def _shape(N, K, H):
    return 2 * ((K - 1) // 2 // H) + 1, -(-N // H)


@pytest.mark.parametrize("K,N,top", [(1, 1, 64), (3, 255, 2), (5, 511, 4), (9, 513, 8),
                                     (17, 1025, 16), (7, 2049, 64), (65, 700, 64)])
def test_fold_chain(emu, K, N, top):
    P = syn.random_plane(N + top, K, N)
    folds = [H for H in (2, 4, 8, 16, 32, 64) if H <= top]
    outs = [_guarded(int(np.prod(_shape(N, K, H)))) for H in folds]
    ptrs = (ctypes.c_void_p * len(folds))(*[o[1].ctypes.data for o in outs])
    assert emu.fdas_harmonic_sums(_p(P), ctypes.c_int64(N), K, top, ptrs, None) == 0
    for H, (buf, out) in zip(folds, outs):
        assert _intact(buf, out.size)
        assert np.array_equal(out.reshape(_shape(N, K, H)), oh.harmonic_sum(P, H)), H


@pytest.mark.parametrize("K", [1, 7, 9, 19])
def test_fold_chain_batched(emu, K):
    lens = [0, 1, 513, 300, 0, 1100]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    planes = [syn.random_plane(7 + b, K, n) for b, n in enumerate(lens)]
    flat = np.concatenate([p.reshape(-1) for p in planes]).astype(np.float32)
    folds = [2, 4, 8, 16]
    sizes = [_shape(0, K, H)[0] * sum(-(-n // H) for n in lens) for H in folds]
    outs = [_guarded(n) for n in sizes]
    ptrs = (ctypes.c_void_p * len(folds))(*[o[1].ctypes.data for o in outs])
    nb = emu.fdas_harmonic_sums_batched_workspace_bytes(len(lens))
    ws = np.zeros(nb, dtype=np.uint8)
    assert emu.fdas_harmonic_sums_batched(_p(flat), _p(offs), len(lens),
                                          ctypes.c_int64(flat.size // K), K, 16, ptrs, _p(ws),
                                          ctypes.c_size_t(nb), None) == 0
    for H, (buf, out) in zip(folds, outs):
        assert _intact(buf, out.size)
        ref = np.concatenate([oh.harmonic_sum(p, H).reshape(-1) for p in planes])
        assert np.array_equal(out, ref), H
