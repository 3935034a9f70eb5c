"""The batched fold chains on offsets that leave the planes (past the capacity,
negative, decreasing, overlapping), in the CPU emulation: the spectra are cut as
the batched correlation cuts them, and nothing outside the planes is read and
nothing outside the stated sums is written."""
import ctypes

import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh
from tests.test_fold_chain_emulated import _guarded, _intact, _p, _shape, emu  # noqa: F401

K, CAP = 9, 700


@pytest.mark.parametrize("offs", [[0, 300, 1500], [-200, 100, 650], [0, 690, 200, 900],
                                  [0, 700, 0, 700, 0, 700], [800, 900, 1000],
                                  [1 << 50, 1 << 51, -(1 << 50), 700]])
def test_offsets_are_clamped(emu, offs):  # noqa: F811
    n = len(offs) - 1
    cut = [(min(max(a, 0), CAP), min(max(a, 0), CAP) if b < min(max(a, 0), CAP) else min(b, CAP))
           for a, b in zip(offs, offs[1:])]
    # NaN on both sides of the planes: a read outside them would reach the sums
    room = np.full(K * (CAP + 3000), np.nan, dtype=np.float32)
    flat = room[K * 1500:K * (1500 + CAP)]
    flat[:] = syn.random_plane(CAP, K, CAP).reshape(-1)
    folds = [2, 4, 8]
    sizes = [_shape(0, K, H)[0] * (CAP // H + n) for H in folds]
    outs = [_guarded(s) for s in sizes]
    ptrs = (ctypes.c_void_p * len(folds))(*[o[1].ctypes.data for o in outs])
    nb = emu.fdas_harmonic_sums_batched_workspace_bytes(n)
    ws = np.zeros(nb, dtype=np.uint8)
    o = np.array(offs, dtype=np.int64)
    assert emu.fdas_harmonic_sums_batched(_p(flat), _p(o), n, ctypes.c_int64(CAP), K, 8, ptrs,
                                          _p(ws), ctypes.c_size_t(nb), None) == 0
    for H, size, (buf, out) in zip(folds, sizes, outs):
        assert _intact(buf, size)
        at, length, KH = 0, 0, _shape(0, K, H)[0]
        for a, b in cut:
            NH = -(-(b - a) // H)
            length += b - a
            if b > a and length <= CAP:
                plane = flat[K * a:K * b].reshape(K, b - a)
                want = oh.harmonic_sum(plane, H).reshape(-1)
                assert np.array_equal(out[KH * at:KH * (at + NH)], want), (H, a, b)
            at += NH
        assert np.all(np.isnan(out[KH * min(at, CAP // H + n):]))
