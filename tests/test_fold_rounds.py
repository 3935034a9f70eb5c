"""The fold chains over several full rounds of the deal to the eight XCDs plus a
remainder, single plane and batch, against the FP32 oracle in its summation order
(exact): in the CPU emulation with runs of 2 chunks, every output inside sentinel
guards, and on the GPU with the kernel's runs."""
import ctypes

import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh
from tests.test_fold_chain_emulated import _guarded, _intact, _p, _shape, emu  # noqa: F401


# 16 places a round of two runs: 35 chunks (two rounds and 3), 16, 31
@pytest.mark.parametrize("K,N,top", [(3, 2 * 256 * 34 + 11, 64), (5, 2 * 256 * 34 + 11, 4),
                                     (3, 2 * 256 * 16, 2), (9, 2 * 256 * 31 - 1, 8)])
def test_rounds_emulated(emu, K, N, top):  # noqa: F811
    P = syn.random_plane(N, K, N)
    folds = [1 << i for i in range(1, top.bit_length())]
    outs = [_guarded(int(np.prod(_shape(N, K, H)))) for H in folds]
    ptrs = (ctypes.c_void_p * len(folds))(*[o[1].ctypes.data for o in outs])
    assert emu.fdas_harmonic_sums(_p(P), ctypes.c_int64(N), K, top, ptrs, None) == 0
    for H, (buf, out) in zip(folds, outs):
        assert _intact(buf, out.size)
        assert np.array_equal(out.reshape(_shape(N, K, H)), oh.harmonic_sum(P, H)), H


@pytest.mark.parametrize("K,lens", [(3, [2 * 256 * 34 + 11, 5, 2 * 256 * 17]), (5, [17000, 0, 9])])
def test_rounds_batched_emulated(emu, K, lens):  # noqa: F811
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    planes = [syn.random_plane(b, K, n) for b, n in enumerate(lens)]
    flat = np.concatenate([p.reshape(-1) for p in planes]).astype(np.float32)
    folds = [2, 4, 8, 16, 32, 64]
    outs = [_guarded(_shape(0, K, H)[0] * sum(-(-n // H) for n in lens)) for H in folds]
    ptrs = (ctypes.c_void_p * len(folds))(*[o[1].ctypes.data for o in outs])
    nb = emu.fdas_harmonic_sums_batched_workspace_bytes(len(lens))
    ws = np.zeros(nb, dtype=np.uint8)
    assert emu.fdas_harmonic_sums_batched(_p(flat), _p(offs), len(lens),
                                          ctypes.c_int64(flat.size // K), K, 64, ptrs, _p(ws),
                                          ctypes.c_size_t(nb), None) == 0
    for H, (buf, out) in zip(folds, outs):
        assert _intact(buf, out.size)
        ref = np.concatenate([oh.harmonic_sum(p, H).reshape(-1) for p in planes])
        assert np.array_equal(out, ref), H


# 256 places a round of eight runs of 32 chunks: 586 and 257 chunks of fold 2
@pytest.mark.gpu
@pytest.mark.parametrize("K,lens", [(7, [300001, 5, 131073]), (9, [263169])])
def test_rounds_batched(K, lens):
    import torch
    import paper_1804_05335_amd as fd
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    planes = [syn.random_plane(b, K, n) for b, n in enumerate(lens)]
    flat = torch.from_numpy(np.concatenate([p.reshape(-1) for p in planes])).cuda()
    folds = fd.harmonic_sums_batched(flat, torch.from_numpy(offs).cuda(), K, 64)
    for i, S in enumerate(folds[1:], 1):
        ref = np.concatenate([oh.harmonic_sum(p, 1 << i).reshape(-1) for p in planes])
        assert np.array_equal(S.cpu().numpy(), ref), 1 << i
