"""The fold chains on the GPU against the FP32 oracle in its summation order
(exact): lengths around the chunk of 256 columns and its octaves, row counts
around the batch's groups of four rows, up to 64 harmonics."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fd():
    import torch
    assert torch.cuda.is_available()
    import paper_1804_05335_amd as fdas
    return fdas


@pytest.mark.parametrize("K,N,top", [(1, 1, 64), (3, 255, 2), (5, 511, 4), (9, 513, 8),
                                     (17, 1025, 16), (7, 65537, 64), (65, 70001, 64),
                                     (129, 20000, 64)])
def test_fold_chain(fd, K, N, top):
    import torch
    P = syn.random_plane(N + top, K, N)
    Pd = torch.from_numpy(P).cuda()
    folds = fd.harmonic_sums(Pd, top)
    H = 2
    for S in folds[1:]:
        assert np.array_equal(S.cpu().numpy(), oh.harmonic_sum(P, H)), H
        one = torch.empty_like(S)
        fd.fdas_harmonic_sum(Pd, N, K, H, None, one)
        assert torch.equal(one, S), H
        H *= 2
    assert H == 2 * top


@pytest.mark.parametrize("K,lens", [(1, [5, 0, 700]), (7, [0, 1, 513, 300, 0, 1100]),
                                    (85, [65537, 3, 40000]), (19, [257] * 300)])
def test_fold_chain_batched(fd, K, lens):
    import torch
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    planes = [syn.random_plane(7 + b, K, n) for b, n in enumerate(lens)]
    flat = torch.from_numpy(np.concatenate([p.reshape(-1) for p in planes])).cuda()
    folds = fd.harmonic_sums_batched(flat, torch.from_numpy(offs).cuda(), K, 32)
    for i, S in enumerate(folds[1:], 1):
        ref = np.concatenate([oh.harmonic_sum(p, 1 << i).reshape(-1) for p in planes])
        assert np.array_equal(S.cpu().numpy()[:ref.size], ref), 1 << i


@pytest.mark.parametrize("N", [1, 2047, 2048, 2049, 4097])
def test_candidates_at_chunk_edges(fd, N):
    # lengths around the 2048 columns of a workgroup, negative powers and a
    # threshold of -inf included (every finite local maximum), one NaN
    import torch
    K = 3
    P = syn.random_plane(N, K, N) - np.float32(0.5)
    if N > 2:
        P[1, N // 2] = np.nan
    want = sorted(map(tuple, oh.peaks(P, -np.inf).tolist()))
    r, row, power, n = fd.candidates(torch.from_numpy(P).cuda(), N, K, 1, -np.inf, capacity=1 << 16)
    assert n == len(want) > 0 and sorted(zip(row.tolist(), r.tolist())) == want
    offs = torch.tensor([0, N, 2 * N], device="cuda")
    flat = torch.from_numpy(np.concatenate([P.reshape(-1)] * 2)).cuda()
    spec, r, row, power, n = fd.candidates_batched(flat, offs, K, 1, -np.inf, capacity=1 << 16)
    assert n == 2 * len(want)
    for b in (0, 1):
        assert sorted(zip(row[spec == b].tolist(), r[spec == b].tolist())) == want
