"""Batched candidates of many short spectra, on both sides of the rule that has each
lane take a column instead of a workgroup a chunk (more chunks than the 512
workgroups, under 256 columns each): every local maximum, empty spectra among them,
against the oracle spectrum by spectrum."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,nspec,n,H", [(7, 512, 60, 1), (7, 513, 60, 1), (7, 700, 255, 1),
                                         (7, 700, 257, 1), (5, 1500, 90, 2), (9, 2500, 70, 4)])
def test_short_spectra(K, nspec, n, H):
    import torch
    import paper_1804_05335_amd as fd
    lens = [0 if b % 97 == 5 else n + b % 3 - 1 for b in range(nspec)]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    planes = [syn.random_plane(b, K, m) for b, m in enumerate(lens)]
    folds = [oh.harmonic_sum(p, H) if H > 1 else p for p in planes]
    want = set()
    for b, S in enumerate(folds):
        shift = (K - 1) // 2 - (S.shape[0] - 1) // 2
        want |= {(b, r, row + shift) for row, r in oh.peaks(S, -1.0).tolist()} if S.size else set()
    sums = torch.from_numpy(np.concatenate([f.reshape(-1) for f in folds])).cuda()
    b, r, row, power, count = fd.candidates_batched(sums, torch.from_numpy(offs).cuda(), K, H, -1.0,
                                                    capacity=1 << 20)
    assert count == len(want) and set(zip(b.tolist(), r.tolist(), row.tolist())) == want
