"""Candidates where a lane takes eight columns (more than 2048 workgroups of 256
columns), at row lengths around those workgroups' 2048 columns: every finite local
maximum, a NaN among the points, against the oracle."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N", [(2049, 255), (2049, 257), (683, 768), (683, 769), (257, 2047),
                                 (257, 2048), (257, 2049)])
def test_candidates_many_rows(K, N):
    import torch
    import paper_1804_05335_amd as fd
    P = syn.random_plane(N, K, N) - np.float32(0.5)
    P[K // 2, N // 2] = np.nan
    want = sorted(map(tuple, oh.peaks(P, -np.inf).tolist()))
    r, row, power, n = fd.candidates(torch.from_numpy(P).cuda(), N, K, 1, -np.inf, capacity=1 << 18)
    assert n == len(want) and sorted(zip(row.tolist(), r.tolist())) == want
    assert np.array_equal(power, P[row, r])
