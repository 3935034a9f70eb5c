"""One fold by fdas_harmonic_sum on both sides of the rule that chooses its kernel,
from the plane and on top of the fold below, against the FP32 oracle in its
summation order (exact)."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import harmonic as oh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,folds", [
    (3, 1 << 10, (1, 2)), (1, (1 << 21) + 5, (2,)), (3, 1 << 20, (2,)),       # 2^21 points
    (1, (1 << 23) - 1, (1, 2)), (1, 1 << 23, (1, 2)),                         # 2^23 points
    (41, 131073, (4, 8, 16)),                   # 363 workgroups, then too few
    (85, 200003, (4, 8, 16, 32)),               # 16 from 256 workgroups on
    (257, 65529, (4,)), (257, 65537, (4,)),     # rows below and from 2^14 columns on
    (1, (1 << 22) - 32, (32,)), (1, 1 << 22, (32,)),                          # 2^17 points
    (1, 1 << 24, (32,)), (1, (1 << 24) + 1, (32,)),                           # 512 workgroups
    (65, 1400001, (32,)),                       # 129 workgroups in three rows
])
def test_one_fold(K, N, folds):
    import torch
    import paper_1804_05335_amd as fd
    P = syn.random_plane(N + K, K, N)
    Pd = torch.from_numpy(P).cuda()
    for H in folds:
        want = oh.harmonic_sum(P, H)
        out = torch.full(want.shape, float("nan"), device="cuda")
        fd.fdas_harmonic_sum(Pd, N, K, H, None, out)
        assert np.array_equal(out.cpu().numpy(), want), (H, "plane")
        if H > 1:
            below = torch.from_numpy(oh.harmonic_sum(P, H // 2)).cuda()
            out.fill_(float("nan"))
            fd.fdas_harmonic_sum(Pd, N, K, H, below, out)
            assert np.array_equal(out.cpu().numpy(), want), (H, "fold below")
