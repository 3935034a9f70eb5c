"""Launch rules of the forward and the adjoint that change which kernel or which split
of the work runs, but not one bit of the results."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import native

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("L,E", [(1024, 8), (2048, 8), (4096, 8), (2048, 16), (4096, 16)])
def test_batch_smaller_than_the_grid(L, E):
    import torch
    import paper_1804_05335_amd as fd
    M, K = L // 8, 3
    specs = [syn.random_spectrum(L + b, n) for b, n in enumerate([L - M, 0, 5, 2 * (L - M) + 1])]
    T = syn.random_taps(M, K, M)
    bank = fd.prepare_bank(_dev(T), L)
    sd, od = fd.pack([_dev(a) for a in specs])
    first = None
    for grid in (5, 14, 15, 16, 0, 1000):         # 15 items; 0: the default, all of the device
        planes = fd.correlate_batched(sd, od, bank, K, M, L, E=E, grid=grid)
        first = planes if first is None else first
        assert torch.equal(planes, first), grid
    at = 0
    for a in specs:
        if len(a):
            ref = native.power(a, T)
            plane = first[K * at:K * (at + len(a))].view(K, -1).cpu().numpy()
            assert np.abs(plane - ref).max() <= TOL * ref.max()
        at += len(a)
