"""Segments of 8192, whose last pass takes its values by half-wave swaps: the plain
and batched planes against the interbinned one, which exchanges
through LDS with the same arithmetic and so must agree bit for bit, and both
gradients against the FP64 oracle, at the smallest, the headline and the largest
tap counts."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import native

pytestmark = pytest.mark.gpu
L = 8192


@pytest.mark.parametrize("M", [2, 500, 512, 1024, 4096])
def test_swapped_last_pass(M):
    import torch
    import paper_1804_05335_amd as fd
    K, B = 3, L - M
    lens = [2 * B + 13, 1, B]
    specs = [syn.random_spectrum(M + b, n) for b, n in enumerate(lens)]
    taps = syn.random_taps(L + M, K, M)
    dev = [torch.from_numpy(a).cuda() for a in specs]
    bank = fd.prepare_bank(torch.from_numpy(taps).cuda(), L)
    ib = [fd.correlate_interbin(a, bank, K, M, L)[:, ::2] for a in dev]
    sd, od = fd.pack(dev)
    planes, at = fd.correlate_batched(sd, od, bank, K, M, L, E=16), 0
    for a, ref in zip(dev, ib):
        n = a.numel()
        assert torch.equal(fd.correlate(a, bank, K, M, L), ref)
        assert torch.equal(planes[at:at + K * n].view(K, n), ref)
        at += K * n

    # both gradients: 1e-5 of the largest, the bound at every other segment length
    w = [np.random.default_rng(M + b).random((K, n), dtype=np.float32)
         for b, n in enumerate(lens)]
    wd = torch.from_numpy(np.concatenate([x.reshape(-1) for x in w])).cuda()
    gA, gT = fd.correlate_backward_batched(sd, od, bank, K, M, L, wd)
    ref = [native.grads(a, taps, x) for a, x in zip(specs, w)]
    rT, at = sum(r[1] for r in ref), 0
    for a, (rA, _) in zip(specs, ref):
        got = gA[at:at + len(a)].cpu().numpy()
        assert np.abs(got - rA).max() <= 1e-5 * np.abs(rA).max()
        at += len(a)
    assert np.abs(gT.cpu().numpy() - rT).max() <= 1e-5 * np.abs(rT).max()
