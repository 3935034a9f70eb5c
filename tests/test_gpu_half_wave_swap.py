"""Segments whose last pass takes its values by lane swaps.  L = 8192: the plain and
batched planes against the interbinned one, which exchanges through LDS with the same
arithmetic and so must agree bit for bit, and both gradients against the FP64 oracle,
at the smallest, the headline and the largest tap counts.  L = 1024: the plain,
interbinned and two-bin planes against the FP64 oracle."""
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


@pytest.mark.parametrize("M", [2, 126, 128, 256, 512])
def test_swapped_rows(M):
    import torch
    import paper_1804_05335_amd as fd
    L1, K = 1024, 3
    n = 2 * (L1 - M) + 13
    a, taps = syn.random_spectrum(M, n), syn.random_taps(L1 + M, K, M)
    half = syn.random_taps(M, K, M + 2)
    dev = torch.from_numpy(a).cuda()
    bank = fd.prepare_bank(torch.from_numpy(taps).cuda(), L1)
    ref = native.power(a, taps)
    plane = fd.correlate(dev, bank, K, M, L1)
    assert np.abs(plane.cpu().numpy() - ref).max() <= 1e-5 * ref.max()
    assert torch.equal(fd.correlate_interbin(dev, bank, K, M, L1)[:, ::2], plane)
    if M + 2 <= L1 // 2:
        both = fd.correlate_fourier2(dev, bank, fd.prepare_bank(torch.from_numpy(half).cuda(), L1),
                                     K, M, L1)
        # segments of L - M - 2 outputs: the even columns round differently from plane
        for got, want in ((both[:, ::2], ref), (both[:, 1::2], native.power(a, half))):
            assert np.abs(got.cpu().numpy() - want).max() <= 1e-5 * want.max()
