"""The transforms split over waves (eight values per lane, L = 1024 to 4096): the
strides of their LDS exchanges against gfx950's bank rules, on the CPU, and both
gradients and the batched forward that run on them, on the GPU, at tap counts
where a whole slot of lanes is lags (M/2 = L/8), at the smallest and the largest."""
import numpy as np
import pytest

import fdas_synth as syn
from oracle import native

STRIDE_A = {1: [36, 1, 2, 72, 140, 280], 2: [36, 72, 1, 2, 140, 280],
            3: [36, 72, 146, 1, 2, 286]}


def _sums(strides, groups):
    """Subset sums of the strides of an aligned group's lane bits."""
    out = np.zeros(1, dtype=np.int64)
    for s in strides[:groups]:
        out = np.concatenate([out, out + s])
    return out


@pytest.mark.parametrize("b", [1, 2, 3])
def test_exchange_strides(b):
    s = STRIDE_A[b]
    region_a = 572 if b == 3 else 560
    n = [4, 8, 16]
    # first exchange: every index of a region once, inside it; 16-lane groups of a
    # write distinct mod 16, 32-lane groups of a read distinct mod 32
    places = _sums(n + s, 9)
    assert len(set(places.tolist())) == 512 and places.max() < region_a
    assert len(set((_sums(s, 4) % 16).tolist())) == 16
    assert len(set((_sums(n + s[b:b + 3], 5) % 32).tolist())) == 32
    # second exchange: lanes n[2..0] p on the write, n[5..0] on the read
    places = _sums([1, 2, 4, 8, 16, 32, 72, 144, 288], 9)
    assert len(set(places.tolist())) == 512 and places.max() < 568
    assert len(set((_sums([1, 2, 4, 72], 4) % 16).tolist())) == 16


@pytest.mark.gpu
@pytest.mark.parametrize("L", [1024, 2048, 4096])
@pytest.mark.parametrize("taps", ["2", "L/4", "L/2"])
def test_gradients_and_batched_forward(L, taps):
    import torch
    import paper_1804_05335_amd as fd
    M = {"2": 2, "L/4": L // 4, "L/2": L // 2}[taps]
    K, B = 3, L - M
    lens = [2 * B + 13, 1, B]
    T = syn.random_taps(L + M, K, M)
    specs = [syn.random_spectrum(L + b, n) for b, n in enumerate(lens)]
    w = [np.random.default_rng(b).random((K, n), dtype=np.float32) for b, n in enumerate(lens)]
    bank = fd.prepare_bank(torch.from_numpy(T).cuda(), L)
    sd, od = fd.pack([torch.from_numpy(a) for a in specs])
    wd = torch.from_numpy(np.concatenate([x.reshape(-1) for x in w])).cuda()
    gs, gt = fd.correlate_backward_batched(sd, od, bank, K, M, L, wd)
    planes = fd.correlate_batched(sd, od, bank, K, M, L, E=8).cpu().numpy()
    refT, at = 0, 0
    for a, x in zip(specs, w):
        n = len(a)
        rA, rT = native.grads(a, T, x)
        refT = refT + rT
        got = gs[at:at + n].cpu().numpy()
        assert np.max(np.abs(got - rA)) <= 1e-5 * np.max(np.abs(rA))
        ref = native.power(a, T)
        plane = planes[K * at:K * (at + n)].reshape(K, n)
        assert np.max(np.abs(plane - ref)) <= 1e-5 * np.max(ref)
        at += n
    assert np.max(np.abs(gt.cpu().numpy() - refT)) <= 1e-5 * np.max(np.abs(refT))
