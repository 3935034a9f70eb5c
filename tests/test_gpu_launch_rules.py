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


# template count K, tap counts with no, one and two dead slots at each end
@pytest.mark.parametrize("L,M", [(2048, 128), (2048, 256), (2048, 512), (4096, 256), (4096, 512),
                                 (4096, 1024)])
def test_templates_per_workgroup(L, M):
    import torch
    import paper_1804_05335_amd as fd
    K, N = 9, 3 * (L - M) + 17
    A, T = syn.random_spectrum(L + M, N), syn.random_taps(M, K, M)
    T[:4] = np.conj(T[5:][::-1])                  # T_{-z} = conj T_z for the symmetric bank
    T[4] = T[4].real
    half = syn.random_taps(M + 1, K, M + 2)
    a, bank = _dev(A), fd.prepare_bank(_dev(T), L)
    sym, bh = fd.prepare_bank_sym(_dev(T), L), fd.prepare_bank(_dev(half), L)
    items = 4 * K
    ref = native.power(A, T)
    # one template per workgroup, three, four (the first with turns), all in two
    for grid in (items, 12, 9, 2):
        got = {"plain": fd.correlate(a, bank, K, M, L, grid=grid),
               "interbin": fd.correlate_interbin(a, bank, K, M, L, grid=grid),
               "sym": fd.correlate_sym(a, sym, K, M, L, grid=grid),
               "two-bin": fd.correlate_fourier2(a, bank, bh, K, M, L, grid=grid)}
        if grid == items:
            first = got
            assert np.abs(got["plain"].cpu().numpy() - ref).max() <= TOL * ref.max()
            assert np.abs(got["sym"].cpu().numpy() - ref).max() <= TOL * ref.max()
            assert torch.equal(got["interbin"][:, ::2], got["plain"])
            for c, want in ((0, ref), (1, native.power(A, half))):
                plane = got["two-bin"][:, c::2].cpu().numpy()
                assert np.abs(plane - want).max() <= TOL * want.max()
        for name, plane in got.items():
            assert torch.equal(plane, first[name]), (name, grid)


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


@pytest.mark.parametrize("M,taps", [(512, False), (1024, False), (1024, True)])
def test_adjoint_plans_at_4096(M, taps):
    # the batch's planes have 2^25 points or more, each spectrum's fewer than 2^24
    import torch
    import paper_1804_05335_amd as fd
    L, K, lens = 4096, 801, [20000, 15001, 7000]
    assert K * sum(lens) >= 1 << 25 and K * max(lens) < 1 << 24
    g = torch.Generator(device="cuda").manual_seed(M)
    s = torch.randn(sum(lens), dtype=torch.complex64, device="cuda", generator=g)
    T = torch.randn(K, M, dtype=torch.complex64, device="cuda", generator=g) / M ** 0.5
    w = torch.rand(K * sum(lens), device="cuda", generator=g)
    bank = fd.prepare_bank(T, L)
    offs = torch.tensor([0] + list(np.cumsum(lens)), device="cuda")
    gs, gt = fd.correlate_backward_batched(s, offs, bank, K, M, L, w, want_taps=taps, zchunk=100)
    at, total = 0, 0
    for n in lens:
        one, t = torch.empty(n, dtype=torch.complex64, device="cuda"), None
        if taps:
            t = torch.empty(K, M, dtype=torch.complex64, device="cuda")
        ws = torch.empty(fd.fdas_backward_workspace_bytes(n, K, M, L, 100), dtype=torch.uint8,
                         device="cuda")
        fd.fdas_correlate_backward_ex(s[at:at + n], n, bank, K, M, L,
                                      w[K * at:K * (at + n)].view(K, n), one, t, 100, ws)
        assert torch.equal(one, gs[at:at + n])
        total = total + t if taps else 0
        at += n
    if taps:
        assert (gt - total).abs().max() <= TOL * total.abs().max()
