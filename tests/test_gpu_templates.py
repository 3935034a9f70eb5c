"""Device templates and bank rows (FP64 on the GPU): the templates equal the
host's bit for bit, and the bank equals an FP64 FFT of the placed taps, at the
edges of the bank kernel's groups of eight taps and of eight rows."""
import numpy as np
import pytest

import fdas_synth as syn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fd():
    import torch
    assert torch.cuda.is_available()
    import paper_1804_05335_amd as fdas
    return fdas


@pytest.mark.parametrize("zmax,dz,M", [(0.0, 2.0, 2), (20.0, 2.0, 64), (84.0, 2.0, 254),
                                       (200.0, 2.0, 512), (3.0, 0.5, 34), (1.25, 0.05, 1000),
                                       (0.003, 0.001, 62), (1000.0, 8.0, 4096)])
def test_device_templates_equal_host(fd, zmax, dz, M):
    import torch
    K = fd.fdas_num_templates(zmax, dz)
    taps = torch.empty(K * M, dtype=torch.complex64, device="cuda")
    fd.fdas_make_templates(zmax, dz, M, 0, taps)
    assert np.array_equal(taps.cpu().numpy().reshape(K, M), fd.fdas_make_templates_host(zmax, dz, M))


def test_device_half_bin_templates_equal_host(fd):
    zmax, dz, M = 40.0, 2.0, 126
    taps, _ = fd.make_bank_half(zmax, dz, M, 512)
    T = taps.cpu().numpy()
    K = T.shape[0]
    assert T.shape == (K, M + 2) and not T[:, :2].any()
    for k in (0, 1, K // 2, K - 1):
        z = (k - 0.5 * (K - 1)) * dz
        ref = np.array([fd.fdas_template_response(0.5 - (j - (M + 2) // 2), z)
                        for j in range(2, M + 2)]).astype(np.complex64)
        assert np.array_equal(T[k, 2:], ref)


@pytest.mark.parametrize("L,M", [(L, M) for L in (256, 512, 1024, 8192)
                                 for M in (2, 6, 8, 10, 62, 128)] +
                         [(2048, 512), (2048, 514), (8192, 4096)])
def test_bank_rows_at_group_edges(fd, L, M):
    import torch
    K = 3
    taps = syn.random_taps(L + M, K, M)
    bank = fd.prepare_bank(torch.from_numpy(taps).cuda(), L).cpu().numpy().reshape(K + 1, L)
    h = np.zeros((K, L), dtype=np.complex128)
    for j in range(M):
        h[:, (M // 2 - j) % L] = np.conj(taps[:, j].astype(np.complex128))
    H = np.fft.fft(h, axis=1) / L
    # FP64 values rounded once per component: 2^-24 sqrt(2) of the largest
    assert np.max(np.abs(bank[:K] - H)) <= 9e-8 * np.max(np.abs(H))
    tw = np.exp(-2j * np.pi * np.arange(L) / L)
    assert np.max(np.abs(bank[K] - tw)) <= 9e-8
