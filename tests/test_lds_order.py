"""The transforms of every plan on the CPU, with the lane swaps and every LDS access
recorded: accesses of different lanes to one place, one of them a write, have a
barrier or a wave fence between them, within a transform and from one transform to
the next, and the transforms' values are those of FP64."""
import ctypes

import numpy as np
import pytest

PLANS = [(256, 4), (512, 8), (1024, 8), (1024, 16), (2048, 8), (2048, 16), (4096, 8),
         (4096, 16), (8192, 8), (8192, 16)]


@pytest.fixture(scope="module")
def lib():
    from tests.emu import build_emu
    L = ctypes.CDLL(build_emu.build_lds_order())
    L.emu_unordered.restype = ctypes.c_longlong
    return L


@pytest.mark.parametrize("swap", [1, 0])
@pytest.mark.parametrize("L,E", PLANS)
def test_lds_accesses_are_ordered(lib, L, E, swap):
    rng = np.random.default_rng(L + E)
    x = (rng.standard_normal(L) + 1j * rng.standard_normal(L)).astype(np.complex64)
    table = np.exp(-2j * np.pi * np.arange(L) / L).astype(np.complex64)
    fwd, inv = np.empty_like(x), np.empty_like(x)
    args = [a.ctypes.data_as(ctypes.c_void_p) for a in (x, table, fwd, inv)]
    assert lib.emu_unordered(L, E, swap, *args) == 0
    # FP32 passes: a few roundings of the rms per pass, at most five passes
    for got, want in ((fwd, np.fft.fft(x.astype(np.complex128))),
                      (inv, L * np.fft.ifft(x.astype(np.complex128)))):
        assert np.max(np.abs(got - want)) <= 1e-5 * np.max(np.abs(want))
