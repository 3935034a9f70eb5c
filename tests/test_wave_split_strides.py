"""The strides and regions of the transforms split over waves, as the header has them,
against gfx950's bank rules: every index of a region once and inside it, 16-lane
groups of a write on distinct values mod 16, 32-lane groups of a read mod 32."""
import ctypes

import pytest

from tests.test_wave_split import STRIDE_A, _sums


@pytest.fixture(scope="module")
def lib():
    from tests.emu import build_emu
    return ctypes.CDLL(build_emu.build_lds_layout())


@pytest.mark.parametrize("b", [1, 2, 3])
def test_header_strides(lib, b):
    region = lib.emu_split_region(b, 0)
    s = [lib.emu_split_stride(b, k) for k in range(6)]
    assert s == STRIDE_A[b]
    # p's wave bits step from region to region
    assert [lib.emu_split_stride(b, 6 + k) for k in range(b)] == [region << k for k in range(b)]
    n = [4, 8, 16]
    places = _sums(n + s, 9)
    assert len(set(places.tolist())) == 512 and places.max() < region
    assert len(set((_sums(s, 4) % 16).tolist())) == 16
    assert len(set((_sums(n + s[b:b + 3], 5) % 32).tolist())) == 32
    # second exchange: 1, 2, 4 (n[2..0]), 8, 16, 32 (n[5..3]), 72, 144, 288 (p)
    places = _sums([1, 2, 4, 8, 16, 32, 72, 144, 288], 9)
    assert len(set(places.tolist())) == 512 and places.max() < lib.emu_split_region(b, 1)
