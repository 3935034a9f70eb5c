"""Batched time series whose workgroups are grouped by XCD (from 2^23 complex values
in all and 128 workgroups per series) against each series by itself, ungrouped: every
tile is taken once, so the bins are the same bits."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("log2n,nseries", [(20, 16), (21, 8), (22, 5), (23, 2)])
def test_grouped_equals_single(log2n, nseries):
    import torch
    import paper_1804_05335_amd as fd
    x = np.random.default_rng(log2n).standard_normal((nseries, 1 << log2n), dtype=np.float32)
    xd = torch.from_numpy(x).cuda()
    got = fd.spectra_from_series(xd)
    for b in range(nseries):
        assert torch.equal(got[b], fd.spectrum_from_series(xd[b]))
