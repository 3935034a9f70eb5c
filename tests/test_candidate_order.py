"""The order in which candidate lists are returned, on records at the ends of their
ranges: rows up to 4095, bins up to 2^32 - 1, spectra that differ in each of them."""
import numpy as np

import paper_1804_05335_amd as fdas


def _records(rng, n):
    rec = np.zeros(n, dtype=fdas._RECORD)
    rec["row"] = rng.choice([0, 1, 41, 4094, 4095], n)
    rec["r"] = rng.choice([0, 1, 2 ** 31, 2 ** 32 - 2, 2 ** 32 - 1], n)
    rec = rec[np.unique(rec[["row", "r"]], return_index=True)[1]]
    rec["power"] = rng.random(len(rec))
    return rng.permutation(rec)


def test_by_row():
    rec = _records(np.random.default_rng(1), 200)
    r, row, power, n = fdas._by_row((rec, 7))
    order = np.lexsort((rec["r"], rec["row"]))
    assert n == 7
    for got, want in ((r, rec["r"]), (row, rec["row"]), (power, rec["power"])):
        assert got.dtype == want.dtype and np.array_equal(got, want[order])


def test_by_spectrum():
    rng = np.random.default_rng(2)
    offs = np.array([0, 0, 1, 5, 5, 2 ** 31, 2 ** 32], dtype=np.int64)
    rec = _records(rng, 300)
    spec, r, row, power, n = fdas._by_spectrum((rec, len(rec)), offs)
    b = np.searchsorted(offs, rec["r"], side="right") - 1
    order = np.lexsort((rec["r"] - offs[b], rec["row"], b))
    for got, want in ((spec, b), (r, rec["r"] - offs[b]), (row, rec["row"]),
                      (power, rec["power"])):
        assert np.array_equal(got, want[order])
