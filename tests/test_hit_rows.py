"""The hit arrays that the Python binding returns, on the CPU: copies of the library's rows
that own their memory, so a caller may write and resize them."""
import numpy as np
import pytest

from paper_1507_02987_amd import gg


@pytest.mark.parametrize("cap,counts", [(5, [0, 1, 4, 5]), (1, [1, 0, 1]), (3, [])])
def test_copies_of_their_own(cap, counts):
    out = np.zeros(max(len(counts) * cap, 1), gg.HIT_DTYPE)
    for f, name in enumerate(gg.HIT_FIELDS):
        out[name] = np.arange(len(out)) * 100 + f
    want = [out[i * cap:i * cap + n].copy() for i, n in enumerate(counts)]
    got = gg._rows(out, range(0, len(counts) * cap, cap), counts)
    out["score"] = -1
    assert len(got) == len(counts)
    for g, w in zip(got, want):
        assert g.dtype == gg.HIT_DTYPE and (g == w).all() and g.shape == w.shape
        assert g.flags.owndata and g.flags.writeable and g.flags.c_contiguous
        g.resize(len(w) + 2, refcheck=False)
        g["score"] = 7
    assert (out["score"] == -1).all()
