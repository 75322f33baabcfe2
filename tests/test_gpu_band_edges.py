"""The banded sweep's ends, bit-exact against the oracle: boxes about the number of
bases staged in LDS and down to a few, the narrowest and widest bands, and scorings
whose gaps or mismatches cost nothing, where a cell past the box's end or beside the
band ties with one inside."""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_filter import check_graph, check_stats, gpu, oracle_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("band", [0, 1, 31, 32, 63])
@pytest.mark.parametrize("score", [dict(), dict(mismatch=0), dict(gap_open=0, gap_extend=0),
                                   dict(match=7, mismatch=1, gap_open=3, gap_extend=0)])
def test_ends_of_box_and_band(ggo, band, score):
    G = gpu()
    rng = np.random.Generator(np.random.PCG64([31, band]))
    bank = rng.choice(list(b"ACGT"), 9_000).astype(np.uint8)
    db = synth.Database(bank, np.array([0, 4_600, 9_000], np.int64), "two sequences")
    parts = []
    for n in (24, 60, 130, 1_000, 4_095, 4_096, 4_097, 4_300):
        a = int(rng.integers(0, 4_600 - n))
        parts.append(bank[a:a + n])  # a whole copy: its box is n by n, to the query's ends
        parts.append(synth.mutate(bank[a:a + n], 0.05, 0.02, rng))
    parts.append(bank[4_500:4_700])  # over the first sequence's end
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    qs = synth.QuerySet(np.concatenate(parts), off, *[np.zeros(len(parts))] * 4)
    gix, oix = G.Index(db.seqs, db.off, 11), ggo.Index(db.seqs, db.off, 11)
    kw = dict(band=band, **score)
    want, wst = oracle_all(oix, qs, ggo.params(20, **kw))
    assert sum(s["n_out"] for s in wst) >= 8
    check_stats(G, gix, qs, G.params(20, **kw), want, wst)
    check_graph(G, gix, qs, G.params(20, **kw), want)


@pytest.mark.parametrize("n", [4_015, 4_016, 4_017, 8_031, 8_033, 9_500])
def test_long_boxes_in_parts(ggo, n):
    """Boxes of more pairs than are staged at a time, and their paths."""
    G = gpu()
    rng = np.random.Generator(np.random.PCG64([32, n]))
    bank = rng.choice(list(b"ACGT"), 12_000).astype(np.uint8)
    db = synth.Database(bank, np.array([0, len(bank)], np.int64), "one sequence")
    q = bank[1_000:1_000 + n].copy()
    q[rng.random(n) < 0.03] = ord("A")
    qs = synth.QuerySet(q, np.array([0, n], np.int64), *[np.zeros(1)] * 4)
    gix, oix = G.Index(db.seqs, db.off, 11), ggo.Index(db.seqs, db.off, 11)
    want, wst = oracle_all(oix, qs, ggo.params(3))
    check_stats(G, gix, qs, G.params(3), want, wst)
    check_graph(G, gix, qs, G.params(3), want)
    rc, hits, k = gix.search(q, G.params(3), cap=3)
    assert rc == 0 and int(hits[0]["q_end"] - hits[0]["q_start"]) > n - 100
    rc, ops = gix.traceback(q, G.params(3), hits)
    assert rc == 0
    for h, got in zip(hits, ops):
        assert got == oix.traceback(q.tobytes(), ggo.params(3), tuple(int(x) for x in h.tolist()))
