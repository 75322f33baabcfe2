"""The per-query orders of merging, selection and reporting (records sorted in
registers by packed keys), bit-exact against the oracle at numbers of records about
the sort's steps: one lane's, one wave's, two waves', the block's, and one more, which
leaves for the global sort.  Boxes of one length and score, several of each query
segment and sequence, so the orders are decided by their last fields."""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_filter import check_graph, check_stats, gpu, oracle_all

pytestmark = pytest.mark.gpu

LEN = 34  # bases of a segment: two whole windows at any phase, so one run and one box


def queries(seed, counts):
    """A bank of segments, one in five twice in its sequence, and
    one query per count: that many segments, random bases after each."""
    rng = np.random.Generator(np.random.PCG64([11, seed]))
    most = max(counts)
    segs = rng.choice(list(b"AC"), (most, LEN)).astype(np.uint8)
    segs[:, ::3] = rng.choice(list(b"GT"), segs[:, ::3].shape)
    seqs, lens = [], []
    for part in np.array_split(np.arange(most), 7):
        body = []
        for s in part:
            body += [segs[s], rng.choice(list(b"ACGT"), 70).astype(np.uint8)]
            if s % 5 == 0:  # a second copy in the same sequence, at the same query start
                body += [segs[s], rng.choice(list(b"ACGT"), 70).astype(np.uint8)]
        seqs += body
        lens.append(sum(len(b) for b in body))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    db = synth.Database(np.concatenate(seqs), off, "segments")
    text, qoff = [], [0]
    for n in counts:
        for s in range(n):
            text += [segs[s], rng.choice(list(b"ACGT"), 40).astype(np.uint8)]
        qoff.append(sum(len(t) for t in text))
    buf = np.concatenate(text)
    return db, synth.QuerySet(buf, np.array(qoff, np.int64), *[np.zeros(len(counts))] * 4)


@pytest.mark.parametrize("counts", [(1, 2, 3, 4, 5, 7), (52, 53, 54, 64), (212, 213, 214, 256),
                                    (426, 427), (851, 852, 853, 854, 855, 856)])
def test_records_about_the_sort_steps(ggo, counts):
    G = gpu()
    db, qs = queries(len(counts), counts)
    gix, oix = G.Index(db.seqs, db.off, 11), ggo.Index(db.seqs, db.off, 11)
    want, wst = oracle_all(oix, qs, ggo.params(1024))
    for n, s in zip(counts, wst):
        assert s["n_cands"] >= n
    check_stats(G, gix, qs, G.params(1024), want, wst)
    check_graph(G, gix, qs, G.params(1024), want, cap=1024)


@pytest.mark.parametrize("n_long,N", [(1, 1), (40, 20), (300, 256), (300, 300), (1030, 1024)])
def test_selection_of_a_prefiltered_query(ggo, n_long, N):
    """Over kSegCap boxes: the global merge, and the longest of them put in selection
    order by query where they fit (or by the global sort: the last case)."""
    G = gpu()
    db, qs = queries(7, (1100,))
    rng = np.random.Generator(np.random.PCG64([12, n_long]))
    # segments of 200 bases and up, each in a sequence of its own: a third share a length
    longs = [rng.choice(list(b"ACGT"), 200 + (0 if s % 3 else 7 * (s % 50))).astype(np.uint8)
             for s in range(n_long)]
    seqs = np.concatenate([db.seqs] + longs)
    off = np.concatenate([db.off, db.off[-1] + np.cumsum([len(x) for x in longs])])
    db = synth.Database(seqs, off.astype(np.int64), "long segments")
    buf = np.concatenate([qs.buf] + longs)
    qs = synth.QuerySet(buf, np.array([0, len(buf)], np.int64), *[np.zeros(1)] * 4)
    gix, oix = G.Index(db.seqs, db.off, 11), ggo.Index(db.seqs, db.off, 11)
    want, wst = oracle_all(oix, qs, ggo.params(N))
    assert wst[0]["n_cands"] > 1024 and wst[0]["n_selected"] == N
    check_stats(G, gix, qs, G.params(N), want, wst)
    check_graph(G, gix, qs, G.params(N), want, cap=1024)
