"""GPU parity of the extension's forms, bit-exact: walks by step tables (scores up to 7
and 15) and mismatch by mismatch, a lane per side and, from 2^19 runs in a wave, a lane
per run, lane caps that queue walks or none, walks that reach the first and last bases
of the query and of the bank, and drop-offs around a table's eight steps."""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_filter import check_graph, check_stats, gpu, oracle_all

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def default_grouping(monkeypatch):
    for v in ("GG_GROUPING", "GG_GRAPH", "GG_SORT", "GG_FILTER", "GG_FUSE"):
        monkeypatch.delenv(v, raising=False)


def edge_bank():
    """A bank whose first and last sequences are whole queries too, with flips."""
    rng = np.random.default_rng(7)
    db = synth.repeat_db(100, n_seqs=60, lmin=12, lmax=700)
    parts = []
    for s in (0, 1, 59, 20, 33):
        a = db.seqs[db.off[s]:db.off[s + 1]].copy()
        parts.append(a.copy())
        flip = rng.random(len(a)) < 0.06
        a[flip] = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, int(flip.sum()))]
        parts.append(a)
        parts.append(a[len(a) // 3:])
    qoff = np.zeros(len(parts) + 1, np.int64)
    np.cumsum([len(p) for p in parts], out=qoff[1:])
    n = len(parts)
    return db, synth.QuerySet(np.concatenate(parts), qoff, np.zeros(n, np.int8),
                              np.full(n, -1, np.int64), np.zeros(n, np.int64),
                              np.zeros(n, np.int64), np.zeros(n))


@pytest.mark.parametrize("match,mismatch,xdrop", [
    (1, 3, 20), (1, 3, 0), (1, 3, 2), (1, 3, 3), (1, 3, 24), (7, 15, 60), (7, 15, 121), (8, 15, 40),
    (7, 16, 40), (1, 0, 5), (5, 1, 7), (2, 7, 1000000)])
@pytest.mark.parametrize("steps", [0, 1, 32, 256])
def test_scores_and_drops(ggo, match, mismatch, xdrop, steps):
    G = gpu()
    db, qs = edge_bank()
    oix, gix = ggo.Index(db.seqs, db.off, 8), G.Index(db.seqs, db.off, 8)
    gix.set_tuning(lane_steps=steps)
    kw = dict(match=match, mismatch=mismatch, xdrop=xdrop, max_gap=8, min_hsp_len=9)
    want, wst = oracle_all(oix, qs, ggo.params(50, **kw))
    assert sum(s["n_cands"] for s in wst) > 0
    check_stats(G, gix, qs, G.params(50, **kw), want, wst)
    check_graph(G, gix, qs, G.params(50, **kw), want)


def tandem_bank(n_seqs, length, flip):
    """Sequences of ACAC... with flipped bases: a run for every stretch and phase."""
    rng = np.random.default_rng(8)
    acgt = np.frombuffer(b"ACGT", np.uint8)
    seqs = np.resize(acgt[:2], n_seqs * length).copy()
    at = rng.random(len(seqs)) < flip
    seqs[at] = acgt[rng.integers(0, 4, int(at.sum()))]
    off = np.arange(n_seqs + 1, dtype=np.int64) * length
    return synth.Database(seqs, off, "tandem")


@pytest.mark.parametrize("match,mismatch,steps", [(1, 3, 256), (1, 3, 16), (9, 20, 256)])
def test_a_lane_per_run(ggo, match, mismatch, steps):
    G = gpu()
    db = tandem_bank(100, 801, 0.04)
    qs = synth.random_queries(102, db, n=2, lmin=500, lmax=700, frac_homolog=1.0, ident_lo=0.99,
                              ident_hi=1.0, indel_rate=0.0)
    oix, gix = ggo.Index(db.seqs, db.off, 8), G.Index(db.seqs, db.off, 8)
    gix.set_tuning(lane_steps=steps)
    kw = dict(match=match, mismatch=mismatch, xdrop=20 * match, max_gap=8, min_hsp_len=9)
    want, wst = oracle_all(oix, qs, ggo.params(20, **kw))
    assert sum(s["n_cands"] for s in wst) >= 1 << 19
    check_stats(G, gix, qs, G.params(20, **kw), want, wst)
