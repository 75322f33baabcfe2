"""Queries of many runs in a replayed batch, on the GPU.

A query with more runs than the per-query LDS sorts hold is left to the regular path, and
the replay must not first find and extend its runs: alone in one block, they took ten times
as long as the whole batch on the regular path.  Results against the oracle, with the
queries' offsets summed by their blocks and (past 4,096 queries) scanned; and the batch's
time, which is the regular path's and that of one pass over the index hits, at most four
times the regular path's alone (the runs' work made it ten to ninety times).
"""
import time

import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_contexts import default_grouping  # noqa: F401
from test_gpu_filter import as_rows, check_graph, gpu, oracle_all

pytestmark = pytest.mark.gpu


def bank_and_queries(n_seqs, tandem, n_light, n_heavy, heavy_len):
    rng = np.random.Generator(np.random.PCG64([51, n_seqs, n_heavy]))
    acgt = np.frombuffer(b"ACGT", np.uint8)
    rand = lambda n: acgt[rng.integers(0, 4, n)]
    ac = lambda n: np.resize(np.frombuffer(b"AC", np.uint8), n)
    seqs = [np.concatenate([rand(300), ac(tandem), rand(300)]) for _ in range(n_seqs)]
    qs = [np.concatenate([rand(40), seqs[i % n_seqs][:120]]) for i in range(n_light)]
    for i in range(n_heavy):
        qs.insert((i + 1) * len(qs) // (n_heavy + 1), ac(heavy_len + i))
    cat = lambda parts: (np.concatenate(parts), np.concatenate([[0], np.cumsum(
        [len(p) for p in parts])]).astype(np.int64))
    return synth.Database(*cat(seqs), "tandem"), synth.QuerySet(*cat(qs), *[np.zeros(len(qs))] * 4)


@pytest.mark.parametrize("n_light,n_heavy", [(0, 1), (30, 3), (4_200, 2)])
def test_results(ggo, n_light, n_heavy):
    G = gpu()
    db, qs = bank_and_queries(60, 200, n_light, n_heavy, 150)
    oix, gix = ggo.Index(db.seqs, db.off, 11), G.Index(db.seqs, db.off, 11)
    want, wst = oracle_all(oix, qs, ggo.params(20))
    assert sorted(s["n_cands"] for s in wst)[-n_heavy] > 1024
    check_graph(G, gix, qs, G.params(20), want, cap=50)
    check_graph(G, gix, qs, G.params(20), want, cap=50)


def test_time(monkeypatch):
    G = gpu()
    db, qs = bank_and_queries(4_000, 150, 100, 40, 150)
    gix, prm = G.Index(db.seqs, db.off, 11), G.params(20)

    def best():
        t, r = [], None
        for _ in range(4):
            t0 = time.perf_counter()
            r = gix.search_batch(qs.buf, qs.off, prm, cap=20)
            t.append(time.perf_counter() - t0)
        return min(t), [as_rows(x) for x in r[1]]

    replayed, got = best()
    monkeypatch.setenv("GG_GRAPH", "0")
    regular, want = best()
    print(f"replayed {1e3 * replayed:.2f} ms, regular {1e3 * regular:.2f} ms")
    assert got == want
    assert replayed < 4 * regular + 1e-3
