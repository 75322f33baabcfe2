"""The list of the largest window code, 4^k - 1 (a window of T alone), on the GPU.

At k = 16 that code is 2^32 - 1, so the head after it lies past what 32 bits count.  The
oracle does not hold 4^16 list heads; but with every base of bank and queries exchanged
for its pair (A-T, C-G) a search finds the same alignments, and T's windows become A's,
whose code is 0.  Both searches must agree in every field and count, in the host-driven,
the replayed and the piecewise form and under each grouping; at k = 8 both equal the
oracle's.
"""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_contexts import default_grouping  # noqa: F401
from test_gpu_filter import as_rows, gpu, oracle_all

pytestmark = pytest.mark.gpu

PAIR = np.zeros(256, np.uint8)
PAIR[list(b"ACGT")] = list(b"TGCA")


def bank_and_queries(k):
    rng = np.random.Generator(np.random.PCG64([41, k]))
    rand = lambda n: rng.choice(list(b"ACGT"), n).astype(np.uint8)
    t = lambda n: np.full(n, ord("T"), np.uint8)
    seqs = [np.concatenate([rand(16 * int(rng.integers(1, 9))), t(int(rng.integers(0, 200))),
                            rand(100)]) for _ in range(40)]
    qs = [np.concatenate([s[:60], t(40), s[-100:]]) for s in seqs[:6]] + [t(100), t(k), rand(200)]
    cat = lambda parts: (np.concatenate(parts), np.concatenate([[0], np.cumsum(
        [len(p) for p in parts])]).astype(np.int64))
    return cat(seqs), cat(qs)


def search_all(G, bank, queries, k, prm):
    out = []
    gix = G.Index(*bank, k)
    for grouping in ("sort", "bucket", "probe"):
        gix.set_tuning(grouping=grouping)
        rc, res, _, st = gix.search_batch(*queries, prm, cap=500, stats=True)
        assert rc == 0
        out.append(([as_rows(r) for r in res], st.tolist()))
        rc, res, _, _ = gix.search_batch(*queries, prm, cap=500)
        assert rc == 0
        out.append(([as_rows(r) for r in res], st.tolist()))
    gix.set_tuning(grouping="sort")
    gix.set_hit_budget(16 * max(512, int(st["n_hits"].max()) // 2))
    rc, res, _, st = gix.search_batch(*queries, prm, cap=500, stats=True)
    assert rc == 0
    out.append(([as_rows(r) for r in res], st.tolist()))
    gix.close()
    return out


@pytest.mark.parametrize("k,gap", [(8, 16), (15, 30), (16, 0), (16, 32)])
def test_windows_of_t_alone(ggo, k, gap):
    G = gpu()
    bank, queries = bank_and_queries(k)
    kw = dict(max_gap=gap, min_hsp_len=k + 1)
    got = search_all(G, bank, queries, k, G.params(20, **kw))
    want = search_all(G, (PAIR[bank[0]], bank[1]), (PAIR[queries[0]], queries[1]), k,
                      G.params(20, **kw))
    for g in got + want:
        assert g == want[0]
    poly_t = want[0][1][7]
    assert poly_t[1] > 0, "a query of T alone has hits"
    if k == 8:
        oix = ggo.Index(*bank, k)
        qs = synth.QuerySet(*queries, *[np.zeros(len(queries[1]) - 1)] * 4)
        res, wst = oracle_all(oix, qs, ggo.params(20, **kw))
        assert [as_rows(r) for r in res] == got[0][0]
        assert [list(s.values()) for s in wst] == [list(s) for s in got[0][1]]
