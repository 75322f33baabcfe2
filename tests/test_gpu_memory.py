"""Indexes and searches on a GPU whose memory is nearly taken.

The rest of the memory is held by buffers that are given back at the end.  A build that
fits has its postings' contexts; a loaded index has them where they leave as much memory as
they take; and a search that finds no memory goes on without them.
"""
import contextlib
import ctypes
import functools
import time

import numpy as np
import pytest

from test_gpu_contexts import default_grouping  # noqa: F401
from test_gpu_filter import as_rows, gpu

pytestmark = pytest.mark.gpu

MB = 1 << 20
SPAN = 11


def free_bytes(G):
    """Of the GPU, from the HIP runtime that the library is linked to."""
    free, total = ctypes.c_size_t(), ctypes.c_size_t()
    assert G.lib().hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
    return free.value


@contextlib.contextmanager
def leave(G, target):
    """Holds all but about `target` bytes of the free memory, what comes back late (some
    milliseconds after a free) included."""
    held = []

    def fill():
        size = 32 << 30
        while size >= 2 * MB:
            if free_bytes(G) - size < target:
                size //= 2
                continue
            try:
                held.append(G.DeviceBuffer(size))
            except G.GGError:
                size //= 2

    try:
        quiet = 0
        while quiet < 10:  # a second without more of it
            n = len(held)
            fill()
            quiet = quiet + 1 if len(held) == n else 0
            time.sleep(0.1)
        yield
    finally:
        for b in held:
            b.close()


@functools.lru_cache(maxsize=1)
def bank(bases, seed=61, n=2000):
    rng = np.random.Generator(np.random.PCG64([seed, bases]))
    seqs = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, bases, dtype=np.uint8)]
    return seqs, np.linspace(0, bases, n + 1).astype(np.int64)


def small_bank():
    return bank.__wrapped__(100_000)


@pytest.mark.parametrize("max_posting", [0, 10])
def test_contexts_of_a_tight_build(max_posting):
    """200 Mbp: 212 MB of index, 291 MB of contexts and, while it is built, 572 MB of
    temporaries, 291 of them the windows' keys.  900 MB hold what the build needs, not that
    and the contexts; with a cutoff, which drops one list in a hundred, a little less."""
    G = gpu()
    G.Index(*small_bank(), SPAN).close()  # kernels loaded, first buffers allocated
    seqs, off = bank(200_000_000)
    with leave(G, 900 * MB):
        ix = G.Index(seqs, off, SPAN, max_posting=max_posting)
        got = ix.contexts(), 16 * ix.info()["n_postings"]
        ix.close()
    assert got[0] == got[1] > 0


def test_contexts_of_an_index_with_a_cutoff():
    """16 bytes for each posting that is kept."""
    G = gpu()
    rng = np.random.Generator(np.random.PCG64(62))
    seqs, off = bank.__wrapped__(300_000, n=100)
    seqs[100_000:200_000] = np.resize(np.frombuffer(b"ACC", np.uint8), 100_000)
    ix = G.Index(seqs, off, SPAN, max_posting=20)
    n = ix.info()["n_postings"]
    assert 0 < n < 25_000 and ix.contexts() == 16 * n
    q = seqs[int(rng.integers(0, 50_000)):][:2000].copy()
    rc, hits, _ = ix.search(q, G.params(5), cap=5)
    assert rc == 0 and len(hits) > 0 and as_rows(hits)[0][3] - as_rows(hits)[0][2] > 1000


def queries(seqs, n, length, seed=63):
    rng = np.random.Generator(np.random.PCG64(seed))
    at = rng.integers(0, len(seqs) - length, n)
    return (np.concatenate([seqs[a:a + length] for a in at]),
            np.arange(n + 1, dtype=np.int64) * length)


def budget_of(G, ix):
    srv = G.Server(ix, G.params(5), 0, 4)
    b = srv.info()["budget_bytes"]
    srv.close()
    return b


def test_loaded_index_leaves_memory_for_others(tmp_path):
    """212 MB of index and 291 MB of contexts: in 650 MB they would leave less than they take.
    The hit budget is a quarter of what the index leaves in any case."""
    G = gpu()
    seqs, off = bank(200_000_000)
    path = str(tmp_path / "a.gg")
    ix = G.Index(seqs, off, SPAN)
    ix.save(path)
    want = budget_of(G, ix)
    ix.close()
    back = G.Index.load(path)
    there = back.contexts()
    back.close()
    with leave(G, 650 * MB):
        ix = G.Index.load(path)
        got = ix.contexts(), budget_of(G, ix)
        ix.close()
    assert want == 16 << 30 and there > 0
    assert got[0] == 0 and abs(got[1] - (650 - 212) * MB // 4) < 8 * MB


def test_a_search_without_memory_goes_on_without_contexts(monkeypatch):
    """The search is told that its buffers by contexts do not fit: batches replayed, with
    statistics and in ranges of sequences, requests to the search service, and batches of
    four threads, each on an index of its own.  Afterwards, with memory, the same results."""
    from concurrent.futures import ThreadPoolExecutor

    G = gpu()
    seqs, off = bank.__wrapped__(3_000_000, n=300)
    prm = G.params(5)
    q, qoff = queries(seqs, 200, 300)

    def batch(ix, stats=False):
        rc, hits, n, st = ix.search_batch(q, qoff, prm, cap=5, stats=stats)
        return rc, [as_rows(h) for h in hits], n.tolist(), st.tolist() if stats else None

    def pieces(ix):
        ix.set_hit_budget(16 * 4096)
        return batch(ix, True)

    def serve(ix):
        srv = G.Server(ix, prm, 0, 16)
        tickets = [srv.submit(q[a:b]) for a, b in zip(qoff[:-1], qoff[1:])]
        got = [srv.poll(t, cap=5, timeout_us=-1) for t in tickets]
        srv.close()
        return max(g[0] for g in got), [(as_rows(g[1]), g[2]) for g in got]

    def threads(ix):
        with ThreadPoolExecutor(4) as ex:
            got = list(ex.map(lambda i: batch(ix, i % 2 == 0), range(16)))
        return max(g[0] for g in got), all(g[:3] == got[0][:3] for g in got), got[0]

    for call in (batch, lambda ix: batch(ix, True), pieces, serve, threads):
        monkeypatch.delenv("GG_ROOM", raising=False)
        ix = G.Index(seqs, off, SPAN)
        ix.profile(True)
        want = call(ix)
        assert want[0] == 0 and ix.contexts() > 0
        ix.close()
        monkeypatch.setenv("GG_ROOM", "none")
        ix = G.Index(seqs, off, SPAN)
        assert ix.contexts() > 0
        got = call(ix)
        assert got[0] == 0 and ix.contexts() == 0
        monkeypatch.delenv("GG_ROOM")
        same = [got == want, call(ix) == want]
        assert all(same)
        ix.close()
