"""Indexes and searches on a GPU whose memory is nearly taken.

The rest of the memory is held by buffers that are given back at the end.  An index keeps
its postings' contexts whenever they fit once the build's temporaries are gone.
"""
import contextlib
import ctypes

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
    """Holds all but about `target` bytes of the free memory."""
    held = []
    size = 32 << 30
    try:
        while size >= 4 * MB:
            if free_bytes(G) - size < target:
                size //= 2
                continue
            try:
                held.append(G.DeviceBuffer(size))
            except G.GGError:
                size //= 2
        yield
    finally:
        for b in held:
            b.close()


def bank(bases, seed=61, n=2000):
    rng = np.random.Generator(np.random.PCG64([seed, bases]))
    seqs = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, bases, dtype=np.uint8)]
    return seqs, np.linspace(0, bases, n + 1).astype(np.int64)


def test_contexts_of_a_tight_build():
    """200 Mbp: 212 MB of index, 291 MB of contexts and, while it is built, 572 MB of
    temporaries, 291 of them the windows' keys.  900 MB hold what the build needs, not that
    and the contexts; 600 MB do not hold the build."""
    G = gpu()
    G.Index(*bank(100_000), SPAN).close()  # kernels loaded, first buffers allocated
    seqs, off = bank(200_000_000)
    with leave(G, 900 * MB):
        ix = G.Index(seqs, off, SPAN)
        assert ix.contexts() == 16 * ix.info()["n_postings"]
        ix.close()
    with leave(G, 600 * MB):
        with pytest.raises(G.GGError) as e:
            G.Index(seqs, off, SPAN)
        assert e.value.status == G.GG_ENOMEM


def test_contexts_of_an_index_with_a_cutoff():
    """16 bytes for each posting that is kept."""
    G = gpu()
    rng = np.random.Generator(np.random.PCG64(62))
    seqs, off = bank(300_000, n=100)
    seqs[100_000:200_000] = np.resize(np.frombuffer(b"ACC", np.uint8), 100_000)
    ix = G.Index(seqs, off, SPAN, max_posting=20)
    n = ix.info()["n_postings"]
    assert 0 < n < 25_000 and ix.contexts() == 16 * n
    q = seqs[int(rng.integers(0, 50_000)):][:2000].copy()
    rc, hits, _ = ix.search(q, G.params(5), cap=5)
    assert rc == 0 and len(hits) > 0 and as_rows(hits)[0][3] - as_rows(hits)[0][2] > 1000
