"""GPU parity of index windows of one to three bases, bit-exact.

A chunk of 64 bases then holds up to 64 windows, all of which the wave that finishes a
long run has to tell apart.  A homopolymer query against a homopolymer sequence has one
run on each diagonal, up to the whole query long: lengths on both sides of the chunks
that a lane takes by itself, queries over and under the per-query LDS sorts, and the
replayed and the regular form, against the oracle, every field and count.
"""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_contexts import both_forms, default_grouping  # noqa: F401
from test_gpu_filter import gpu

pytestmark = pytest.mark.gpu

LENGTHS = (1, 63, 64, 65, 257, 290, 300, 511)


def pack(parts):
    off = np.zeros(len(parts) + 1, np.int64)
    np.cumsum([len(p) for p in parts], out=off[1:])
    return np.frombuffer(b"".join(parts), np.uint8).copy(), off


def query_set(parts):
    return synth.QuerySet(*pack(parts), *[np.zeros(len(parts))] * 4)


@pytest.mark.parametrize("span,gap,mask", [(1, 0, None), (1, 1, None), (1, 2, None), (2, 0, None),
                                           (2, 4, None), (3, 6, None), (3, 6, "101")])
def test_homopolymers(ggo, span, gap, mask):
    G = gpu()
    seqs, off = pack([b"A" * n for n in LENGTHS] + [b"C" * 300])
    how = dict(mask=mask) if mask else dict(k=span)
    gix, oix = G.Index(seqs, off, **how), ggo.Index(seqs, off, **how)
    # under the per-query LDS sorts each alone, over them among all sequences
    for n in LENGTHS:
        one, alone = pack([b"A" * n])
        g1, o1 = G.Index(one, alone, **how), ggo.Index(one, alone, **how)
        probed, _ = both_forms(G, ggo, g1, o1, query_set([b"A" * n]), 20, max_gap=gap,
                               min_hsp_len=span + 1)
        assert probed > 0 or n < span
    qs = query_set([b"A" * n for n in LENGTHS] + [b"C" * 290, b"A" * 150 + b"C" * 290])
    _, wst = both_forms(G, ggo, gix, oix, qs, 20, max_gap=gap, min_hsp_len=span + 1)
    assert max(s["n_cands"] for s in wst) > 1024


@pytest.mark.parametrize("span,gap,min_len", [(1, 2, 30), (2, 4, 30), (3, 6, 20)])
def test_copies_of_5000_bases(ggo, span, gap, min_len):
    """A query equal to a sequence, and one equal to its middle."""
    G = gpu()
    rng = np.random.Generator(np.random.PCG64([31, span]))
    body = rng.choice(list(b"ACGT"), 5000).astype(np.uint8).tobytes()
    seqs, off = pack([body, body[700:900]])
    gix, oix = G.Index(seqs, off, span), ggo.Index(seqs, off, span)
    qs = query_set([body, body[1000:1300]])
    _, wst = both_forms(G, ggo, gix, oix, qs, 20, max_gap=gap, min_hsp_len=min_len)
    assert all(s["n_cands"] > 0 for s in wst)
