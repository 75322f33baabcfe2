"""GPU parity of runs taken from the postings' contexts, bit-exact.

Where M exceeds the seed span and the gap limit stays within three windows, the
default grouping stores no hit: the codes of the windows around each posting tell
which hits start a run.  Checked against the oracle, every field and count, over the
widths of a context's fields (k = 8 .. 16, plain and masked), gap limits of one to
three windows and one past them, minimum lengths around two hits, both strands, a
repeat cutoff, lists of two-letter banks that fill many tiles, sequence ranges, and
an index file whose lists are not the bank's.
"""
import numpy as np
import pytest

from paper_1507_02987_amd import synth
from test_gpu_filter import as_rows, check_graph, check_stats, gpu, oracle_all

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def default_grouping(monkeypatch):
    for v in ("GG_GROUPING", "GG_GRAPH", "GG_SORT", "GG_FILTER", "GG_FUSE"):
        monkeypatch.delenv(v, raising=False)


def two_letter(seed, n_seqs, lmax, letters=b"AC"):
    """Sequences of long tandem repeats of two letters: long lists, long runs, and
    runs joined over mismatched windows."""
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([150702987, seed])))
    ab = np.frombuffer(letters, np.uint8)
    lens = rng.integers(0, lmax + 1, n_seqs)
    off = np.zeros(n_seqs + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    seqs = np.empty(int(off[-1]), np.uint8)
    for s in range(n_seqs):
        unit = ab[rng.integers(0, 2, int(rng.integers(1, 7)))]
        body = np.resize(unit, int(lens[s]))
        flips = rng.random(len(body)) < 0.02
        body[flips] = ab[rng.integers(0, 2, int(flips.sum()))]
        seqs[off[s]:off[s + 1]] = body
    return synth.Database(seqs, off, "two")


def both_forms(G, ggo, gix, oix, qs, N, **kw):
    want, wst = oracle_all(oix, qs, ggo.params(N, **kw))
    gix.profile(True)
    check_stats(G, gix, qs, G.params(N, **kw), want, wst)
    probed = gix.profile_read("probe")["units"]
    check_graph(G, gix, qs, G.params(N, **kw), want)
    gix.profile(False)
    return probed, wst


@pytest.mark.parametrize("k,mask,gap,min_len", [
    (8, None, 22, 22), (10, None, 22, 22), (11, None, 0, 12), (11, None, 10, 22),
    (11, None, 11, 22), (11, None, 32, 23), (11, None, 22, 34), (12, None, 22, 24),
    (12, None, 24, 25), (13, None, 26, 15), (11, "111010010100110111", 22, 22),
    (11, "111010010100110111", 36, 37), (9, "0110111011011", 39, 14),
    (10, "11111" + "0" * 22 + "11111", 32, 33)])
def test_fields_gaps_and_lengths(ggo, k, mask, gap, min_len):
    G = gpu()
    db = synth.repeat_db(70 + k, n_seqs=300, lmin=0, lmax=1500)
    qs = synth.random_queries(70 + k, db, n=24, lmin=0, lmax=900, frac_homolog=0.8,
                              ident_lo=0.85, ident_hi=1.0, indel_rate=0.01)
    if mask:
        oix, gix = ggo.Index(db.seqs, db.off, mask=mask), G.Index(db.seqs, db.off, mask=mask)
    else:
        oix, gix = ggo.Index(db.seqs, db.off, k), G.Index(db.seqs, db.off, k)
    probed, wst = both_forms(G, ggo, gix, oix, qs, 20, max_gap=gap, min_hsp_len=min_len)
    span = len(mask) if mask else k
    assert (probed > 0) == (min_len > span and gap // span + 1 <= 3)
    assert sum(s["n_cands"] for s in wst) > 0


@pytest.mark.parametrize("lmax,n_seqs,gap,min_len", [(300, 120, 22, 22), (2000, 60, 22, 22),
                                                     (2000, 60, 32, 60)])
def test_long_lists(ggo, lmax, n_seqs, gap, min_len):
    """Lists over many tiles, queries over and under the per-query LDS sorts."""
    G = gpu()
    db = two_letter(80 + lmax, n_seqs, lmax)
    qs = synth.random_queries(81, db, n=10, lmin=0, lmax=min(lmax, 400), frac_homolog=0.9,
                              ident_lo=0.9, ident_hi=1.0, indel_rate=0.01)
    oix, gix = ggo.Index(db.seqs, db.off, 11), G.Index(db.seqs, db.off, 11)
    probed, wst = both_forms(G, ggo, gix, oix, qs, 20, max_gap=gap, min_hsp_len=min_len)
    assert probed > 0
    # the same in ranges of sequences
    gix.set_hit_budget(16 * max(4096, max(s["n_hits"] for s in wst) // 3))
    both_forms(G, ggo, gix, oix, qs, 20, max_gap=gap, min_hsp_len=min_len)


def test_k16_against_stored_hits(monkeypatch):
    """No field but window 2's is whole at k = 16 (its 4^16 list heads are too many
    for the oracle here): against the sort of every hit."""
    G = gpu()
    db = two_letter(85, 200, 900)
    qs = synth.random_queries(86, db, n=12, lmin=0, lmax=500, frac_homolog=0.9, ident_lo=0.93,
                              ident_hi=1.0, indel_rate=0.005)
    gix = G.Index(db.seqs, db.off, 16)
    prm = G.params(20, max_gap=32, min_hsp_len=17)
    gix.profile(True)
    rc, got, _, st = gix.search_batch(qs.buf, qs.off, prm, cap=1000, stats=True)
    assert rc == 0 and gix.profile_read("probe")["units"] > 0
    monkeypatch.setenv("GG_GROUPING", "sort")
    rc, want, _, wst = gix.search_batch(qs.buf, qs.off, prm, cap=1000, stats=True)
    assert rc == 0 and (st == wst).all() and wst["n_cands"].sum() > 0
    for a, b in zip(got, want):
        assert as_rows(a) == as_rows(b)


@pytest.mark.parametrize("strands,max_posting", [(2, 0), (1, 40), (2, 40), (1, 3)])
def test_strands_and_cutoff(ggo, strands, max_posting):
    """A window whose list was dropped is no hit, whatever its neighbours' contexts."""
    G = gpu()
    db = synth.repeat_db(90, n_seqs=400, lmin=0, lmax=1200)
    qs = synth.random_queries(91, db, n=16, lmin=20, lmax=700, frac_homolog=0.9, ident_lo=0.9,
                              ident_hi=1.0, indel_rate=0.005)
    oix = ggo.Index(db.seqs, db.off, 9, strands=strands, max_posting=max_posting)
    gix = G.Index(db.seqs, db.off, 9, strands=strands, max_posting=max_posting)
    probed, _ = both_forms(G, ggo, gix, oix, qs, 20, max_gap=18, min_hsp_len=19)
    assert probed > 0


def test_loaded_index(ggo, tmp_path):
    """A saved index keeps its contexts; one whose lists miss a window of the bank is
    searched by its lists."""
    import struct

    from test_index_file import file_hash

    G = gpu()
    db = synth.repeat_db(95, n_seqs=100, lmin=100, lmax=1200)
    qs = synth.random_queries(96, db, n=8, lmin=50, lmax=700, frac_homolog=1.0, ident_lo=0.9,
                              ident_hi=1.0, indel_rate=0.005)
    oix, gix = ggo.Index(db.seqs, db.off, 8), G.Index(db.seqs, db.off, 8)
    path = str(tmp_path / "a.gg")
    gix.save(path)
    back = G.Index.load(path)
    probed, _ = both_forms(G, ggo, back, oix, qs, 20, max_gap=16, min_hsp_len=17)
    assert probed > 0
    # drop the last posting of the longest list
    heads, post = gix.export()
    c = int(np.argmax(np.diff(heads.astype(np.int64))))
    gone = int(heads[c + 1]) - 1
    raw = open(path, "rb").read()
    n_seqs = gix.info()["n_seqs"]
    at_heads = 72 + 8 * (n_seqs + 1)
    at_post = at_heads + 4 * len(heads)
    heads2 = heads.copy()
    heads2[c + 1:] -= 1
    post2 = np.delete(post, gone, axis=0)
    head = bytearray(raw[:72])
    struct.pack_into("<q", head, 48, len(post2))
    body = bytes(head[8:]) + raw[72:at_heads] + heads2.tobytes() + post2.tobytes() + \
        raw[at_post + 8 * len(post):-8]
    path2 = str(tmp_path / "b.gg")
    with open(path2, "wb") as f:
        f.write(raw[:8] + body + struct.pack("<Q", file_hash(body)))
    part = G.Index.load(path2)
    part.profile(True)
    rc, got, _, st = part.search_batch(qs.buf, qs.off, G.params(20, max_gap=16, min_hsp_len=17),
                                       cap=1000, stats=True)
    assert rc == 0 and part.profile_read("probe")["units"] == 0
    part.set_tuning(grouping="bucket")
    rc, want, _, wst = part.search_batch(qs.buf, qs.off, G.params(20, max_gap=16, min_hsp_len=17),
                                         cap=1000, stats=True)
    assert rc == 0 and (st == wst).all()
    for a, b in zip(got, want):
        assert as_rows(a) == as_rows(b)


@pytest.mark.parametrize("copies", [1, 511, 512, 513, 2049, 40_000])
def test_one_long_list_among_short_ones(ggo, copies):
    """A window that the bank holds `copies` times, alone each time, in a query of random
    bases: one position's hits span many waves' parts while the lists stay short on
    average, and starts lie on both sides of them."""
    G = gpu()
    rng = np.random.Generator(np.random.PCG64([21, copies]))
    rand = lambda n: rng.choice(list(b"ACGT"), n).astype(np.uint8)
    word = np.frombuffer(b"ACCGTTGACAG", np.uint8)
    plain = rand(30_000)
    body = rand(22 * copies).reshape(copies, 22)
    body[:, :11] = word  # at a multiple of the span, so indexed; the window after is random
    seqs = np.concatenate([plain, body.reshape(-1)])
    db = synth.Database(seqs, np.array([0, len(plain), len(seqs)], np.int64), "one long list")
    parts, off = [], [0]
    for _ in range(3):
        a = int(rng.integers(0, 25_000))
        parts += [plain[a:a + 300], word, rand(900), plain[a + 400:a + 700]]
        off.append(sum(len(p) for p in parts))
    qs = synth.QuerySet(np.concatenate(parts), np.array(off, np.int64), *[np.zeros(3)] * 4)
    gix, oix = G.Index(db.seqs, db.off, 11), ggo.Index(db.seqs, db.off, 11)
    probed, wst = both_forms(G, ggo, gix, oix, qs, 20)
    assert probed >= 3 * copies and all(s["n_cands"] >= 2 for s in wst)
