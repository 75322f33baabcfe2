"""The traceback's walk by stretches of 64 cells and its sweep by pairs, against the
oracle byte for byte: pairs and gaps of lengths about a stretch, gaps up to the band's
whole width in either direction, rectangles of few rows (fewer than a step's lanes),
and rows and columns about the number staged in LDS."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def rand(rng, n):
    return rng.choice(list(b"ACGT"), n).astype(np.uint8)


def check(ggo, q, bank, d0, score, band, mark):
    from paper_1507_02987_amd import gg as G

    off = np.array([0, len(bank)], np.int64)
    gix, oix = G.Index(bank, off, 8), ggo.Index(bank, off, 8)
    hit = np.zeros(1, G.HIT_DTYPE)
    hit["score"], hit["q_end"], hit["d_end"], hit["band_d0"] = score, len(q), len(bank), d0
    rc, ops = gix.traceback(q.tobytes(), G.params(5, band=band), hit)
    assert rc == G.GG_OK, mark
    want = oix.traceback(q.tobytes(), ggo.params(5, band=band), tuple(hit[0].tolist()))
    assert ops[0] == want, mark


@pytest.mark.parametrize("gap", [1, 2, 63, 64, 65, 100, 126])
@pytest.mark.parametrize("in_query", [True, False])
def test_gaps_about_a_stretch(ggo, gap, in_query):
    rng = np.random.Generator(np.random.PCG64([7, gap, in_query]))
    a, b, g = rand(rng, 301 + gap), rand(rng, 300), rand(rng, gap)
    short, long = np.concatenate([a, b]), np.concatenate([a, g, b])
    score = len(a) + len(b) - 5 - 2 * gap
    q, bank, d0 = (short, long, gap // 2) if in_query else (long, short, -(gap // 2))
    check(ggo, q, bank, d0, score, 63, (gap, in_query))


@pytest.mark.parametrize("n", [8, 31, 63, 64, 65, 127, 128, 129, 4095, 4096, 4097])
@pytest.mark.parametrize("band", [0, 31, 63])
def test_lengths_about_a_stretch(ggo, n, band):
    rng = np.random.Generator(np.random.PCG64([8, n, band]))
    bank = rand(rng, n)
    q, score = bank.copy(), n
    if n > 32:  # a mismatch not too near either end
        q[n // 2] = other(q[n // 2])
        score -= 4
    check(ggo, q, bank, 0, score, band, (n, band))


def other(base):
    return b"ACGT"[(b"ACGT".index(bytes([base])) + 1) % 4]


@pytest.mark.parametrize("d", [-3, 3])
def test_one_row_or_column_more_than_staged(ggo, d):
    rng = np.random.Generator(np.random.PCG64([9, d + 3]))
    a, b, g = rand(rng, 2048), rand(rng, 2047), rand(rng, 3)
    short, long = np.concatenate([a, b]), np.concatenate([a, g, b])
    q, bank = (short, long) if d > 0 else (long, short)
    check(ggo, q, bank, d // 2, 4095 - 5 - 6, 32, d)
