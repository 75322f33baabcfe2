"""The build's packing and list kernels at their edges: every byte value inside a
whole 16-base word and in the bank's last, part one; banks around the word, tile and
block sizes; one code holding every window.  Lists and postings equal the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def gpu():
    from paper_1507_02987_amd import gg

    gg.lib()
    return gg


def same_lists(G, ggo, seqs, off, k):
    oix = ggo.Index(seqs, off, k)
    gix = G.Index(seqs, off, k)
    heads, post = gix.export()
    seq, pos = oix.postings()
    assert (heads.astype(np.int64) == oix.list_off()).all()
    assert (post[:, 0] == seq).all() and (post[:, 1] == pos).all()


@pytest.mark.parametrize("n,at", [(15, 3), (16, 0), (16, 15), (17, 16), (48, 21)])
def test_every_byte(n, at):
    G = gpu()
    bank = np.frombuffer(b"ACGT" * 12, np.uint8)[:n].copy()
    off = np.array([0, n], np.int64)
    for b in range(256):
        bank[at] = b
        if chr(b) in "ACGTUacgtu":
            gix = G.Index(bank, off, 3)
            code = {"A": 0, "C": 1, "G": 2, "T": 3, "U": 3}
            heads, post = gix.export()
            for c in range(64):
                for s, p in post[heads[c]:heads[c + 1]]:
                    w = [code[chr(x).upper()] for x in bank[p:p + 3]]
                    assert s == 0 and c == 16 * w[0] + 4 * w[1] + w[2]
        else:
            with pytest.raises(G.GGError) as e:
                G.Index(bank, off, 3)
            assert e.value.status == G.GG_EINVAL


@pytest.mark.parametrize("k,lens", [
    (4, [0, 3, 4, 0, 5]), (11, [16] * 255 + [11]), (11, [22, 0, 0] * 171), (5, [5 * 2048]),
    (5, [5 * 2049 + 4]), (8, [1] * 300 + [4096] + [7] * 9), (1, [4099])])
def test_lists_at_tile_edges(ggo, k, lens):
    rng = np.random.default_rng(sum(lens) + k)
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    acgt = np.frombuffer(b"ACGT", np.uint8)
    same_lists(gpu(), ggo, acgt[rng.integers(0, 4, int(off[-1]))], off, k)
    same_lists(gpu(), ggo, np.full(int(off[-1]), ord("T"), np.uint8), off, k)
