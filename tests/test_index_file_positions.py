"""Which posting positions of an index file are accepted, on the host: multiples of the
window span whose window lies inside the sequence, at every span."""
import struct

import numpy as np
import pytest

from paper_1507_02987_amd import gg
from test_index_file import file_hash, load_status

BASES = 100_000  # one sequence, all A: every window has code 0


def one_posting(span, pos):
    """An index of windows of `span` bases, their first one coded, with one posting."""
    n_words = (BASES + 15) // 16 + 1
    hdr = struct.pack("<I3iII5q", 1, 1, span, 1, 1, 0, 1, BASES, 1, BASES, n_words)
    body = (hdr + np.array([0, BASES], np.int64).tobytes() +
            np.array([0, 1, 1, 1, 1], np.uint32).tobytes() + struct.pack("<ii", 0, pos) +
            np.zeros(n_words, np.uint32).tobytes())
    return b"GGINDEX1" + body + struct.pack("<Q", file_hash(body))


@pytest.mark.parametrize("span", [1, 2, 3, 7, 11, 16, 31, 32])
def test_positions(tmp_path, span):
    last = (BASES // span - 1) * span
    p = tmp_path / "x.ggi"
    for pos in sorted({0, 1, span - 1, span, span + 1, 2 * span, 3 * span + 1, last - 1, last,
                       last + 1, last + span, -span}):
        p.write_bytes(one_posting(span, pos))
        ok = pos >= 0 and pos % span == 0 and pos + span <= BASES
        got = load_status(p)
        assert got in ((gg.GG_OK, gg.GG_EDEVICE) if ok else (gg.GG_EINVAL,)), (pos, got)
