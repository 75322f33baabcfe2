"""The words of a batch's packed queries, on the CPU: for every number of bases around the
sizes of words and blocks, each word that the buffer has room for is written once and none
past it.  The rule that the encoding kernel follows is compiled for the host from the
library's own header."""
import subprocess

from paper_1507_02987_amd import build as gbuild

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "gg_internal.h"
int main()
{
    for (int64_t T = 1; T <= 5 * gg::kBlock; ++T) {
        const int64_t n = gg::packed_words(T);
        if (n < (T + 15) / 16 + gg::kPackSlack) return std::printf("T %ld: no room\n", (long)T), 1;
        std::vector<int> written((size_t)n, 0);
        for (int64_t b = 0; b * gg::kBlock < T; ++b)
            for (int32_t t = 0; t < gg::kBlock; ++t) {
                const int64_t w = gg::packed_word(b, t, T);
                if (w < 0) continue;
                if (w >= n) return std::printf("T %ld: word %ld of %ld\n", (long)T, (long)w, (long)n), 1;
                ++written[(size_t)w];
                // a thread of the first words packs its own block's bases
                if (t < gg::kPackWords && w != b * gg::kPackWords + t) return std::printf("order\n"), 1;
            }
        for (int c : written)
            if (c != 1) return std::printf("T %ld: a word written %d times\n", (long)T, c), 1;
    }
    return 0;
}
"""


def test_every_word_once_and_none_past_the_end(tmp_path):
    src, exe = tmp_path / "words.hip", tmp_path / "words"
    src.write_text(PROGRAM)
    r = subprocess.run(["hipcc", *gbuild.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
