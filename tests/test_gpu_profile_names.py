"""Stage names of gg_profile_read that programs read, on the GPU."""
import pytest

from paper_1507_02987_amd import synth
from test_gpu_contexts import default_grouping  # noqa: F401
from test_gpu_filter import gpu

pytestmark = pytest.mark.gpu


def test_sweep_of_queries_merged_by_a_block_each():
    """Queries of a few runs: every merge is a sweep by one block per query."""
    G = gpu()
    db = synth.small_db(n_seqs=400)
    qs = synth.small_queries(db, n_homolog=6, n_random=2)
    gix = G.Index(db.seqs, db.off, 11)
    gix.profile(True)
    rc, _, _, st = gix.search_batch(qs.buf, qs.off, G.params(20), cap=64, stats=True)
    assert rc == 0
    merge, sweep = gix.profile_read("merge"), gix.profile_read("merge_sweep")
    assert sweep["units"] == st["n_cands"].sum() > 0
    assert sweep == merge and sweep["launches"] >= 1 and sweep["ms"] > 0
