"""Launch records of the sampling walk's fused contractions: ttn_launch_rec.splits
has to say when a reduction launch follows.  The amplitudes of a (64, 64, 64)
node over 8192 shots, 64 x 8192 outputs and K = 4096, split K."""
import pytest

from paper_2210_03763_amd import ttn as T
from paper_2210_03763_amd import workload as W

pytestmark = pytest.mark.gpu


def test_fused_launches_record_their_split():
    shots = 8192
    w = W.make_random_drive(4, 4, 3, 64, 2, 0.01, 2, 5, plus_sites=tuple(range(16)), eps=0.5)
    g = T.TTN(w)
    g.profile_begin(timed=False)
    g.sample(shots, 1)
    g.profile_end()
    recs = [r for r in g.profile_launches() if r["flops"] == 8.0 * 64 * shots * 64 * 64]
    g.close()
    print(f"[records] {[(r['kernel'], r['splits']) for r in recs]}", flush=True)
    # the node states (4096 x 8192 outputs, K = 64) have as many flops and never split K
    split = [r for r in recs if r["splits"] > 1]
    assert recs and 2 * len(split) == len(recs) and all(r["kernel"] == 2 for r in recs)
