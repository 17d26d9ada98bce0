"""Rosenbluth problems in a chained launch: one row of pooled sums for all
sequences, in every epoch.  Bit for bit against the oracle."""
import pytest

from parity_util import assert_pooled_equal, assert_stats_equal, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n_max,N,kw", [(3, 200, 3000, {}), (2, 40, 1, {}), (3, 250, 700, dict(sums_global=True))])
def test_rosenbluth_job_matches_oracle(dim, n_max, N, kw):
    from paper_2002_03000_amd import run_job
    schedule = [1, 2, 3]
    g, o = make_pair(dim, n_max, N, 99, mode="rosenbluth", **kw)
    run_job([g], [schedule])
    for T in schedule:
        o.run_tours(T)
        o.merge_epoch()
    assert_pooled_equal(g, o, f"N={N}")
    assert_stats_equal(g.sequence_stats(), o.stats)
