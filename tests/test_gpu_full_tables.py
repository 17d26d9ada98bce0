"""Walks in tables two thirds full, the longest there are: their last steps pass by
sites outside their places.  Bit for bit against the oracle."""
import pytest

from parity_util import assert_epoch_equal, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_max,N,kw", [(10921, 96, {}), (1022, 400, dict(hash_slots=1536, sums_global=True)),
                                        (2046, 300, dict(hash_slots=3072, sums_global=True))])
def test_full_tables_match_oracle(n_max, N, kw):
    g, o = make_pair(3, n_max, N, 3, mode="rosenbluth", **kw)
    for T in (1, 2):
        g.run_tours(T)
        o.run_tours(T)
        assert_epoch_equal(g, o, label=f"n_max={n_max}")
    assert int(o.H[:, n_max].sum()) > 0                 # (some walks have the full length)
