"""The wave walker where its table, its key formats and its run-ahead block
change over: tables so small that sites find all their places taken, the last
length of the short cubic keys and the first of the long ones, step caps inside
and at the edges of a random block.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from parity_util import assert_epoch_equal, assert_pooled_equal, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n_max,N,slots,mode,kw", [
    (3, 63, 300, 96, "shared", dict(sums_global=True)),
    (3, 63, 300, 96, "rosenbluth", dict(sums_global=True)),
    (3, 126, 200, 192, "independent", dict(sums_global=True)),
    (3, 63, 200, 96, "shared", dict(sums_global=True, observables=True)),
    (2, 41, 300, 64, "shared", dict(sums_global=True)),
    (2, 1, 5, 64, "shared", dict()),
    (3, 2, 5, 64, "rosenbluth", dict()),
])
def test_small_tables_match_oracle(dim, n_max, N, slots, mode, kw):
    # (a full cubic walk of 63 steps in 96 slots meets a site with all places
    # taken about once in nine)
    from paper_2002_03000_amd import ParallelFlatPERM
    codes = {"shared": oracle.MODE_SHARED, "independent": oracle.MODE_INDEPENDENT,
             "rosenbluth": oracle.MODE_ROSENBLUTH}
    g = ParallelFlatPERM(dim, n_max, N, 91, mode=mode, hash_slots=slots, **kw)
    o = oracle.Oracle(dim, n_max, N, 91, mode=codes[mode], observables=kw.get("observables", False))
    for T in (1, 6, 20):
        g.run_tours(T)
        o.run_tours(T)
        assert_epoch_equal(g, o, label=f"small table T={T}")
        g.merge_epoch()
        o.merge_epoch()
        assert_pooled_equal(g, o, f"small table T={T}")
    if kw.get("observables"):
        rec = g.records("obs_G")[: n_max + 1]
        assert np.array_equal(rec["m"], o.GR["m"]) and np.array_equal(rec["e"], o.GR["e"])


@pytest.mark.parametrize("n_max", [2063, 2064])
@pytest.mark.parametrize("sums_global", [False, True])
def test_key_formats_match_oracle(n_max, sums_global):
    g, o = make_pair(3, n_max, 40, 92, sums_global=sums_global)
    for T in (1, 2):
        g.run_tours(T)
        o.run_tours(T)
        assert_epoch_equal(g, o, label=f"n_max={n_max}")
        g.merge_epoch()
        o.merge_epoch()
        assert_pooled_equal(g, o, f"n_max={n_max}")


@pytest.mark.parametrize("cap", [1, 62, 63, 64, 65, 127, 200])
def test_step_cap_stops_at_the_step(cap):
    from paper_2002_03000_amd import ParallelFlatPERM
    g = ParallelFlatPERM(3, 120, 30, 93, step_cap=cap)
    o = oracle.Oracle(3, 120, 30, 93, step_cap=cap)
    g.run_tours(3)
    o.run_tours(3)
    st = g.sequence_stats()
    for f in ("steps", "events", "digest", "capped", "tours"):
        assert np.array_equal(st[f], o.stats[f]), f
    assert st["capped"].any()


@pytest.mark.parametrize("n_max", [14, 15, 16, 30, 31])
@pytest.mark.parametrize("mode", ["shared", "rosenbluth"])
def test_walks_stop_at_n_max_with_and_without_a_guard_record(n_max, mode):
    # (rows are padded to 16 records: 15 and 31 leave no room for the guard)
    codes = {"shared": oracle.MODE_SHARED, "rosenbluth": oracle.MODE_ROSENBLUTH}
    from paper_2002_03000_amd import ParallelFlatPERM
    for obs in (False, True):
        g = ParallelFlatPERM(2, n_max, 60, 94, mode=mode, observables=obs)
        o = oracle.Oracle(2, n_max, 60, 94, mode=codes[mode], observables=obs)
        for T in (1, 9):
            g.run_tours(T)
            o.run_tours(T)
            assert_epoch_equal(g, o, label=f"n_max={n_max}")
            g.merge_epoch()
            o.merge_epoch()
            assert_pooled_equal(g, o, f"n_max={n_max}")
