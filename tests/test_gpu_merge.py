"""The merge at the edges of its blocks of 1024 rows and 64-row waves, and the
work queue that a launch leaves cleared for the next.  Bit for bit against the
oracle."""
import numpy as np
import pytest

import oracle
from parity_util import assert_epoch_equal, assert_pooled_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kw", [
    (1, {}), (2, {}), (64, {}), (65, {}), (1023, {}), (1024, {}), (1025, {}), (2049, {}),
    (1025, dict(observables=True)), (1030, dict(walks_per_wave=2)),
])
def test_merge_block_edges_match_oracle(N, kw):
    from paper_2002_03000_amd import ParallelFlatPERM
    n_max = 9                      # (10 lengths: one full strip of 8 columns and a short one)
    g = ParallelFlatPERM(2, n_max, N, 95, **kw)
    o = oracle.Oracle(2, n_max, N, 95, observables=kw.get("observables", False))
    for runs in ((1,), (2, 1), (1, 1, 1)):
        for T in runs:             # (several launches before a merge share the queue)
            g.run_tours(T)
            o.run_tours(T)
        assert_epoch_equal(g, o, label=f"N={N} runs={runs}")
        g.merge_epoch()
        o.merge_epoch()
        assert_pooled_equal(g, o, f"N={N} runs={runs}")
    if kw.get("observables"):
        rec = g.records("obs_G")[: n_max + 1]
        assert np.array_equal(rec["m"], o.GR["m"]) and np.array_equal(rec["e"], o.GR["e"])
