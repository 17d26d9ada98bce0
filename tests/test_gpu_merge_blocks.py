"""The merge where its blocks change size (64, 128, 256, 512 and 1024 rows, one, two
and three passes).  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from parity_util import assert_pooled_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_max,N,kw", [
    (9, 512, {}), (9, 513, {}), (9, 4096, {}), (9, 4097, {}), (9, 8193, dict(observables=True)), (9, 20001, {}),
    (5000, 900, {}), (600, 700, {}), (600, 1024, dict(observables=True)), (600, 1030, {}), (1100, 1500, {}),
    (2, 524289, {}), (1, 1100000, {}),
])
def test_merge_blocks_match_oracle(n_max, N, kw):
    from paper_2002_03000_amd import ParallelFlatPERM
    g = ParallelFlatPERM(3, n_max, N, 103, mode="rosenbluth", **kw)
    o = oracle.Oracle(3, n_max, N, 103, mode=oracle.MODE_ROSENBLUTH, observables=kw.get("observables", False))
    for _ in range(2):
        g.run_tours(1)
        g.merge_epoch()
        o.run_tours(1)
        o.merge_epoch()
        assert_pooled_equal(g, o, f"n_max={n_max} N={N}")
    assert not g.records("L")["m"].any() and not g.view("m").cpu().numpy().any()
    if kw.get("observables"):
        rec = g.records("obs_G")[: n_max + 1]
        assert np.array_equal(rec["m"], o.GR["m"]) and np.array_equal(rec["e"], o.GR["e"])
