"""Runs whose sequences are more than the waves of the launch: their tours go out
in parts, handed from wave to wave.  Bit for bit against the oracle, over sums in
LDS and in global memory, every key format and mode, and a step cap that stops
some sequences in a part of theirs."""
import numpy as np
import pytest

import oracle
from parity_util import assert_epoch_equal, assert_pooled_equal

pytestmark = pytest.mark.gpu

MODES = {"shared": oracle.MODE_SHARED, "independent": oracle.MODE_INDEPENDENT,
         "rosenbluth": oracle.MODE_ROSENBLUTH}


@pytest.mark.parametrize("dim,n_max,N,tours,mode,kw", [
    (2, 127, 9000, (1, 33), "shared", {}),
    (2, 1023, 1600, (1, 5), "shared", {}),
    (3, 250, 9001, (1, 17), "shared", dict(sums_global=True)),
    (3, 255, 5000, (1, 17), "independent", {}),
    (3, 700, 9000, (7,), "rosenbluth", dict(sums_global=True)),
    (3, 2300, 2600, (2,), "rosenbluth", dict(sums_global=True)),
])
def test_parts_match_oracle(dim, n_max, N, tours, mode, kw):
    from paper_2002_03000_amd import ParallelFlatPERM
    g = ParallelFlatPERM(dim, n_max, N, 96, mode=mode, **kw)
    o = oracle.Oracle(dim, n_max, N, 96, mode=MODES[mode])
    for T in tours:
        g.run_tours(T)
        o.run_tours(T)
        assert_epoch_equal(g, o, label=f"N={N} T={T}")
        g.merge_epoch()
        o.merge_epoch()
        assert_pooled_equal(g, o, f"N={N} T={T}")


def test_step_cap_counts_over_the_parts():
    from paper_2002_03000_amd import ParallelFlatPERM, PPermError
    g = ParallelFlatPERM(2, 127, 9000, 97, step_cap=6000)
    o = oracle.Oracle(2, 127, 9000, 97, step_cap=6000)
    for T in (1, 40):
        g.run_tours(T)
        o.run_tours(T)
    st = g.sequence_stats()
    for f in ("steps", "events", "digest", "capped", "tours"):
        assert np.array_equal(st[f], o.stats[f]), f
    assert 0 < int((st["capped"] != 0).sum()) < 9000
    with pytest.raises(PPermError, match="EOVERFLOW"):
        g.sync()


def test_captured_epoch_of_parts_replays():
    import torch
    from paper_2002_03000_amd import ParallelFlatPERM
    g = ParallelFlatPERM(2, 127, 9000, 98)
    o = oracle.Oracle(2, 127, 9000, 98)
    graph = g.epoch_graph(33)
    for rep in range(3):
        graph.launch()
        torch.cuda.synchronize()
        o.run_tours(33)
        o.merge_epoch()
        assert_pooled_equal(g, o, f"replay {rep}")
    graph.close()
