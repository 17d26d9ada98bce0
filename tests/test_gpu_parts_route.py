"""That the launches in parts, and the calls that must not become one, take the
route they are meant to: a launch in parts leaves the number of hand-overs at the
head of its list, which lies in the merge's scratch; any other leaves the scratch
alone."""
import importlib.util
import os

import numpy as np
import pytest
import torch

import oracle
import test_gpu_parts

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
UNTOUCHED = 0x5A5A5A5A5A5A


def _hand_overs(g, tours):
    """Entries of the list of a call's launch in parts, or None."""
    at = g.layout.scratch
    head = g.workspace[at:at + 8].view(torch.int64)
    head.fill_(UNTOUCHED)
    g.run_tours(tours)
    n = int(head.item())
    return None if n == UNTOUCHED else n


def _cases():
    mark = next(m for m in test_gpu_parts.test_parts_match_oracle.pytestmark if m.name == "parametrize")
    return mark.args[1]


@pytest.mark.parametrize("dim,n_max,N,tours,mode,kw", _cases())
def test_the_parts_tests_run_in_parts(dim, n_max, N, tours, mode, kw):
    from paper_2002_03000_amd import ParallelFlatPERM
    spec = importlib.util.spec_from_file_location("bench_parts", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    g = ParallelFlatPERM(dim, n_max, N, 96, mode=mode, **kw)
    for T in tours:
        shape = g.launch_shape()
        assert shape["workgroups"] < N
        part = max(-(-T // 4), -(-2048 // (n_max + 1)))
        parts = -(-T // part)
        name = bench.growth_kernel(N, n_max, T, shape, bool(kw.get("sums_global")))
        assert name.startswith("part" if parts > 1 else "batch")
        assert _hand_overs(g, T) == (N * (parts - 1) if parts > 1 else None), T
        g.merge_epoch()
    assert parts > 1


def test_short_rosenbluth_tours_stay_whole():
    # (square walks are trapped after 71 steps on average, however long n_max)
    from paper_2002_03000_amd import ParallelFlatPERM
    g = ParallelFlatPERM(2, 2000, 4400, 100, mode="rosenbluth", sums_global=True)
    assert g.launch_shape()["workgroups"] < 4400
    assert _hand_overs(g, 8) is None
    assert _hand_overs(g, 64) is None
    assert _hand_overs(g, 200) == 4400                   # (parts of 113 tours)


def test_as_many_tours_as_a_call_may_ask_for():
    from paper_2002_03000_amd import ParallelFlatPERM
    N, T = 4200, 2 ** 32 - 1
    g = ParallelFlatPERM(2, 60, N, 101, mode="independent", step_cap=300)
    o = oracle.Oracle(2, 60, N, 101, mode=oracle.MODE_INDEPENDENT, step_cap=300)
    assert _hand_overs(g, T) == 3 * N
    o.run_tours(T)
    st = g.sequence_stats()
    for f in ("steps", "events", "digest", "capped", "tours"):
        assert np.array_equal(st[f], o.stats[f]), f
    assert st["capped"].all()
