"""Estimates read right after work that another stream than the context's own did."""
import pytest
import torch

from parity_util import assert_pooled_equal, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own", [False, True])
def test_estimates_wait_for_a_job_on_the_default_stream(own):
    # (about 0.1 s of chained epochs; the context's own stream has nothing to do)
    from paper_2002_03000_amd import run_job
    schedule = [1, 1, 2, 4, 8, 16]
    stream = torch.cuda.Stream() if own else torch.cuda.current_stream()
    g, o = make_pair(2, 400, 64, 102, stream=stream)
    torch.cuda.synchronize()
    scratch = run_job([g], [schedule], stream=torch.cuda.default_stream())
    log_cn, hist, tours = g.estimates()
    for T in schedule:
        o.run_tours(T)
        o.merge_epoch()
    assert tours == 64 * sum(schedule) and (hist == o.HG).all()
    assert abs(log_cn - o.log_estimates()).max() < 1e-9
    torch.cuda.synchronize()
    assert_pooled_equal(g, o)
    del scratch


@pytest.mark.parametrize("N", [1, 388, 389, 600])
def test_estimates_of_large_independent_sums(N):
    # (112 records and counts a sequence: 388 sequences are the last below 1 MiB)
    g, o = make_pair(2, 100, N, 104, mode="independent")
    for T in (1, 2):
        g.run_tours(T)
        g.merge_epoch()
        o.run_tours(T)
        o.merge_epoch()
    log_cn, hist, tours = g.estimates()
    assert tours == int(o.MG.sum()) and (hist == o.HG.sum(axis=0)).all()
    assert abs(log_cn - o.log_estimates()).max() < 1e-9
