"""The growth kernel that a bench line names, for the workloads' launch shapes,
and its committed counter summaries."""
import importlib.util
import os

import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_kernel_name", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("p,workgroups,long_walk,kernel", [
    (workloads.PARALLEL_3D, 4096, True, "part_long_kernel"),
    (workloads.PARALLEL_3D, 1024, False, "part_kernel"),
    (workloads.PARALLEL_2D, 3072, False, "part_kernel"),
    (workloads.PARALLEL_2D, 4096, True, "batch_long_kernel"),
    (workloads.LONG_2D, 256, True, "batch_long_kernel"),
    (workloads.PLAIN_2D, 1, False, "batch_kernel"),
])
def test_growth_kernel(bench, p, workgroups, long_walk, kernel):
    shape = {"walks_per_wave": 1, "workgroups": workgroups}
    assert bench.growth_kernel(p.n_sequences, p.n_max, p.tours_per_epoch, shape, long_walk) == kernel
    shape["walks_per_wave"] = 4
    assert bench.growth_kernel(p.n_sequences, p.n_max, p.tours_per_epoch, shape, False) == "run_kernel"


@pytest.mark.parametrize("summary", ["part_long_kernel_parallel3d", "part_kernel_parallel2d"])
def test_summaries_are_found_under_the_kernel_name(bench, summary):
    for kind in ("kernel_trace", "sq_counters", "traffic"):
        assert os.path.exists(os.path.join(bench.PROFILES, f"{summary}_{kind}.md"))


def test_bytes_per_step_follow_the_key_format(bench):
    import re
    src = open(os.path.join(ROOT, "paper_2002_03000_amd", "csrc", "pperm_internal.h")).read()
    last = int(re.search(r"COMPACT3_MAX_N = (\d+);", src).group(1))
    assert [bench.lds_bytes_per_step(3, n) for n in (1, last, last + 1)] == [24, 24, 48]
    assert bench.lds_bytes_per_step(2, last + 1) == 16
