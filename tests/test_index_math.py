"""Index arithmetic that the host code and the kernels share, compiled for the
host and called at sizes no test could allocate."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHARED, INDEPENDENT, ROSENBLUTH = 0, 1, 2


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    (d / "w.cpp").write_text(
        '#include "pperm_internal.h"\n'
        'extern "C" uint32_t row_of(uint32_t mode, uint32_t s) { return pperm::pooled_row(mode, s); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "paper_2002_03000_amd", "csrc"),
                    str(d / "w.cpp"), "-o", str(d / "w.so")], check=True, timeout=120)
    return ctypes.CDLL(str(d / "w.so"))


@pytest.mark.parametrize("mode,rows", [(SHARED, 1), (INDEPENDENT, 4096), (ROSENBLUTH, 1)])
def test_pooled_rows_lie_in_the_pooled_sums(lib, mode, rows):
    # (a chained launch keeps such a row per epoch, with nothing after the last)
    for s in (0, 1, 16, 4095):
        assert lib.row_of(mode, s) == (s if rows > 1 else 0) < rows
