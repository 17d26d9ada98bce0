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
        'extern "C" uint32_t row_of(uint32_t mode, uint32_t s) { return pperm::pooled_row(mode, s); }\n'
        'extern "C" bool digest_word(uint64_t k) { return pperm::is_digest_word(k); }\n'
        'extern "C" uint64_t part(uint32_t dim, uint32_t mode, uint32_t n, uint32_t T)'
        ' { return pperm::part_tours(dim, mode, n, T); }\n'
        'extern "C" uint32_t block(uint32_t rows, uint32_t ncols, bool first)'
        ' { return pperm::merge_block(rows, ncols, first); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "paper_2002_03000_amd", "csrc"),
                    str(d / "w.cpp"), "-o", str(d / "w.so")], check=True, timeout=120)
    lib = ctypes.CDLL(str(d / "w.so"))
    lib.digest_word.argtypes, lib.digest_word.restype = [ctypes.c_uint64], ctypes.c_bool
    lib.part.restype = ctypes.c_uint64
    lib.block.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_bool]
    return lib


@pytest.mark.parametrize("mode,rows", [(SHARED, 1), (INDEPENDENT, 4096), (ROSENBLUTH, 1)])
def test_pooled_rows_lie_in_the_pooled_sums(lib, mode, rows):
    # (a chained launch keeps such a row per epoch, with nothing after the last)
    for s in (0, 1, 16, 4095):
        assert lib.row_of(mode, s) == (s if rows > 1 else 0) < rows


def test_a_new_context_seeds_the_digest_of_every_sequence(lib):
    # ten 64-bit counters a sequence, the digest the ninth; word 2^32 of the
    # statistics belongs to sequence 214,748,364
    for s in (0, 1, 214748363, 214748364, 214748365, 429496729, 2 ** 32 - 1):
        assert [w for w in range(20) if lib.digest_word(20 * s + w)] == [16], s


@pytest.mark.parametrize("dim,mode,n_max,tours,part", [
    (2, SHARED, 500, 64, 16), (3, SHARED, 1000, 32, 8), (2, SHARED, 127, 33, 16), (2, SHARED, 1, 4096, 1024),
    (3, INDEPENDENT, 255, 17, 8),
    # a trapped walk's steps, not n_max: 2048 / 71 = 28.8, and 2048 / 3950 < 1;
    # on the square lattice four rows of them: 4 * 2001 / 71 = 112.7
    (2, ROSENBLUTH, 500, 8, 29), (2, ROSENBLUTH, 2000, 8, 113), (2, ROSENBLUTH, 16383, 256, 924), (2, ROSENBLUTH, 500, 200, 50), (2, ROSENBLUTH, 60, 8, 34),
    (3, ROSENBLUTH, 700, 9, 3), (3, ROSENBLUTH, 9000, 3, 1),
    # as many tours as a call may ask for
    (3, INDEPENDENT, 2, 2 ** 32 - 1, 2 ** 30), (2, ROSENBLUTH, 5000, 2 ** 32 - 4, 2 ** 30 - 1),
])
def test_a_part_has_a_quarter_of_the_tours_or_2048_steps(lib, dim, mode, n_max, tours, part):
    assert lib.part(dim, mode, n_max, tours) == part


def test_merge_blocks(lib):
    # (rows, columns, first pass): the block
    for args, block in [((1, 2, True), 1024), ((512, 21, True), 1024), ((513, 21, True), 64), ((1000, 51, True), 64),
                        ((1024, 513, True), 1024), ((1025, 513, True), 64), ((1025, 51, True), 64),
                        ((4096, 51, True), 64), ((4097, 51, True), 128), ((16384, 21, True), 256),
                        ((1025, 1600, True), 512), ((16384, 1001, True), 512), ((524288, 2, True), 512),
                        ((524289, 2, True), 1024), ((1024, 51, False), 1024), ((1025, 51, False), 64),
                        ((700, 5001, True), 1024), ((1000, 5001, True), 64), ((1065, 2501, True), 512),
                        ((1279, 10001, True), 64), ((1280, 10001, True), 512), ((1000, 10001, False), 1024)]:
        assert lib.block(*args) == block, args
    # every merge ends, takes at most two passes up to 2^20 sequences, and its partial sums
    # fit the scratch of ceil(N / 64) rows, whatever its size
    for ncols in (2, 17, 501, 513, 10001, 32767):
        for N in [2 ** k + d for k in range(32) for d in (-1, 0, 1) if 0 < 2 ** k + d < 2 ** 32]:
            rows, passes = N, 0
            while True:
                block = lib.block(rows, ncols, passes == 0)
                passes += 1
                assert 64 <= block <= 1024 and block & (block - 1) == 0
                if rows <= block:
                    break
                rows = -(-rows // block)
                assert rows <= -(-N // 64)
            assert passes <= (1 if N <= 512 else 2 if N <= 2 ** 20 else 4), (N, ncols)
