"""Rules of the forward that splits keys over waves: where its key tiles cross from one shard into the next, and how many rows an
fp32 workgroup has.  Compiled from the library's internal header and checked on the CPU."""
import ctypes
import os
import subprocess

import pytest

from tests import usp_testlib as tl
from tests.test_gpu_wave_split import CROSSING

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "usp_internal.h"
extern "C" int cross(int64_t n, int U, int R, int bs, int64_t row_bytes, int dtype, int hs, int rows) {
  return usp::wave_split_crossing(n, U, R, bs, row_bytes, dtype, hs, rows);
}
extern "C" int rows(int64_t Lq, int64_t heads, int64_t key_tiles, int causal) { return usp::wave_split_fp32_rows(Lq, heads, key_tiles, causal); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    where = tmp_path_factory.mktemp("wave_split")
    src, lib = where / "cross.cpp", where / "cross.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_07719_amd", "csrc"), str(src), "-o",
                    str(lib), "-Wl,--unresolved-symbols=ignore-all"], check=True)
    lib = ctypes.CDLL(str(lib))
    lib.cross.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 3
    lib.rows.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return lib


@pytest.fixture(scope="module")
def cross(lib):
    return lib.cross


KERNELS = [(tl.BF16, 32), (tl.FP32, 32), (tl.FP32, 16)]      # data type, rows per workgroup


@pytest.mark.parametrize("case", CROSSING)
def test_the_gpu_cases_cross(cross, case):
    """... whatever the data type and the rows per workgroup."""
    bs, L, hc, hk, hs, U, R, causal, zigzag, how = case
    for dtype, rows in KERNELS:
        assert cross(L // (U * R), U, R, bs, hk * hs * 4, dtype, hs, rows) == how


@pytest.mark.parametrize("dtype,rows", KERNELS)
@pytest.mark.parametrize("hs", [64, 128])
def test_short_shards_cross(cross, dtype, rows, hs):
    """Eight shards of 34 rows are nine tiles and not sixteen; a batch of one, whole tiles and one shard have nothing to cross."""
    assert cross(34, 8, 1, 2, 2048, dtype, hs, rows) == 1
    assert cross(24, 8, 4, 2, 2048, dtype, hs, rows) == 2
    assert cross(34, 8, 1, 1, 2048, dtype, hs, rows) == 0
    assert cross(64, 8, 1, 2, 2048, dtype, hs, rows) == 0
    assert cross(34, 1, 8, 2, 2048, dtype, hs, rows) == 0
    assert cross(66, 2, 2, 2, 2048, dtype, hs, rows) == (hs == 128 and rows == 32)      # ten tiles for twelve


def test_offsets_stay_within_32_bits(cross):
    """The last row of a tile lies at most 31 rows and (31 + n - 1) // n jumps of n (bs - 1) rows from its first."""
    for n in [1, 2, 3, 7, 31, 33, 100, 1000, 4097, 100001]:
        for row_bytes in [128, 2048, 16384]:
            for bs in [2, 3, 9, 100, 1000, 20000]:
                if cross(n, 8, 8, bs, row_bytes, tl.BF16, 128, 32):
                    jumps = (31 + n - 1) // n
                    assert (31 + jumps * n * (bs - 1)) * row_bytes + row_bytes < 2 ** 31
    assert cross(33, 8, 8, 2, 2048, tl.BF16, 128, 32) == 1 and cross(100001, 8, 8, 20, 2048, tl.BF16, 128, 32) == 0


@pytest.mark.parametrize("L,heads,R,causal,want", [
    (256, 4, 1, 0, 16), (1024, 4, 1, 0, 16), (1024, 5, 1, 0, 32),       # up to 128 workgroups of 32 rows
    (128, 36, 1, 1, 32), (104, 64, 4, 1, 32), (18, 256, 16, 1, 32),     # short walks under a mask: not above 128
    (64, 64, 1, 1, 16), (384, 12, 1, 1, 16), (512, 12, 1, 1, 16), (512, 16, 1, 1, 32), (1024, 8, 1, 1, 16), (1024, 9, 1, 1, 32),
])
def test_rows_of_an_fp32_workgroup(lib, L, heads, R, causal, want):
    """L rows of each ring rank; `heads` of all ranks and batch entries."""
    assert lib.rows(L, heads, R * -(-L // 32), causal) == want
