"""The 256-row tiles that the attention kernels cut rows and keys into: compiled from the library's internal header and
checked on the CPU."""
import ctypes
import os
import subprocess

import pytest

import paper_2405_07719_amd as usp
from tests import usp_testlib as tl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "usp_internal.h"
// tiles of the n blocks' common cut: their count is returned, their first and last rows are written
extern "C" int tiles(const usp_posdesc* d, int n, int64_t len, int causal, int64_t* begin, int64_t* end, int* in_run0) {
  const usp::RowTiles t = usp::common_row_tiles(d, n, len, causal);
  for (int i = 0; i < t.n; ++i) { begin[i] = t.begin(i); end[i] = t.end(i); }
  *in_run0 = t.in_run0;
  return t.n;
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    where = tmp_path_factory.mktemp("row_tiles")
    src, lib = where / "tiles.cpp", where / "tiles.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_07719_amd", "csrc"), str(src), "-o",
                    str(lib), "-Wl,--unresolved-symbols=ignore-all"], check=True)
    f = ctypes.CDLL(str(lib)).tiles

    def call(descs, length, causal=1):
        begin, end, in_run0 = (ctypes.c_int64 * 4096)(), (ctypes.c_int64 * 4096)(), ctypes.c_int()
        n = f((usp.usp_posdesc * len(descs))(*descs), len(descs), ctypes.c_int64(length), causal, begin, end, ctypes.byref(in_run0))
        return list(zip(begin[:n], end[:n])), in_run0.value

    return call


def ring(R, c):
    return [usp.usp_posdesc(r * c, c, (2 * R - 1 - r) * c, c) for r in range(R)]


def whole(cut, length):
    """Tiles follow one another without a gap, none is empty or longer than 256."""
    return cut[0][0] == 0 and cut[-1][1] == length and all(0 < e - b <= 256 for b, e in cut) and all(
        x[1] == y[0] for x, y in zip(cut, cut[1:]))


@pytest.mark.parametrize("R", [1, 2, 3, 4, 8, 16])
@pytest.mark.parametrize("c", [1, 20, 128, 255, 256, 257, 300, 513, 600, 1000, 1025, 1100, 1536, 2047])
def test_tiles_cover_every_block(tiles, R, c):
    blocks = ring(R, c)
    for descs in [[d] for d in blocks] + [blocks]:
        cut, in_run0 = tiles(descs, 2 * c)
        assert whole(cut, 2 * c)
        assert in_run0 == 0 or (cut[in_run0 - 1][1] == c == cut[in_run0][0])
    # the last ring rank's runs adjoin, and so the ring as a whole is cut in a row: as many tiles for every block
    assert tiles(blocks[-1:], 2 * c)[1] == 0
    assert len(tiles(blocks, 2 * c)[0]) == -(-2 * c // 256)
    # without a mask rows are cut in a row
    assert tiles(blocks[:1], 2 * c, 0)[1] == 0


@pytest.mark.parametrize("R", [2, 3, 8])
def test_blocks_that_are_cut_apart(tiles, R):
    """The rule as the GPU tests of these tiles state it."""
    for c in [*range(1, 1400), 2047, 4400]:
        for r in range(R):
            assert (tiles(ring(R, c)[r:r + 1], 2 * c)[1] > 0) == tl.cut_apart(c, R, r)
