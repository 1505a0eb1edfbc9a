"""Where the second product of the head-size-64 forward runs a tile behind: blocks that are long enough, and of cut blocks pieces that
are.  Compiled from the library's internal header and checked on the CPU."""
import ctypes

import pytest

from tests.host_side import compile_host_side

SOURCE = """
#include "usp_internal.h"
extern "C" int trails(int64_t Lk, int64_t piece) { return usp::second_product_trails(Lk, piece); }
"""


@pytest.fixture(scope="module")
def trails(tmp_path_factory):
    f = compile_host_side(tmp_path_factory.mktemp("trailing"), SOURCE).trails
    f.argtypes = [ctypes.c_int64, ctypes.c_int64]
    return f


# keys of a block, keys of a piece on the average
@pytest.mark.parametrize("Lk,piece,yes", [(2047, 2047, False), (2048, 2048, True), (4444, 888, False), (2312, 1156, False),
                                          (4890, 1222, False), (8888, 1269, True), (9128, 1521, True), (17776, 2222, True)])
def test_rule(trails, Lk, piece, yes):
    assert bool(trails(Lk, piece)) == yes
