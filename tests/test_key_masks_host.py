"""Which key tiles a wave of the 256-row forward masks: compiled from the library's internal header and checked on the CPU
against the positions themselves."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KT = 64
SOURCE = """
#include "usp_internal.h"
extern "C" void unmasked(int causal, int has_rows, int all, int qmin, const int* run, int Lk, int na, int t0, int t1, int* out) {
  const usp::UnmaskedTiles u = usp::unmasked_key_tiles(64, causal, has_rows != 0, all != 0, qmin, run[0], run[1], run[2], run[3], Lk, na, t0, t1);
  out[0] = u.a; out[1] = u.b0; out[2] = u.b1;
}
"""


@pytest.fixture(scope="module")
def unmasked(tmp_path_factory):
    where = tmp_path_factory.mktemp("key_masks")
    src, lib = where / "masks.cpp", where / "masks.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_07719_amd", "csrc"), str(src), "-o",
                    str(lib), "-Wl,--unresolved-symbols=ignore-all"], check=True)
    f = ctypes.CDLL(str(lib)).unmasked

    def call(causal, has_rows, every, qmin, runs, Lk, na, t0, t1):
        out = (ctypes.c_int * 3)()
        f(causal, has_rows, every, qmin, (ctypes.c_int * 4)(*runs), Lk, na, t0, t1, out)
        return out

    return call


def walk(causal, qmax, runs, Lk):
    """The key tiles that a query tile walks, whose last row stands at qmax: first and last of both visible ranges."""
    if not causal:
        n = -(-Lk // KT)
        return n, n, n
    s0, n0, s1, n1 = runs
    c0, c1 = max(0, min(qmax - s0 + 1, n0)), max(0, min(qmax - s1 + 1, n1))
    na = -(-c0 // KT)
    t0 = max(n0 // KT, na) if c1 else na
    return na, t0, max(-(-(n0 + c1) // KT), t0) if c1 else t0


@pytest.mark.parametrize("seed", range(4))
def test_masks_follow_the_positions(unmasked, seed):
    rng = random.Random(seed)
    for _ in range(400):
        n0, n1 = rng.choice([0, 32, 64, 100, 640, 1000]), rng.choice([0, 40, 64, 700, 1024])
        if n0 + n1 == 0:
            continue
        s0 = rng.randrange(0, 2000)
        runs = (s0, n0, s0 + n0 + rng.choice([0, 1, 500, 3000]), n1)
        Lk = n0 + n1
        pos = [runs[0] + i if i < n0 else runs[2] + i - n0 for i in range(Lk)]
        causal = rng.random() < 0.85
        has_rows = rng.random() < 0.6
        qmin = rng.randrange(0, 7000)
        qmax = qmin + rng.randrange(0, 256)          # of the whole query tile
        na, t0, t1 = walk(causal, qmax, runs, Lk)
        places = list(range(na)) + list(range(t0, t1))
        every = rng.random() < 0.7                   # whether a wave without rows leaves out the second range's masks too
        a, b0, b1 = unmasked(causal, has_rows, every, qmin, runs, Lk, na, t0, t1)
        for place, tile in enumerate(places):
            keys = range(tile * KT, min(Lk, tile * KT + KT))
            full = len(keys) == KT
            one_run = not causal or keys[-1] < n0 or keys[0] >= n0
            free = place < a or b0 <= place < b1
            if causal and has_rows:
                assert free == (full and one_run and pos[keys[-1]] <= qmin), (runs, qmin, tile)
            elif not causal or every or place < na:          # nothing to hide but the keys that are not there
                assert free == full, (runs, causal, tile)
