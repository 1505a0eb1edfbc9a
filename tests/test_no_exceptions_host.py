"""No C++ exception leaves a C entry point: the library's host side is compiled with an allocator that can be told to fail, and
called where it works out how to cut a problem."""
import ctypes
import os
import subprocess

import pytest

import paper_2405_07719_amd as usp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include <hip/hip_runtime.h>
#define __align__(n)
#define HIP_SYMBOL(x) ((const void*)&(x))
#include "usp_api.cpp"
#include <cstdlib>
#include <new>
static int failing = 0;
extern "C" void fail_allocations(int on) { failing = on; }
void* operator new(size_t n) { if (failing) throw std::bad_alloc(); return malloc(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
// (of a .hip file; any cut will do)
namespace usp { BwdCut plan_bwd_cut(int, int64_t, int64_t, int, int, int, bool, bool) { return BwdCut{1, 2, 2}; } }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    where = tmp_path_factory.mktemp("host_side")
    src, out = where / "host.cpp", where / "host.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_07719_amd", "csrc"), str(src), "-o",
                    str(out), "-Wl,-Bsymbolic", "-Wl,--unresolved-symbols=ignore-all"], check=True)
    lib = ctypes.CDLL(str(out), mode=os.RTLD_LAZY)      # the launches of the .hip files stay unresolved
    lib.usp_attn_fwd_workspace_bytes.restype = ctypes.c_size_t
    lib.usp_attn_bwd_workspace_bytes.restype = ctypes.c_size_t
    return lib


def test_host_memory_runs_out(lib):
    p = usp.problem(1, 20480, 32, 8, 128, 8, 1, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    ptr = [ctypes.c_void_p(i << 40) for i in range(1, 11)]     # never followed: the calls end before any launch
    room = ctypes.c_size_t(lib.usp_attn_bwd_workspace_bytes(ctypes.byref(p), 1))     # (the larger of the two; no room for dS)
    lib.fail_allocations(1)
    try:
        assert lib.usp_attn_fwd_workspace_bytes(ctypes.byref(p), 1) == 0
        assert lib.usp_attn_fwd(ctypes.byref(p), *ptr[:5], 0, 1, ptr[5], room, None) == 7
        assert lib.usp_attn_bwd(ctypes.byref(p), *ptr[:9], 0, 1, ptr[9], room, None) == 7
    finally:
        lib.fail_allocations(0)
    assert lib.usp_attn_fwd_workspace_bytes(ctypes.byref(p), 1) > 0     # nothing half done was kept
    assert lib.usp_attn_bwd_workspace_bytes(ctypes.byref(p), 1) > 0
