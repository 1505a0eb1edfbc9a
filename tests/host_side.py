"""The library's host side, compiled with g++ for the CPU, with launchers that record what they are asked to launch."""
from __future__ import annotations

import ctypes
import os
import subprocess

import paper_2405_07719_amd as usp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
#include <hip/hip_runtime.h>
#define __align__(n)
#define HIP_SYMBOL(x) ((const void*)&(x))
#include "usp_api.cpp"
namespace usp {
// (of a .hip file; any cut will do)
BwdCut plan_bwd_cut(int, int64_t, int64_t, int, int, int, bool, bool) { return BwdCut{1, 2, 2}; }
"""
RECORDERS = """
// kind of the last launch that attends: 1 waves, 2 whole, 3 every tile cut, 4 the last tiles cut, 5 listed, 6 a block
struct Route { int kind, parts, whole, cut, different_rows, launches, v_transposed; };
static Route route;
int launch_wave_split_usp_fwd(const usp_problem&, const void*, const void*, const void*, void*, float*, int, int, float, hipStream_t) {
  route.kind = 1; ++route.launches;
  return USP_OK;
}
int launch_ring_attn_fwd(const void*, const void* const*, const void* const*, const usp_posdesc*, int, void*, float*, int, int64_t, int64_t,
                         int, int, int, float, int, const usp_posdesc&, int, int, hipStream_t, const SeqLayoutIO*, const RingState*, bool v_transposed) {
  route.kind = 2; ++route.launches;
  route.v_transposed = v_transposed;
  return USP_OK;
}
int launch_attn_fwd_partials(const void*, const void* const*, const void* const*, const usp_posdesc*, const int*, int n_blocks, float* const*,
                             float* const*, int, int64_t, int64_t, int, int, int, float, int, const usp_posdesc&, hipStream_t,
                             const SeqLayoutIO*, const MixedLaunch* mixed) {
  route.kind = !mixed ? 3 : mixed->n_listed ? 5 : 4; ++route.launches;
  route.parts = n_blocks;
  if (mixed) route.cut = mixed->n_split_tiles, route.v_transposed = mixed->v_transposed;
  if (mixed && mixed->n_listed) {
    for (int i = 0; i < mixed->n_listed; ++i) ++(mixed->listed[i] >> kListedTileBits == kListedWhole ? route.whole : route.cut);
    for (int j = 1; j < n_blocks; ++j) route.different_rows |= mixed->part_row0[j] != mixed->part_row0[0];
  }
  return USP_OK;
}
int launch_block_attn_fwd(const void*, const void*, const void*, void*, float*, int, int64_t, int64_t, int, int, int, float, int,
                          const usp_posdesc&, const usp_posdesc&, int, int, hipStream_t, const RingState*) {
  route.kind = 6; ++route.launches;
  return USP_OK;
}
int launch_lse_merge(const void* const*, const float* const*, int, void*, float*, int, int64_t, int, int, int, int, hipStream_t,
                     const SeqLayoutIO*, int64_t, const int64_t*) { return USP_OK; }
int launch_layout_a2a(const usp_problem&, int, int, const void*, void*, int, int, int, hipStream_t, int) { return USP_OK; }
int launch_layout_a2a_multi(const usp_problem&, int, int, int, const void* const*, void* const*, int, int, int, hipStream_t, int) { return USP_OK; }
int launch_layout_a2a_vt(const usp_problem&, int, const void*, void*, int, int, int, hipStream_t, int) { return USP_OK; }
}  // namespace usp
extern "C" void last_route(int* out) {
  using usp::route;
  const int r[] = {route.kind, route.parts, route.whole, route.cut, route.different_rows, route.launches, route.v_transposed};
  for (int i = 0; i < 7; ++i) out[i] = r[i];
  route = usp::Route{};
}
// ring ranks whose items have been worked out
extern "C" int ranks_listed(const usp_problem* p) {
  int n = 0;
  if (ring_in_one_launch(*p))
    for (const auto& items : plans_of(*p)->items) n += items != nullptr;
  return n;
}
// when the last of n items, each for `heads` heads, is done
extern "C" double played(int heads, const double* us, int n) {
  PlayedLaunch launch(heads);
  for (int i = 0; i < n; ++i) launch.give(us[i], 1e30);
  return launch.end();
}
extern "C" int block_goes_to_waves(int bs, int64_t Lq, int64_t Lk, int hq, int hs, int causal, int dtype) {
  return usp::block_goes_to_waves(bs, Lq, Lk, hq, hs, causal, dtype);
}
"""
KINDS = {1: "waves", 2: "whole", 3: "every tile cut", 4: "last tiles cut", 5: "listed", 6: "blocks"}


def compile_host_side(where, source):
    """The shared library made of `source`; launches of .hip files that it does not define stay unresolved."""
    src, out = where / "host.cpp", where / "host.so"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_07719_amd", "csrc"), str(src), "-o",
                    str(out), "-Wl,-Bsymbolic", "-Wl,--unresolved-symbols=ignore-all"], check=True)
    return ctypes.CDLL(str(out), mode=os.RTLD_LAZY)


class HostSide:
    def __init__(self, where):
        self.lib = compile_host_side(where, HEAD + RECORDERS)
        self.lib.usp_attn_fwd_workspace_bytes.restype = ctypes.c_size_t
        self.lib.played.restype = ctypes.c_double

    long = staticmethod(ctypes.c_int64)

    def query(self, p, n_ranks=1):
        return self.lib.usp_attn_fwd_workspace_bytes(ctypes.byref(p), n_ranks)

    def forward(self, p, rank_begin, rank_end):
        """What usp_attn_fwd launches last: dict of kind, parts (of the keys), whole and cut (listed items; or cut tiles),
        different_rows (partial results that begin with different rows), launches, v_transposed (V in transposed tiles)."""
        ptr = [ctypes.c_void_p(i << 40) for i in range(1, 7)]     # aligned, apart, never followed
        room = ctypes.c_size_t(self.query(p, rank_end - rank_begin))
        st = self.lib.usp_attn_fwd(ctypes.byref(p), *ptr[:5], rank_begin, rank_end, ptr[5], room, None)
        out = (ctypes.c_int * 7)()
        self.lib.last_route(out)
        assert st == 0, st
        return dict(zip(("kind", "parts", "whole", "cut", "different_rows", "launches", "v_transposed"), [KINDS[out[0]], *out[1:]]))

    def ranks_listed(self, p):
        return self.lib.ranks_listed(ctypes.byref(p))

    def played(self, heads, us):
        return self.lib.played(heads, (ctypes.c_double * len(us))(*us), len(us))


def problem(bs, L, hc, hk, hs, U, R, causal=True, zigzag=True, dtype=usp.USP_BF16):
    return usp.problem(bs, L, hc, hk, hs, U, R, causal, usp.USP_SPLIT_ZIGZAG if zigzag else usp.USP_SPLIT_CONTIG, dtype)
