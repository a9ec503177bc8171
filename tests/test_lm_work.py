"""The division of the LM head's work (csrc/lm_work.h), compiled for the host:
every position tile meets the same vocabulary ranges, the ranges cover the
vocabulary once and in order, the workgroups take every (position tile, range)
once, and the partial results fit the room that is reserved for them."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_02955_amd", "csrc")
SHIM = r"""
#include "lm_work.h"
using namespace fdllm;
extern "C" void work(int n, int V, int d, int* out) {
  const LmWork w = lm_work(n, V, d);
  out[0] = w.mt; out[1] = w.pt; out[2] = w.unit; out[3] = w.nb; out[4] = w.k;
}
extern "C" void ranges(int n, int V, int d, int* first) {
  const LmWork w = lm_work(n, V, d);
  for (int s = 0; s <= w.k; ++s) first[s] = lm_first(w, s);
}
extern "C" int segments(int n, int V, int d, int* times) {      // the longest workgroup's, -1 for one out of range
  const LmWork w = lm_work(n, V, d);
  int most = 0;
  for (int g = 0; g < kLmGroups; ++g) {
    int own = 0;
    for (int u = lm_seg_first(w, g); u < lm_seg_end(w, g); u += kLmGroups / kLmXcds, ++own) {
      if (u < 0 || u >= w.mt * w.k) return -1;
      ++times[u];
    }
    if (own > most) most = own;
  }
  return most;
}
extern "C" long long max_partials(long long n, int V) { return (long long)lm_max_partials(n, V); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("lm_work")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.max_partials.restype = ctypes.c_longlong
    lib.max_partials.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return lib


COUNTS = [1, 31, 32, 33, 64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513, 700, 768, 769, 1280, 1281, 2500,
          4096, 4097, 11000, 33000, 65536, 65537, 70000, 300000]


@pytest.mark.parametrize("V", [1, 15, 16, 255, 256, 257, 4099, 16000, 50257, 126464, 152000, 1 << 21])
@pytest.mark.parametrize("d", [64, 1024, 4096])
def test_division(lib, V, d):
    for n in COUNTS:
        o = (ctypes.c_int * 5)()
        lib.work(n, V, d, o)
        mt, pt, unit, nb, k = o
        assert (mt - 1) * pt < n <= mt * pt and pt <= 256 and mt == (n + 255) // 256
        assert unit * (nb - 1) < V <= unit * nb and 1 <= k <= min(nb, 256)
        first = (ctypes.c_int * (k + 1))()
        lib.ranges(n, V, d, first)
        assert first[0] == 0 and first[k] == nb
        assert all(a < b for a, b in zip(first, list(first)[1:]))
        times = (ctypes.c_int * (mt * k))()
        most = lib.segments(n, V, d, times)
        assert set(times) == {1}
        # no workgroup has more segments than an even share rounded up
        assert most == -(-mt * k // 256)
        assert n * k <= lib.max_partials(n, V)


def test_partials_reserved_for_any_number_of_candidates(lib):
    for N, V, d in [(64, 126464, 4096), (300, 5000, 64), (4096, 126464, 64), (40000, 700, 4096)]:
        room = lib.max_partials(N, V)
        for n in list(range(1, min(N, 1200))) + list(range(1200, N + 1, 37)) + [N]:
            o = (ctypes.c_int * 5)()
            lib.work(n, V, d, o)
            assert n * o[4] <= room, (n, V, d)
