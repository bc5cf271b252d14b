"""The library's rules on sizes (csrc/gemm_choose.h), compiled for the host, so that a test can say which kernel its sizes reach."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1711_09846_amd", "csrc")
TILE_256, TILE_128, TILE_128x64, TILE_64 = range(4)
_SOURCE = r"""
#include "gemm_choose.h"
extern "C" int tile(int M, int N, int K, int batch, int heavy, int square, long long pitch, int upper) {
  return pbt::gl_choose(M, N, K, batch, heavy, square, pitch, upper);
}
extern "C" int in_parts(int P, int rows, int K, int N) { return pbt::wgrad_in_parts(P, rows, K, N); }
"""


@functools.lru_cache(None)
def _lib():
    d = tempfile.mkdtemp()
    src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
    with open(src, "w") as f:
        f.write(_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.tile.argtypes = [ctypes.c_int] * 6 + [ctypes.c_longlong, ctypes.c_int]
    return lib


def tile(M, N, K, batch, heavy=False, square=False, upper=False):
    """Tile shape of a product whose rows are as long as its sizes say.  heavy: an epilogue with an exponential, a Philox block or another array per
    element; square / upper: RBF sums, of a symmetric product."""
    return _lib().tile(M, N, K, batch, heavy, square, max(N, K), upper)


def weight_gradient_in_parts(P, rows, K, N):
    return bool(_lib().in_parts(P, rows, K, N))
