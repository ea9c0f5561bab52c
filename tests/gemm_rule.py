"""The tiling rule of the bf16 linear layers (csrc/gemm_rule.h, plain C++), compiled for the host and callable."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_16843_amd", "csrc")
TILINGS = ("128x192", "128x128", "64x128", "64x64", "32x64")


@functools.lru_cache(maxsize=None)
def _lib():
    d = tempfile.mkdtemp(prefix="gemm_rule_")
    try:
        src, so = os.path.join(d, "rule.cpp"), os.path.join(d, "rule.so")
        with open(src, "w") as f:
            f.write('#include "gemm_rule.h"\n'
                    'extern "C" void pick(int M, int N, int nk, int act, int* out) {\n'
                    '  const llmc::GemmPick p = llmc::gemm_pick(M, N, nk, act != 0);\n'
                    '  out[0] = p.path; out[1] = p.tiles;\n}\n')
        subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                        src, "-o", so], check=True)
        return ctypes.CDLL(so)
    finally:
        shutil.rmtree(d)


def pick(M, N, K, act=False):
    """(number of the tiling, tiles) that a launch of M rows, N columns and K steps of the contraction takes."""
    out = (ctypes.c_int * 2)()
    _lib().pick(M, N, K // 64, int(act), out)
    return out[0], out[1]


def block(d, dff, rows):
    """The tilings of a block's four linear layers (QKV, output projection, both feed-forward layers)."""
    return [TILINGS[pick(rows, n, k, act)[0]] for n, k, act in ((3 * d, d, False), (d, d, False), (dff, d, True), (d, dff, False))]
