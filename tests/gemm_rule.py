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
                    'extern "C" void pick(int M, int N, int nk, int act, int resid, int* out) {\n'
                    '  const llmc::GemmPick p = llmc::gemm_pick(M, N, nk, act != 0, resid != 0);\n'
                    '  out[0] = p.path; out[1] = p.tiles;\n}\n')
        subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                        src, "-o", so], check=True)
        return ctypes.CDLL(so)
    finally:
        shutil.rmtree(d)


def pick(M, N, K, epilogue="plain"):
    """(number of the tiling, tiles) that a launch of M rows and N columns contracted over K takes; the epilogue is "plain",
    "act" or "residual"."""
    out = (ctypes.c_int * 2)()
    _lib().pick(M, N, K // 64, int(epilogue == "act"), int(epilogue == "residual"), out)
    return out[0], out[1]


def block(d, dff, rows):
    """The tilings of a block's four linear layers (QKV, output projection, both feed-forward layers)."""
    return [TILINGS[pick(rows, n, k, e)[0]] for n, k, e in layers(d, dff)]


def layers(d, dff):
    """Columns, contraction and epilogue of a block's four linear layers."""
    return [(3 * d, d, "plain"), (d, d, "residual"), (dff, d, "act"), (d, dff, "residual")]


# Blocks (width, feed-forward width, tokens of a sequence, sequences) with the tilings that their four linear layers take: QKV,
# output projection (residual), feed-forward with its activation, feed-forward back (residual).
FEW_ROWS = [
    (64, 64, 1, 1, "32x64 32x64 32x64 32x64"),          # one token, one step of k, one column tile
    (64, 320, 31, 1, "32x64 32x64 32x64 32x64"),        # one row short of a tile; five steps of k in the last layer
    (192, 384, 33, 3, "32x64 32x64 32x64 32x64"),       # three steps (fewer than the ring's six stages) and six (as many)
    (448, 704, 65, 2, "32x64 32x64 32x64 32x64"),       # seven and eleven steps, columns that are odd multiples of 64
    (576, 1152, 50, 10, "64x64 32x64 64x64 32x64"),     # 500 rows: 52 in the last row of 64-row tiles
    (768, 3072, 96, 12, "64x128 64x64 64x128 64x64"),   # 1152 rows
]
MANY_ROWS = [
    # two steps of k, as many as the ring starts with, 320 columns in tiles of 128; 17,030 rows, six in the last row of tiles
    (128, 320, 131, 130, "128x128 64x64 128x128 64x128"),
    (128, 512, 131, 306, "128x128 64x64 128x128 64x128"),        # two steps, and second and third tiles of a workgroup
    (448, 704, 97, 90, "128x192 64x64 128x128 64x64"),           # 1344 columns in tiles of 192, 704 in tiles of 128
    (576, 1152, 67, 61, "128x128 64x128 64x128 64x128"),         # 4087 rows
    (576, 1152, 131, 229, "128x192 128x192 128x192 128x192"),    # 47 rows in the last row of tiles, second tiles with a residual
    (640, 1216, 131, 130, "128x128 128x128 128x192 128x128"),    # the same for 128 x 128; 1216 columns in tiles of 192
    (1024, 4096, 128, 33, "128x128 64x128 128x192 128x192"),     # columns that divide by eight tiles
]
