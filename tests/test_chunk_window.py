"""The staging bounds of a ragged tile (csrc/chunk_window.hpp), compiled for
the host, against unbounded integers: every staged row and column of first,
inner and last tiles reads the clamped image position, at extents up to the
2^31 - 1 that a batch item may have."""
import ctypes
import os
import subprocess

import pytest

from paper_2504_01266_amd import build

TILES = [(64, 64, 3), (32, 64, 9), (128, 64, 5), (32, 128, 7)]  # rows, columns, K
TOP = 2 ** 31 - 1
EXTENTS = [1, 2, 3, 4, 5, 63, 64, 65, 127, 129, TOP - 130, TOP - 64, TOP - 63, TOP - 4, TOP - 3, TOP - 1, TOP]


def pitch(tw, k):
    return (4 + tw + (k - 1) // 2 + 3) // 4 * 4


@pytest.fixture(scope="module")
def window(tmp_path_factory):
    d = tmp_path_factory.mktemp("window")
    cases = "".join(f"  if (pitch == {p}) w = f2d::chunk_window<{p}>(row0, col0, H, W);\n"
                    for p in {pitch(tw, k) for _, tw, k in TILES})
    src = d / "w.cpp"
    src.write_text('#include "chunk_window.hpp"\n'
                   'extern "C" void window(int pitch, int row0, int col0, int H, int W, int y, int x, int* out) {\n'
                   '  f2d::ChunkWindow w{};\n' + cases +
                   '  out[0] = w.row(y);\n  out[1] = w.four(x, &out[2]);\n  out[3] = w.inside;\n}\n')
    lib = d / "w.so"
    clang = os.path.join(os.path.dirname(build.HIPCC), "amdclang++")
    subprocess.run([clang, "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", build.CSRC, str(src), "-o",
                    str(lib)], check=True)
    so = ctypes.CDLL(str(lib))

    def call(*a):
        out = (ctypes.c_int32 * 4)()
        so.window(*a, out)
        return list(out)

    return call


def clamp(v, n):
    return min(max(v, 0), n - 1)


@pytest.mark.parametrize("th,tw,k", TILES)
def test_staged_rows_and_columns_are_the_clamped_ones(window, th, tw, k):
    r, lh, p = (k - 1) // 2, th + k - 1, pitch(tw, k)
    for n in EXTENTS:
        last = (n - 1) // th
        for t in {0, min(1, last), last // 2, max(last - 1, 0), last}:
            row0 = t * th - r
            for y in range(lh):
                assert window(p, row0, 0, n, 4, y, 0)[0] == clamp(row0 + y, n), (n, t, y)
        if n < 4:  # (rows of fewer columns are read by elements)
            continue
        last = (n - 1) // tw
        for t in {0, min(1, last), last // 2, max(last - 1, 0), last}:
            col0 = t * tw - 4
            for x in range(0, p, 4):
                _, first, shift, inside = window(p, 0, col0, 4, n, 0, x)
                assert bool(inside) == (col0 >= 0 and col0 + p <= n), (n, t)
                assert 0 <= first <= n - 4
                got = [first + min(max(shift + q, 0), 3) for q in range(4)]
                assert got == [clamp(col0 + x + q, n) for q in range(4)], (n, t, x)
