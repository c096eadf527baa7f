"""The eight-element loads of the product's activations stay inside X: the
rule the kernels go by, compiled for the host and checked on every piece of
small X."""

import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2602_08376_amd", "csrc")


@pytest.fixture(scope="module")
def inside(tmp_path_factory):
    d = tmp_path_factory.mktemp("x_piece")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text('#include "x_piece.h"\n'
                   'extern "C" int inside(int64_t r, int64_t t, int64_t m, int64_t T) {\n'
                   "  return ojbkq::x_piece_inside(r, t, m, T);\n}\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)],
                   check=True)
    f = ctypes.CDLL(str(lib)).inside
    f.argtypes = [ctypes.c_int64] * 4
    return f


@pytest.mark.parametrize("T", range(1, 20))
def test_pieces_end_inside_x(inside, T):
    for ld in range(T, T + 9):
        for m in range(1, 12):
            end = (m - 1) * ld + T   # one past X's last element
            for r in range(m):
                for t in range(0, T, 8):   # a loader's pieces start at multiples of 8
                    if inside(r, t, m, T):
                        assert r * ld + t + 8 <= end, (T, ld, m, r, t)
                    # a whole piece, and from eight tokens on every row but the
                    # last, is read at once
                    elif t + 8 <= T or (T >= 8 and r < m - 1):
                        raise AssertionError((T, ld, m, r, t))
