"""Where the streaming bf16 forward reads W as fp32: every 16-byte load of every lane lies inside the matrix, also in slices
that are wider than the row, and columns inside the row are read from their own place.  The kernel's index functions,
compiled for the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fwd_w_column(tmp_path_factory):
    d = tmp_path_factory.mktemp("forward_index")
    src, so = str(d / "probe.cpp"), str(d / "probe.so")
    with open(src, "w") as f:
        f.write('#include "forward_index.h"\n'
                'extern "C" int64_t column(int64_t k0, int part, int64_t D) { return sfb::fwd_w_column(k0, part, D); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1409_5705_amd", "csrc"),
                    "-o", so, src], check=True)
    fn = ctypes.CDLL(so).column
    fn.restype, fn.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    return fn


@pytest.mark.parametrize("D", list(range(8, 200, 8)) + [1000, 4096, 10000])
def test_loads_of_fp32_rows_stay_inside_the_matrix(fwd_w_column, D):
    for k0 in range(0, D, 64):
        for part in range(16):
            c = fwd_w_column(k0, part, D)
            assert c >= 0 and c % 4 == 0
            if k0 + 4 * part < D:
                assert c == k0 + 4 * part
            for J in (1, 8, 40, 16384):          # four floats from column c of the last row (rows past it are clamped to it)
                assert (J - 1) * D + c + 4 <= J * D, (D, k0, part)
