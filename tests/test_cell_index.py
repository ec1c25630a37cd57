"""The byte offset of a bilinear cell's corner (csrc/cell_index.h, the gathers
of the demons kernels) in images of up to 16384 x 16384 px: compiled for the
host and compared with whole-number arithmetic.  CPU only."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_05993_amd", "csrc")


@pytest.fixture(scope="module")
def offsets(tmp_path_factory):
    d = tmp_path_factory.mktemp("cell")
    src, so = d / "cell.cpp", d / "cell.so"
    src.write_text('#include "cell_index.h"\n'
                   'extern "C" void offsets(const float* x, const float* y, int n, unsigned row_bytes, unsigned* o)\n'
                   '{ for (int i = 0; i < n; i++) o[i] = ebsd::cell_offset(x[i], y[i], row_bytes); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(so)], check=True)
    f = C.CDLL(str(so)).offsets

    def run(x, y, w):
        x, y = np.ascontiguousarray(x, np.float32), np.ascontiguousarray(y, np.float32)
        out = np.empty(x.size, np.uint32)
        f(x.ctypes.data_as(C.c_void_p), y.ctypes.data_as(C.c_void_p), C.c_int(x.size), C.c_uint(4 * w),
          out.ctypes.data_as(C.c_void_p))
        return out
    return run


@pytest.mark.parametrize("H,W", [(4, 4), (256, 256), (4096, 4096), (4097, 4097), (4099, 4099), (16384, 1025),
                                 (1025, 16384), (16383, 16383), (16384, 16384)])
def test_offsets_are_exact_and_inside_the_image(offsets, H, W):
    rng = np.random.default_rng(H * 3 + W)
    # corners of a cell lie in [0, W - 2] x [0, H - 2]
    x = np.concatenate([[0, W - 2, 0, W - 2, W - 3], rng.integers(0, W - 1, 20000)])
    y = np.concatenate([[0, 0, H - 2, H - 2, H - 2], rng.integers(0, H - 1, 20000)])
    o = offsets(x, y, W).astype(np.int64)
    assert np.array_equal(o, 4 * (y.astype(np.int64) * W + x))
    # the cell's two 8-byte loads end inside the image
    assert (o + 4 * W + 8).max() <= 4 * H * W
