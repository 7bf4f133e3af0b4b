"""Host check of the voxel passes' pixel index (csrc/pixel.hpp, compiled here
as plain C++): v W + u for every corner of the accepted image sizes and around
the 2^24 pixels up to which FP32 holds whole numbers."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def index(tmp_path_factory):
    d = tmp_path_factory.mktemp("pixel")
    src, so = d / "pixel.cpp", d / "libpixel.so"
    src.write_text('#include "pixel.hpp"\n'
                   'extern "C" void index_of(const float* u, const float* v, uint32_t w, uint32_t* out, long n)\n'
                   '{ for (long i = 0; i < n; ++i) out[i] = sc::pixel_index(u[i], v[i], w); }\n')
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC",
                           f"-I{os.path.join(ROOT, 'paper_1709_03763_amd', 'csrc')}", str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))

    def run(u, v, w):
        u, v = np.ascontiguousarray(u, np.float32), np.ascontiguousarray(v, np.float32)
        out = np.empty(u.size, np.uint32)
        lib.index_of(u.ctypes.data_as(ctypes.c_void_p), v.ctypes.data_as(ctypes.c_void_p), ctypes.c_uint32(w),
                     out.ctypes.data_as(ctypes.c_void_p), ctypes.c_long(u.size))
        return out

    return run


@pytest.mark.parametrize("W,H", [(1, 1), (640, 480), (4096, 4096), (4097, 4096), (5000, 4000), (16384, 1025),
                                 (1025, 16384), (16384, 16384)])
def test_pixel_index(index, W, H):
    rng = np.random.default_rng(W + H)
    u = np.concatenate([rng.integers(0, W, 4000), [0, W - 1, 0, W - 1, max(W - 2, 0)]])
    v = np.concatenate([rng.integers(0, H, 4000), [0, 0, H - 1, H - 1, H - 1]])
    near = np.arange((1 << 24) - 50, (1 << 24) + 50)  # pixels around 2^24
    near = near[near < W * H]
    u, v = np.concatenate([u, near % W]), np.concatenate([v, near // W])
    np.testing.assert_array_equal(index(u, v, W).astype(np.int64), v * W + u)
