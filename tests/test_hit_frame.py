"""The local frame of a hit in 64 bits: the azimuth's cosine and sine are the
correctly rounded quotients of the hit's coordinates and its radius.  The
device header is compiled for the host; a float32 coordinate's square is exact
in 64 bits, so numpy's quotients are the same in every bit."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_1906_02253_amd.build as B

SRC = r"""
#include "kf_math.hpp"
extern "C" void frames(const float* x, const float* y, long n, double* c, double* s)
{
    for (long i = 0; i < n; ++i) {
        const kfmi::HitFrame<double> f = kfmi::hit_frame<double>(x[i], y[i], 0.0f, 0.01f, 0.05f);
        c[i] = f.c;
        s[i] = f.s;
    }
}
"""


@pytest.fixture(scope="module")
def frames(tmp_path_factory):
    d = tmp_path_factory.mktemp("frame")
    src, so = os.path.join(d, "frame.cpp"), os.path.join(d, "frame.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", B.CSRC, "-o", so, src], check=True, capture_output=True)
    return ctypes.CDLL(so).frames


@pytest.mark.parametrize("scale", [1e-3, 4.0, 100.0])
def test_quotients_are_correctly_rounded(frames, scale):
    rng = np.random.default_rng(3)
    n = 200_000
    x, y = (rng.normal(0, scale, n).astype(np.float32) for _ in range(2))
    c, s = np.empty(n), np.empty(n)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    frames(p(x), p(y), ctypes.c_long(n), p(c), p(s))
    X, Y = x.astype(np.float64), y.astype(np.float64)
    rho = np.sqrt(X * X + Y * Y)
    assert np.array_equal(c, X / rho)
    assert np.array_equal(s, Y / rho)
