"""The rounding rules of the float form of the exhaustive search (knn_bound.h), compiled for the CPU: what its first
thresholds count is admitted."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_07048_amd", "csrc")
SOURCE = """
#include <math.h>
#include "knn_bound.h"
extern "C" void thresholds(const float* lim, const float* qq, float* out, long n) {
    for (long i = 0; i < n; i++) out[i] = jx::knn_threshold(lim[i], qq[i]);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("knn_bound")
    (d / "b.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(d / "b.cpp"), "-o", str(d / "b.so")], check=True)
    return C.CDLL(str(d / "b.so"))


def _ptr(a):
    return a.ctypes.data_as(C.c_void_p)


@pytest.mark.parametrize("offset", [0.0, 1.0, 30.0, 1000.0])
@pytest.mark.parametrize("scale", [1e-20, 1.0, 1e15])
def test_counted_vectors_are_admitted(lib, offset, scale):
    """The vector that a first threshold just counts is let in behind that threshold: sums as the kernel takes them."""
    rng = np.random.default_rng(7)
    n, d, f = 200_000, 8, np.float32
    q = ((rng.standard_normal((n, d)) + offset) * scale).astype(f)
    b = (q + rng.standard_normal((n, d)) * scale * 10.0 ** rng.uniform(-4, 0.5, (n, 1))).astype(f)
    qq, bb, x = (np.zeros(n, f) for _ in range(3))
    for j in range(d):  # float32 products are exact in float64: one rounding per step, as a fused multiply-add
        qq = (qq + q[:, j].astype(np.float64) * q[:, j]).astype(f)
        bb = (bb + b[:, j].astype(np.float64) * b[:, j]).astype(f)
        x = (x + q[:, j].astype(np.float64) * b[:, j]).astype(f)
    code = np.maximum(qq - (f(2) * x - bb), f(0))
    lim = np.nextafter(code, f(np.inf))
    t = np.empty(n, f)
    lib.thresholds(_ptr(lim), _ptr(qq), _ptr(t), C.c_long(n))
    assert ((2.0 * x.astype(np.float64) + t).astype(f) > bb).all()
