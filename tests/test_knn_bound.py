"""The rounding rules of the float form of the exhaustive search (knn_bound.h), compiled for the CPU: what its first
thresholds count is admitted, and the two forms of a distance are no further apart than its bound says.  Counting of base
vectors and scratch as well."""
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
extern "C" void bounds_parts(int d, const float* qq, const float* e, const float* bb_max, float* out, long n) {
    for (long i = 0; i < n; i++) out[i] = jx::knn_eps(d, qq[i], e[i], bb_max[i], jx::knn_parts(d));
}
extern "C" void bounds(int d, const float* qq, const float* e, const float* bb_max, float* out, long n) {
    for (long i = 0; i < n; i++) out[i] = jx::knn_eps(d, qq[i], e[i], bb_max[i]);
}
extern "C" long long fits(long long bytes, long long nq, int kp) { return jx::knn_slices_that_fit(bytes, nq, kp); }
extern "C" int published_bytes() { return KNN_PUB * 4; }
// the loop of knn_u8_kernel over a slice: steps, rows that are staged as if they were of the set, the row that is fetched last
extern "C" void walk(long long n, int nsplit, int split, long long out[4]) {
    jx::knn_row begin, end;
    jx::knn_slice(n, nsplit, split, &begin, &end);
    long long steps = 0, outside = 0, last = -1;
    for (jx::knn_row b0 = begin;; b0 += KT) {
        if (b0 >= end || steps > (1LL << 31) / KT) break;  // the second: it does not end by itself
        steps++;
        if (jx::knn_whole_step(b0, end)) outside += (long long)b0 + KT > n;
        if (!jx::knn_last_step(b0, end)) last = (long long)b0 + KT;
    }
    out[0] = (long long)end - (long long)begin;
    out[1] = steps;
    out[2] = outside;
    out[3] = last;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("knn_bound")
    (d / "b.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-fwrapv", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(d / "b.cpp"), "-o", str(d / "b.so")], check=True)
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


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("d", [4, 128, 1536])
@pytest.mark.parametrize("offset", [0.0, 3.0, 1000.0])
@pytest.mark.parametrize("scale", [3e-23, 1e-19, 1.0, 1e15])
def test_bound_covers_both_forms(lib, d, offset, scale):
    """|norm form - form of the result| <= knn_eps, for a longest vector of known and of unknown length.  Where
    norms overflow the bound is not finite, and nothing is proven."""
    rng = np.random.default_rng(8)
    n, f = 2_000, np.float32
    q = ((rng.standard_normal((n, d)) + offset) * scale).astype(f)
    b = (q + rng.standard_normal((n, d)) * scale * 10.0 ** rng.uniform(-3, 1, (n, 1))).astype(f)
    qq, bb, x, e = (np.zeros(n, f) for _ in range(4))
    for j in range(d):
        qq = (qq + q[:, j].astype(np.float64) * q[:, j]).astype(f)
        bb = (bb + b[:, j].astype(np.float64) * b[:, j]).astype(f)
        x = (x + q[:, j].astype(np.float64) * b[:, j]).astype(f)
        t = (q[:, j] - b[:, j]).astype(np.float64)
        e = (e + t * t).astype(f)
    apart = np.abs((qq + bb - f(2) * x).astype(np.float64) - e)
    for longest in (np.inf, max(1e38, bb.max()), bb.max()):
        eps = np.empty(n, f)
        lib.bounds(C.c_int(d), _ptr(qq), _ptr(e), _ptr(np.full(n, longest, f)), _ptr(eps), C.c_long(n))
        assert (~(eps < np.inf) | (apart <= eps)).all()


def test_one_long_vector_does_not_widen_the_bound(lib):
    qq, e = np.array([1.0], np.float32), np.array([0.5], np.float32)
    out = []
    for longest in (2.0, 1e6, 3e38, np.inf):
        eps = np.empty(1, np.float32)
        lib.bounds(C.c_int(960), _ptr(qq), _ptr(e), _ptr(np.array([longest], np.float32)), _ptr(eps), C.c_long(1))
        out.append(eps[0])
    assert out[0] < out[1] == out[2] == out[3] < 1.5 * out[0]
    for bad in (np.nan, np.inf):  # a query that cannot be proven
        eps = np.empty(1, np.float32)
        lib.bounds(C.c_int(960), _ptr(np.array([bad], np.float32)), _ptr(e), _ptr(np.array([2.0], np.float32)), _ptr(eps), C.c_long(1))
        assert not eps[0] < np.inf


def _bf16(x):
    """Rounded to bfloat16, to nearest even."""
    u = x.view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def _parts(x):
    """Three bfloat16 parts of float32 values, in 64 bits."""
    h = _bf16(x)
    l = _bf16(x - h)
    return h.astype(np.float64), l.astype(np.float64), (x - h - l).astype(np.float64)


def _products(q, b):
    """What the matrix cores add of each coordinate, smallest first: of two parts, and of three up to 16 dimensions."""
    (h, l, r), (hb, lb, rb) = _parts(q), _parts(b)
    three = [l * hb, h * lb, h * hb]
    return [r * hb, h * rb, l * lb, *three] if q.shape[-1] <= 16 else three


def _sums(products, sign):
    """Sums of rows as matrix instructions take them: 16 products and the sum before them, each time off by 8 2^-24 of the largest
    of these, towards the given side."""
    d, total = products[0].shape[1], np.zeros(products[0].shape[0])
    for j in range(0, d, 16):
        for p in products:
            group = p[:, j:j + 16]
            total = total + group.sum(1) + sign * 8 * 2.0 ** -24 * np.maximum(np.abs(total), np.abs(group).max(1))
    return total


@pytest.mark.parametrize("d", [4, 16, 32, 128, 1536])
@pytest.mark.parametrize("offset", [0.0, 3.0, 1000.0])
@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("scale", [1e-19, 1.0, 1e15])
def test_bound_covers_the_parts(lib, d, offset, scale):
    """The norm form on bfloat16 parts of each value, what the parts lack alone (products summed in 64 bits) and with every
    matrix instruction off by the most there is, to either side."""
    rng = np.random.default_rng(9)
    n, f = 2_000, np.float32
    q = ((rng.standard_normal((n, d)) + offset) * scale).astype(f)
    b = (q + rng.standard_normal((n, d)) * scale * 10.0 ** rng.uniform(-3, 1, (n, 1))).astype(f)
    products = _products(q, b)
    qq, bb = (q.astype(np.float64) ** 2).sum(1), (b.astype(np.float64) ** 2).sum(1)
    e = ((q.astype(np.float64) - b) ** 2).sum(1)
    eps = np.empty(n, f)
    lib.bounds_parts(C.c_int(d), _ptr(qq.astype(f)), _ptr(e.astype(f)), _ptr(np.full(n, np.inf, f)), _ptr(eps), C.c_long(n))
    assert scale > 1 or np.isfinite(eps).all()
    for sign in (-1, 0, 1):  # as above: no proof where norms of that length could overflow
        assert (~(eps < np.inf) | (np.abs(qq + bb - 2 * _sums(products, sign) - e) <= eps)).all()


def test_what_parts_leave_of_any_value():
    """All significands: roundings to 8 bits leave up to 2^-8 and 2^-17 of a value, a third part leaves nothing, and the three products
    of two parts that are taken of a value's own square lack up to 2^-15 of it, the six of three parts up to 2^-24."""
    x = (np.arange(1 << 23, dtype=np.uint32) | 0x3F800000).view(np.float32)
    h, l, r = _parts(x)
    assert (np.abs(l) <= 2.0 ** -8 * x).all() and np.abs(l / x).max() > 0.99 * 2.0 ** -8
    assert (np.abs(r) <= 2.0 ** -17 * x).all() and np.abs(r / x).max() > 0.99 * 2.0 ** -17
    assert np.array_equal(_bf16(r.astype(np.float32)), r) and np.array_equal(h + l + r, x)
    lacks = (l * l + 2 * h * r) / x.astype(np.float64) ** 2
    assert 0.98 * 2.0 ** -15 < np.abs(lacks).max() <= 2.0 ** -15 * (1 + 2.0 ** -9)
    lacks = (r * r + 2 * l * r) / x.astype(np.float64) ** 2
    assert 0.98 * 2.0 ** -24 < np.abs(lacks).max() <= 2.0 ** -24 * (1 + 2.0 ** -10)


# the significand whose parts lack most (the search above finds it): 1.0039139
WORST = np.array([0x3F808040], np.uint32).view(np.float32)[0]


@pytest.mark.parametrize("d", [4, 8, 16, 20, 32, 48, 52, 64, 128, 960])
@pytest.mark.parametrize("scale", [2.0 ** -40, 1.0, 2.0 ** 40])
def test_bound_covers_the_worst_significands(lib, d, scale):
    """A duplicate of a query whose every coordinate lacks the most there is: nothing cancels.  With every rounding of the norm
    form against it as well: matrix instructions as above, and the sums behind by half a unit in the last place each."""
    u = 2.0 ** -24
    x = np.full((1, d), WORST * np.float32(scale), np.float32)
    total = _sums(_products(x, x), -1)[0]
    norm = (x.astype(np.float64) ** 2).sum()
    longest_chain = 4 * ((d + 31) // 32) + 3  # squares of a norm that one thread adds, and the eight threads of a row
    apart = 2 * norm * (1 + longest_chain * u) * (1 + u) - 2 * total + 2 * u * norm
    eps = np.empty(1, np.float32)
    for e in (0.0, norm * 1e-3):
        lib.bounds_parts(C.c_int(d), _ptr(np.array([norm], np.float32)), _ptr(np.array([e], np.float32)), _ptr(np.array([norm], np.float32)),
                         _ptr(eps), C.c_long(1))
        assert apart <= eps[0], (apart, eps[0])


@pytest.mark.parametrize("n", [6_000, 16_383, 1_000_000, 2 ** 31 - 257, 2 ** 31 - 129, 2 ** 31 - 128, 2 ** 31 - 127, 2 ** 31 - 100, 2 ** 31 - 2])
@pytest.mark.parametrize("nsplit", [1, 2, 5])
def test_steps_of_a_slice_end_with_the_set(lib, n, nsplit):
    """Up to the largest set there can be: a step is whole only where the set has all its rows, nothing is fetched beyond it, and
    the steps end."""
    total, out = 0, (C.c_longlong * 4)()
    for split in range(nsplit):
        lib.walk(C.c_longlong(n), C.c_int(nsplit), C.c_int(split), out)
        total += out[0]
        assert out[1] == -(-out[0] // 128) and out[2] == 0 and out[3] < n
    assert total == n


@pytest.mark.parametrize("kp", [1, 2, 3, 4, 10, 29, 128, 156])
def test_lists_and_published_distances_fit_the_scratch(lib, kp):
    """At every size around which a slice more or less fits, one-slice scratch (which publishes nothing) included."""
    lib.fits.restype = C.c_longlong
    for nq in (1, 7, 128, 16_384, 100_000):
        for slices in (0, 1, 2, 3, 4, 5, 64):
            for publish in (0, 1):
                for off in (-1, 0, 1):
                    size = nq * slices * (kp * 8 + publish * lib.published_bytes()) + off
                    n = lib.fits(C.c_longlong(size), C.c_longlong(nq), C.c_int(kp))
                    assert n >= (1 if size >= nq * kp * 8 else 0)
                    assert n == 0 or nq * n * (kp * 8 + (lib.published_bytes() if n > 1 else 0)) <= size
