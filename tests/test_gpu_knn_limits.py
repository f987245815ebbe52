"""The exhaustive search on the matrix cores at the ends of what it takes: rows so long that uint8 distances leave its
integer range, floats so small that squares are subnormal, rows that no threshold can judge, sets far from the
origin.  Every result is compared with the tiled kernel's, which rows on 4-byte boundaries take."""
import pytest
import torch

from test_gpu_knn import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


@pytest.mark.parametrize("d", [16_384, 16_400, 20_640, 20_656, 43_696, 50_176])
def test_uint8_rows_of_any_length(jx, d):
    """Rows of nothing but 0 and nothing but 255 lie d x 255^2 apart: 2^30.3 at 20,656 dimensions, 2^31.6 at 50,176."""
    b = torch.zeros((16_400, d), dtype=torch.uint8, device="cuda")
    b[9_000:] = 255
    b[100, 0] = 3
    q = torch.zeros((4, d), dtype=torch.uint8, device="cuda")
    q[1:] = 255
    q[2, ::2] = 0
    ids, dist = check(jx, b, q, 10)
    assert ids[0].tolist() == list(range(10)) and ids[1].tolist() == list(range(9_000, 9_010))
    assert not dist[:2].any()
    _, dist = check(jx, b[:9_000].repeat(2, 1), q, 10)  # no base vector near; 100 and 9,100 a little nearer
    assert dist[1, 2:].eq(float(d * 255 ** 2)).all()


@pytest.mark.parametrize("scale", [1e-18, 1e-20, 1e-22, 7e-23, 5e-23, 2e-23])
def test_tiny_floats(jx, scale):
    """Where squares are subnormal an operation is off by up to half of 2^-149 however small its result."""
    g = torch.Generator(device="cuda").manual_seed(1)
    for _ in range(4):
        b, q = (torch.randn((n, 32), device="cuda", generator=g) * scale for n in (20_000, 400))
        check(jx, b, q, 10)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("rows", [1, 30, 31, 2_000])
def test_rows_with_nan_and_infinities(jx, dtype, rows):
    """Up to 30 rows that no threshold can judge are evaluated for every query; beyond that the tiled kernel runs."""
    g = torch.Generator(device="cuda").manual_seed(2)
    b, q = (torch.randn((n, 64), device="cuda", generator=g).to(dtype) for n in (20_000, 250))
    at = torch.randperm(20_000, device="cuda", generator=g)[:rows]
    for value in (float("nan"), -float("nan"), float("inf"), -float("inf")):
        x = b.clone()
        x[at, 5] = value
        for k in (1, 30, 50, 128):
            check(jx, x, q, k)
    x = b.clone()
    x[at[::2], 5], x[at[1::2], 6] = float("nan"), float("inf")
    y = q.clone()
    y[::50, 7] = float("nan")
    y[1::50, 7] = float("inf")
    check(jx, x, y, 10)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("far", ["all", "every other query", "one tile of queries", "the base set's end"])
def test_sets_far_from_the_origin(jx, dtype, far):
    """Distances small against the norms cannot be proven.  Tiles of such queries alone leave early; others hold some."""
    g = torch.Generator(device="cuda").manual_seed(3)
    b, q = (torch.randn((n, 64), device="cuda", generator=g) for n in (20_000, 400))
    if far == "all":
        b, q = b + 500, q + 500
    else:
        b[10_000:] += 500
    if far == "every other query":
        q[::2] += 500
    if far == "one tile of queries":
        q[128:256] += 500
    for k in (1, 10, 60):
        check(jx, b.to(dtype), q.to(dtype), k)
