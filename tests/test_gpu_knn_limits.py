"""The exhaustive search on the matrix cores at the ends of what it takes: rows so long that uint8 distances leave its
integer range, floats so small that squares are subnormal, rows that no threshold can decide on, sets far from the
origin.  Every result is compared with the tiled kernel's, which rows on 4-byte boundaries take."""
import numpy as np
import pytest
import torch

from test_gpu_knn import check, off4

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
    kernel = "knn_tile_kernel" if d <= 16_384 else "bruteforce_tile_kernel"
    ids, dist = check(jx, b, q, 10, kernel)
    assert ids[0].tolist() == list(range(10)) and ids[1].tolist() == list(range(9_000, 9_010))
    assert not dist[:2].any()
    _, dist = check(jx, b[:9_000].repeat(2, 1), q, 10, kernel)  # no base vector near; 100 and 9,100 a little nearer
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
    """Up to 30 rows that no threshold can decide on are evaluated for every query; beyond that the tiled kernel runs."""
    g = torch.Generator(device="cuda").manual_seed(2)
    b, q = (torch.randn((n, 64), device="cuda", generator=g).to(dtype) for n in (20_000, 250))
    at = torch.randperm(20_000, device="cuda", generator=g)[:rows]
    for value in (float("nan"), -float("nan"), float("inf"), -float("inf")):
        x = b.clone()
        x[at, 5] = value
        for k in (8, 30, 50, 128):
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
    for k in (8, 10, 60):
        check(jx, b.to(dtype), q.to(dtype), k)


@pytest.mark.parametrize("d", [4, 8, 12, 16, 20])
@pytest.mark.parametrize("offset", [0, 10, 40])
def test_few_dimensions(jx, d, offset):
    """Up to 16 dimensions values are taken whole: what two parts could not prove far from the origin is proven there."""
    g = torch.Generator(device="cuda").manual_seed(14)
    b, q = (torch.randn((n, d), device="cuda", generator=g) + offset for n in (40_000, 300))
    b[7_000, 1], b[8_000, 2] = float("nan"), float("inf")
    for k in (8, 10, 60):
        check(jx, b, q, k)
    check(jx, b, q[:7], 1)


def rows(dtype, n, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n, d), device="cuda", generator=g)
    return (x * 40 + 128).clamp_(0, 255).to(torch.uint8) if dtype == torch.uint8 else x.to(dtype)


@pytest.mark.parametrize("dtype,nq,k", [(torch.uint8, 65_536, 10), (torch.float32, 40_000, 4), (torch.float16, 40_000, 4)])
def test_one_slice(jx, dtype, nq, k):
    """So many queries that one workgroup takes the whole base set for its own: no distances are published."""
    check(jx, rows(dtype, 16_500, 16, 4), rows(dtype, nq, 16, 5), k)
    jx.bruteforce_static(rows(dtype, 16_500, 16, 4), rows(dtype, nq, 16, 5), k)
    assert " nsplit=1 " in jx.bruteforce_kernel() and jx.bruteforce_kernel().endswith(" seed_steps=0"), jx.bruteforce_kernel()


def index(jx, x, max_batch=1024):
    kind = {torch.uint8: jx.U8, torch.float32: jx.F32, torch.float16: jx.F16}[x.dtype]
    g = jx.Index(x.shape[1], kind, 8, 8, 1.2, capacity=x.shape[0], max_batch=max_batch)
    g.import_graph(x, torch.full((x.shape[0], 8), -1, dtype=torch.int32, device="cuda"), 0)
    return g


def check_samples(jx, x, q, k, ids, dist, at):
    for i in at:
        i0, d0 = jx.bruteforce_static(off4(x), off4(q[i:i + 128]), k)
        assert torch.equal(ids[i:i + 128], i0)
        assert torch.equal(dist[i:i + 128].view(torch.int32), d0.view(torch.int32))


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float32, torch.float16])
def test_lists_too_long_for_a_first_threshold(jx, dtype):
    """More than 32 entries of every slice count: thresholds begin at infinity and are published as lists fill."""
    x, q = rows(dtype, 16_500, 16, 6), rows(dtype, 16_384, 16, 7)
    if dtype != torch.uint8:
        x[[3, 11_000], 4] = float("nan")
    ids, dist = index(jx, x).bruteforce(q, 128)
    name = jx.bruteforce_kernel()
    assert name.startswith("knn_tile_kernel<") and " nsplit=1 " not in name and name.endswith(" seed_steps=0"), name
    check_samples(jx, x, q, 128, ids, dist, (0, 7_000, 16_256))


def test_batches_that_the_tiled_kernel_keeps(jx):
    """Few vectors: one split for all queries, in slices that fit the workspace (83,840 queries of 100 neighbours)."""
    x, q = rows(torch.uint8, 2_000, 32, 8), rows(torch.uint8, 150_000, 32, 9)
    ids, dist = index(jx, x).bruteforce(q, 100)
    assert jx.bruteforce_kernel() == "bruteforce_tile_kernel<0> nsplit=1"
    check_samples(jx, x, q, 100, ids, dist, (0, 83_776, 83_840, 149_872))


@pytest.mark.parametrize("dtype,d,nq,k,fewest", [
    (torch.uint8, 64, 1, 3, 25_000), (torch.uint8, 64, 300, 1, 130_000), (torch.uint8, 64, 700, 1, 85_715), (torch.float32, 16, 1, 1, 81_250),
    (torch.float32, 16, 4, 2, 40_625), (torch.float16, 64, 2, 1, 31_250), (torch.float32, 16, 40, 1, 137_500), (torch.float16, 64, 64, 1, 125_000),
    (torch.float32, 32, 400, 3, 162_500), (torch.float32, 16, 1_000, 5, 262_500), (torch.float32, 36, 200, 1, 100_000), (torch.float32, 16, 2_000, 3, 62_500),
    (torch.float16, 32, 400, 2, 328_125), (torch.float16, 16, 601, 4, 99_834), (torch.float32, 16, 33, 2, 16_384)])
def test_few_neighbours_of_short_vectors(jx, dtype, d, nq, k, fewest):
    """The tiled kernel keeps what it does faster: on both sides of the number of vectors from which it does not."""
    x, q = rows(dtype, fewest, d, 10), rows(dtype, nq, d, 11)
    check(jx, x, q, k)
    jx.bruteforce_static(x[:fewest - 1], q, k)
    assert jx.bruteforce_kernel().startswith("bruteforce_tile_kernel<")


@pytest.mark.parametrize("d,k", [(4, 1), (8, 1), (16, 1), (16, 10), (32, 1), (48, 1), (64, 1)])
def test_significands_that_two_parts_hold_worst(jx, d, k):
    """Coordinates of 1.0039139 (0x3F808040): both roundings to bfloat16 leave the most they can, and the norm form of a duplicate of
    such a query is 2^-14 |q|^2 too far.  Vectors that differ from it in two coordinates, which hold on their own, come before it in
    that form, more of them than the lists keep; the duplicates have to be found all the same."""
    worst = float(np.array([0x3F808040], np.uint32).view(np.float32)[0])
    g = torch.Generator(device="cuda").manual_seed(12)
    b = torch.randn((20_000, d), device="cuda", generator=g) * 3
    q = torch.full((8, d), worst, device="cuda")
    near = torch.randperm(20_000, device="cuda", generator=g)[:120]
    b[near] = worst
    i = torch.arange(120, device="cuda")
    b[near[:100], (i % d)[:100]] = 1.0078125
    b[near[:100], ((i + 1 + i // d) % d)[:100]] = 1.0
    ids, dist = check(jx, b, q, k)
    assert not dist.any()
    assert ids[0].tolist() == sorted(near[100:].tolist())[:k]


def test_one_matrix_instruction(jx):
    """What knn_bound.h takes for granted of v_mfma_f32_32x32x16_bf16: off by at most 8 2^-24 of its largest term (of 16 products
    and the sum before them), subnormal values kept.  The rotation of bfloat16 values by a matrix of bfloat16 values that is zero
    outside sixteen columns is one such instruction; its sum before them is zero, or, with a second half, of the same order."""
    d, n, f = 32, 512, np.float64
    rng = np.random.default_rng(13)

    def bf16(x):
        return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).float()

    index_ = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=64, max_batch=1024, quant_bits=1)
    index_.import_graph(torch.ones((64, d), device="cuda"), torch.full((64, 8), -1, dtype=torch.int32, device="cuda"), 0)
    for spread, scale in ((0, 1.0), (4, 1.0), (12, 1.0), (30, 1.0), (4, 1e-37), (2, 1e-39)):
        for columns in (16, 32):
            x = bf16(rng.standard_normal((n, d)) * 2.0 ** rng.uniform(-spread, 0, (n, d)) * scale)
            p = bf16(rng.standard_normal((d, d)) * 2.0 ** rng.uniform(-spread, 0, (d, d)))
            x[:, columns:] = 0
            x[::7, 1] = -x[::7, 0]  # cancellation of the two largest
            p[::5, 1] = p[::5, 0]
            index_.quantize(1, p.cuda(), torch.zeros(d, device="cuda"), query_bits=4)
            got = index_.rotate(x.cuda()).cpu().numpy().astype(f)
            products = x.numpy().astype(f)[:, None, :] * p.numpy().astype(f)[None, :, :]
            first, both = products[:, :, :16], products[:, :, :columns]
            bound = 8 * 2.0 ** -24 * np.abs(first).max(2)
            if columns == 32:
                bound += 8 * 2.0 ** -24 * np.maximum(np.abs(first.sum(2)) + bound, np.abs(products[:, :, 16:]).max(2))
            off = np.abs(got - both.sum(2))
            assert (off <= bound + 2.0 ** -149).all()
