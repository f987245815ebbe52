"""The exhaustive search on the matrix cores (rows on 16-byte boundaries) against the tiled kernel that rows on 4-byte
boundaries take: ids and distances are equal to the last bit, ties, infinities and NaN included."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import dev, random_data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


def off4(t):
    """The same rows, four bytes behind a 16-byte boundary."""
    k = 4 // t.element_size()
    flat = torch.empty(t.numel() + k, dtype=t.dtype, device=t.device)
    flat[k:] = t.reshape(-1)
    out = flat[k:].view(t.shape)
    assert out.data_ptr() % 16 == 4
    return out


def check(jx, b, q, k, kernel="knn_tile_kernel"):
    ids, dist = jx.bruteforce_static(b, q, k)
    assert jx.bruteforce_kernel().startswith(kernel + "<"), jx.bruteforce_kernel()
    ids0, dist0 = jx.bruteforce_static(off4(b), off4(q), k)
    assert jx.bruteforce_kernel().startswith("bruteforce_tile_kernel<")
    assert torch.equal(ids, ids0)
    assert torch.equal(dist.view(torch.int32), dist0.view(torch.int32))
    return ids, dist


@pytest.mark.parametrize("dtype,n,d,nq,k", [
    ("uint8", 40_000, 128, 300, 10), ("uint8", 133_333, 16, 129, 1), ("uint8", 20_001, 144, 127, 100), ("uint8", 20_000, 6144, 65, 128),
    ("uint8", 300_000, 128, 1, 10), ("uint8", 100_000, 256, 2_000, 10),
    ("float32", 40_000, 128, 300, 10), ("float32", 130_001, 4, 257, 3), ("float32", 130_001, 4, 257, 9), ("float32", 20_000, 36, 128, 128), ("float32", 20_003, 960, 200, 100),
    ("float32", 100_000, 96, 3, 1),
    ("float16", 40_000, 128, 300, 10), ("float16", 30_001, 8, 129, 37), ("float16", 20_003, 960, 200, 100)])
def test_equals_the_tiled_kernel(jx, dtype, n, d, nq, k):
    t = np.uint8 if dtype == "uint8" else np.float32
    b, q = random_data(n, d, t, 21).astype(dtype), random_data(nq, d, t, 22).astype(dtype)
    few = dtype == "float32" and d == 4 and k == 3  # too few coordinates for three neighbours
    ids, dist = check(jx, dev(b), dev(q), k, "bruteforce_tile_kernel" if few else "knn_tile_kernel")
    if dtype == "uint8" and d <= 256:
        some = np.unique(np.linspace(0, nq - 1, 12).astype(int))
        want = oracle.bruteforce(b, q[some], k)
        assert np.array_equal(ids.cpu().numpy().view(np.uint32)[some], want[0])


@pytest.mark.parametrize("dtype", ["uint8", "float32", "float16"])
def test_ties_and_slices(jx, dtype):
    """Many equal distances: every slice is full of them, and the smallest ids win."""
    rng = np.random.default_rng(3)
    b = rng.integers(0, 3, (40_000, 32)).astype(dtype)
    b[5_000:30_000] = b[17]
    q = rng.integers(0, 3, (200, 32)).astype(dtype)
    q[:100] = b[17]
    check(jx, dev(b), dev(q), 10)
    check(jx, dev(b), dev(q), 80)


@pytest.mark.parametrize("dtype", ["float32", "float16"])
def test_infinities_and_nan(jx, dtype):
    x = random_data(20_000, 64, np.float32, 5).astype(dtype)
    q = random_data(300, 64, np.float32, 6).astype(dtype)
    for value in (np.inf, -np.inf, np.nan, np.finfo(dtype).max):
        y, p = x.copy(), q.copy()
        y[7_777, 3] = value
        p[5, 60] = value
        check(jx, dev(y), dev(q), 10)
        check(jx, dev(x), dev(p), 10)
        check(jx, dev(y), dev(p), 10)
    far = (x.astype(np.float32) + 1000).astype(dtype)  # distances small against the norms: nothing can be proven
    check(jx, dev(far), dev((q.astype(np.float32) + 1000).astype(dtype)), 10)


def test_index_search_slices_queries(jx):
    """jx_bruteforce of an index takes the same path; more queries than its workspace holds lists for go in slices."""
    b, q = random_data(10_000, 32, np.uint8, 8), random_data(150_000, 32, np.uint8, 9)
    g = jx.Index(32, jx.U8, 8, 8, 1.2, capacity=10_000, max_batch=1024)
    g.import_graph(dev(b), torch.full((10_000, 8), -1, dtype=torch.int32, device="cuda"), 0)
    ids, dist = g.bruteforce(dev(q), 64)
    assert jx.bruteforce_kernel().startswith("knn_tile_kernel<")
    for at in (0, 75_000, 149_872):
        i0, d0 = jx.bruteforce_static(dev(b), dev(q[at:at + 128]), 64)
        assert torch.equal(ids[at:at + 128], i0) and torch.equal(dist[at:at + 128], d0)


@pytest.mark.parametrize("dtype", ["uint8", "float32", "float16"])
@pytest.mark.parametrize("d,n,nq,k", [(128, 40_000, 130, 10), (96, 30_000, 300, 100), (112, 60_001, 64, 8)])
def test_vectors_that_come_nearer_and_nearer(jx, dtype, d, n, nq, k):
    """Sorted from far to near: whatever the first limits are, every vector of a step passes, each buffer overflows many times
    over, and what it had no room for is offered again until it fits."""
    t = np.uint8 if dtype == "uint8" else np.float32
    b, q = random_data(n, d, t, 31).astype(np.float64), random_data(nq, d, t, 32)
    q[:] = q[0]
    q[1::2, 0] += 1
    b = b[np.argsort(-((b - q[0]) ** 2).sum(1))].astype(dtype)
    check(jx, dev(b), dev(q.astype(dtype)), k)
