"""robustPrune on the matrix cores.  As one Gram matrix per workgroup: candidate lists around the edges of its 32-row blocks and of its two
sizes (128, 256), with rows that end inside a 128-byte piece.  The data lie on a dyadic grid, where every partial sum is
exact in float32 (and in the three bfloat16 parts of a value), so the adjacency table is the oracle's, bit for bit.
In rounds of 32 pivots (uint8): the same edges, rows of one and of two 128-byte pieces, and hubs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_07048_amd import datagen
from gpu_common import dev, u32, jx_dtype, random_data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


# (d, R, L): the frontier is the candidate list, L entries long; rows of R plus new edges are pruned when they overflow
SHAPES = [(36, 8, 31), (4, 12, 32), (64, 30, 33), (100, 63, 64), (32, 32, 65), (36, 95, 96), (132, 64, 97), (8, 100, 127), (36, 127, 128),
          (36, 64, 129), (68, 128, 160), (32, 40, 161), (36, 192, 255), (4, 64, 256), (36, 200, 257), (36, 48, 300)]


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("d,R,L", SHAPES)
def test_block_edges(jx, dtype, d, R, L):
    n = 700
    d = d if dtype == np.float32 else (d + 7) // 8 * 8
    x = datagen.dyadic_grid(n, d, seed=d + L).astype(dtype)
    ref = oracle.Index(d, dtype, R, L, 1.2, n, batch_growth=1.0)
    g = jx.Index(d, jx_dtype(jx, x), R, L, 1.2, capacity=n, max_batch=n, batch_growth=1.0)
    for lo, hi in ((0, 300), (300, n)):
        ref.insert(x[lo:hi])
        g.insert(dev(x[lo:hi]))
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), (lo, hi)
    gone = np.random.default_rng(L).choice(n, n // 5, replace=False).astype(np.uint32)
    ref.delete(gone); g.delete(dev(gone)); ref.consolidate(); g.consolidate()
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), "consolidated"


def test_copies_of_one_point(jx):
    """Distances that are all zero: one block of ties, where order is by id alone and everything is discarded."""
    x = np.repeat(datagen.dyadic_grid(40, 64, seed=3), 8, axis=0)
    ref = oracle.Index(64, np.float32, 24, 100, 1.2, len(x))
    g = jx.Index(64, jx.F32, 24, 100, 1.2, capacity=len(x), max_batch=len(x))
    ref.insert(x)
    g.insert(dev(x))
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0])


def test_rows_that_are_not_finite(jx):
    """A row with NaN and one with infinities among ordinary ones: every call ends, every id is one of the index."""
    n = 600
    x = random_data(n, 100, np.float32, seed=4)
    x[317, 3] = np.nan
    x[400, :] = np.inf
    x[401, 5] = -3.0e38
    g = jx.Index(100, jx.F32, 16, 140, 1.2, capacity=n, max_batch=n)
    g.insert(dev(x[:300]))
    g.insert(dev(x[300:]))
    adj = u32(g.export_graph()[0])
    assert np.all((adj < n) | (adj == 0xFFFFFFFF))


def test_distances_that_overflow(jx):
    """Rows whose squared distance to every other one is infinite: products of the parts of such a value are infinite with
    both signs, and the distance of a present neighbour has to stay infinite, as the list-based kernels have it."""
    n, d = 600, 100
    x = datagen.dyadic_grid(n, d, seed=5).astype(np.float32)
    rng = np.random.default_rng(6)
    far = rng.choice(n, 40, replace=False)
    x[far] = (rng.uniform(1, 2, (40, d)) * 1e22).astype(np.float32)
    for R, L in ((16, 60), (32, 140)):
        gs = [jx.Index(d, jx.F32, R, L, 1.2, capacity=n, max_batch=n, batch_growth=1.0, flags=f) for f in (0, jx.FLAG_NO_GRAM)]
        for lo, hi in ((0, 200), (200, 350), (350, n)):
            for g in gs:
                g.insert(dev(x[lo:hi]))
            a, b = (u32(g.export_graph()[0]) for g in gs)
            assert np.array_equal(a, b), (R, lo, np.flatnonzero((a != b).any(1))[:5])


@pytest.mark.parametrize("d", [16, 96, 128, 144, 256, 272])
@pytest.mark.parametrize("R,L", [(8, 31), (12, 33), (31, 64), (33, 65), (64, 96), (63, 128), (100, 200), (256, 300)])
def test_pivot_rounds_u8(jx, d, R, L):
    """Frontiers of 31 to 300 entries, rows of 8 to 256; 272 bytes take the Gram matrix again."""
    n = 700
    x = random_data(n, d, np.uint8, seed=d + L)
    ref = oracle.Index(d, np.uint8, R, L, 1.2, n, batch_growth=1.0)
    gs = [jx.Index(d, jx.U8, R, L, 1.2, capacity=n, max_batch=n, batch_growth=1.0, flags=f) for f in (0, jx.FLAG_NO_GRAM)]
    gone = np.random.default_rng(L).choice(n, n // 5, replace=False).astype(np.uint32)
    ref.insert(x[:300]); ref.insert(x[300:])
    before = ref.graph()[0].copy()
    ref.delete(gone); ref.consolidate()
    for g in gs:
        g.insert(dev(x[:300])); g.insert(dev(x[300:]))
        assert np.array_equal(u32(g.export_graph()[0]), before)
        g.delete(dev(gone)); g.consolidate()
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), "consolidated"


@pytest.mark.parametrize("alpha", [1.0, 1.05, 1.9, 16.0, 1e30])
def test_discard_limit_u8(jx, alpha):
    """The largest distance at which a candidate is discarded is an integer found from d / alpha: extreme vectors, whose
    distances reach 128 * 255^2, many equal distances, and factors that round either way."""
    rng = np.random.default_rng(3)
    x = rng.choice(np.array([0, 1, 254, 255], np.uint8), (600, 128))
    x[::7] = rng.integers(0, 2, (len(x[::7]), 128), dtype=np.uint8)
    ref = oracle.Index(128, np.uint8, 24, 100, alpha, 600)
    g = jx.Index(128, jx.U8, 24, 100, alpha, capacity=600, max_batch=600)
    ref.insert(x)
    g.insert(dev(x))
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0])


@pytest.mark.parametrize("d", [128, 256])
@pytest.mark.parametrize("copies", [0, 900, 4000])
def test_hub_u8(jx, copies, d):
    """A centre that every point links to: more reverse edges than the first pool (512) and the second (2,048) hold.  With
    copies of three points next to it the closest 512 or 2,048 yield fewer than R neighbours, and the next kernel goes on."""
    rng = np.random.default_rng(8)
    R = 16
    shell = np.clip(np.rint(128 + rng.normal(0, 25, (1500, d))), 0, 255).astype(np.uint8)
    near = 128 + 4 * np.eye(d, dtype=np.int64)[rng.integers(0, 3, copies)]
    x = np.concatenate([np.full((1, d), 128, np.uint8), near.astype(np.uint8), shell])
    n = len(x)
    ref = oracle.Index(d, np.uint8, R, 24, 1.2, n, batch_growth=1.0)
    g = jx.Index(d, jx.U8, R, 24, 1.2, capacity=n, max_batch=n, batch_growth=1.0)
    ref.insert(x[:1]); g.insert(dev(x[:1]))
    for lo in range(1, n, 2700):  # the first of these batches is as large as max_batch lets it be
        ref.insert(x[lo:lo + 2700]); g.insert(dev(x[lo:lo + 2700]))
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), lo


@pytest.mark.parametrize("d", [32, 144, 256])
def test_many_edges_u8(jx, d):
    """A batch of more than 2^20 edges into full rows: merges of at most 128 candidates in a form of their own."""
    n0, batch, R = 263_000, 65_700, 16
    x = random_data(n0 + batch, d, np.uint8, seed=9)
    gs = [jx.Index(d, jx.U8, R, 24, 1.2, capacity=n0 + batch, max_batch=70_000, flags=f) for f in (0, jx.FLAG_NO_GRAM)]
    for g in gs:
        g.insert(dev(x[:n0]))
        g.insert(dev(x[n0:]))
    a, b = (u32(g.export_graph()[0]) for g in gs)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("d", [32, 128, 144, 256])
@pytest.mark.parametrize("R,alpha", [(16, 1.2), (31, 1.0), (32, 1.2), (33, 1.2), (48, 1.05), (64, 1.2), (64, 2.0), (65, 1.2), (96, 1.2)])
def test_rows_that_remember_their_last_prune(jx, d, R, alpha):
    """Streams of batches from one that gives a row an edge now and then to one that gives it more than it takes, with what one
    prune selected at the head of a row: 1 to 15 others behind 1 to 64 of them, and more of either.  The memory has to survive
    other prune kernels, import, deletion and compaction; the table is that of whole prunes after every call."""
    n0, calls = 50_000, [2_048, 2_600, 3_100, 2_100, 2_300, 3_000]
    x = torch.from_numpy(random_data(n0 + sum(calls), d, np.uint8, seed=R + d)).cuda()
    gs = [jx.Index(d, jx.U8, R, 48, alpha, capacity=len(x), max_batch=len(x), batch_growth=1.0, flags=f) for f in (0, jx.FLAG_NO_INCR_PRUNE)]
    at = 0
    for step, m in enumerate([n0, *calls]):
        if step == 2:  # rows are rewritten by the list-based kernels, then by the Gram-matrix ones
            gs[0].set_flags(jx.FLAG_NO_GRAM)
        if step == 3:
            gs[0].set_flags(jx.FLAG_GRAM_U8)
        if step == 4:  # the same graph from outside, its rows in another order: nothing is known about them
            gs[0].set_flags(0)
            adj, deg = gs[1].export_graph()
            place = torch.arange(R, device="cuda")
            turned = adj.gather(1, (deg.long()[:, None] - 1 - place).clamp(min=0))
            turned[place >= deg.long()[:, None]] = -1
            for g in gs:
                g.import_graph(x[:at], turned, g.size()[1])
        if step == 5:
            gone = torch.randperm(at, generator=torch.Generator().manual_seed(R))[:at // 40].int().cuda()
            for g in gs:
                g.delete(gone)
                g.consolidate()
        if step == 6:
            for g in gs:
                g.compact()
        for g in gs:
            g.insert(x[at:at + m])
        at += m
        a, b = (g.export_graph()[0] for g in gs)
        assert torch.equal(a, b), (step, int((a != b).any(1).sum()))


@pytest.mark.parametrize("L,logB", [(8, 24), (129, 23)])
def test_batches_of_more_workgroups_than_one_launch_takes(jx, L, logB):
    """A launch has fewer than 2^32 threads: 2^24 workgroups of 256 (lists of at most 128) and 2^23 of 512 (longer ones) are more.
    Whole numbers below 1,024 in four dimensions are exact in every form, so the table is that of the list-based kernels."""
    n = 2 << logB
    gen = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randint(0, 1024, (n, 4), device="cuda", generator=gen).float()
    tables = []
    for flags in (0, jx.FLAG_NO_GRAM):
        g = jx.Index(4, jx.F32, 4, L, 1.2, capacity=n, max_batch=1 << logB, batch_growth=1.0, flags=flags)
        g.insert(x)
        tables.append(g.export_graph()[0])
        g.close()
    assert torch.equal(*tables)


@pytest.mark.parametrize("d,R,L", [(160, 8, 31), (164, 63, 64), (260, 64, 129), (160, 40, 161), (516, 64, 256), (960, 30, 128), (1536, 48, 300)])
@pytest.mark.parametrize("kind,alpha", [("wide", 1.2), ("wide", 1.0), ("bits", 1.0), ("bits", 1.25), ("tiny", 1.2), ("copies", 1.2)])
def test_long_rows_take_two_parts_first(jx, d, R, L, kind, alpha):
    """Rows of integers that take two bfloat16 parts first, and shorter ones: squared distances below 2^24, of coordinates of as many
    bits as that allows (nine up to 164 dimensions, seven at 1536), of one bit (ties), scaled by 2^-55 (subnormal squares), and
    with many copies.  Every float32 sum is exact, so the table is the oracle's.  The products of two parts are exact as well but
    for the nine bits: test_two_parts_decide_nothing_within_their_error has rows where they are not."""
    n = 600
    rng = np.random.default_rng(d + L)
    lim = 1 if kind == "bits" else int(np.sqrt(2.0 ** 24 / d) / 2 * 0.99)
    x = rng.integers(0 if kind == "bits" else -lim, lim + 1, (n, d)).astype(np.float32)
    if kind == "tiny":
        x *= np.float32(2.0 ** -55)
    if kind == "copies":
        x[rng.permutation(n)[:n // 2]] = x[0]
    ref = oracle.Index(d, np.float32, R, L, alpha, n, batch_growth=1.0)
    g = jx.Index(d, jx.F32, R, L, alpha, capacity=n, max_batch=n, batch_growth=1.0)
    for lo, hi in ((0, 250), (250, n)):
        ref.insert(x[lo:hi])
        g.insert(dev(x[lo:hi]))
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), (lo, hi)
    gone = rng.choice(n, n // 5, replace=False).astype(np.uint32)
    ref.delete(gone); g.delete(dev(gone)); ref.consolidate(); g.consolidate()
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), "consolidated"


@pytest.mark.parametrize("dtype,d", [(np.uint8, 128), (np.uint8, 256), (np.float32, 36), (np.float32, 164), (np.float16, 40)])
@pytest.mark.parametrize("R,most", [(16, 512), (40, 512), (60, 256), (24, 128), (200, 256)])
@pytest.mark.parametrize("over", [0, 1])
def test_segments_as_large_as_a_batch_allows(jx, dtype, d, R, most, over):
    """A hub that every point of a batch links to: its segment holds a full row and the whole batch, as many candidates as the
    kernels that such a batch launches take, and one more.  The table is the oracle's."""
    B = most - R + over
    rng = np.random.default_rng(most + R)
    near = rng.integers(0, 3, (520, d))
    near[0] = 1
    x = np.concatenate([near + 40, rng.integers(0, 90, (300, d))]).astype(dtype) if dtype == np.uint8 else \
        np.concatenate([near, rng.integers(-30, 30, (300, d))]).astype(dtype)
    hub = x[:1].repeat(B, axis=0).astype(np.int64)
    hub[np.arange(B), rng.integers(0, d, B)] += rng.integers(1, 6, B)  # each nearest to the hub
    n = len(x) + B
    ref = oracle.Index(d, dtype, R, 64, 1.2, n, batch_growth=1.0)
    g = jx.Index(d, jx_dtype(jx, x), R, 64, 1.2, capacity=n, max_batch=n, batch_growth=1.0)
    for part in (x, hub.astype(dtype)):
        ref.insert(part)
        g.insert(dev(part))
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0])


@pytest.mark.parametrize("d,R,L", [(316, 30, 100), (320, 8, 31), (320, 63, 64), (516, 64, 129), (960, 64, 256), (1536, 48, 300)])
@pytest.mark.parametrize("kind", ["near", "ties"])
@pytest.mark.parametrize("alpha", [1.04, 1.5, 2.0])
def test_two_parts_decide_nothing_within_their_error(jx, d, R, L, kind, alpha):
    """Rows with one or two coordinates of +-1005, or of +-1004 .. 1006: ten bits, so a product of two second parts is missing
    from what two parts give.  Squared distances are multiples of 1005^2, or a few units off: at alpha = 1.5 / 2 two parts alone
    decide 16 / 6 comparisons of the 128 closest candidates wrongly where some 160 / 20 are undecided (near), and 2,100 / 77 of as
    many (ties), on either side of what a prune settles pair by pair.  |x_i - p|^2 + |x_j - p|^2 stays below 2^24, where every sum is
    exact, so the table is the oracle's."""
    n = 600
    rng = np.random.default_rng(d + L)
    at = rng.choice(d, 24, replace=False)
    x = np.zeros((n, d), np.float32)
    for row in x[1:]:  # the first one stays at the origin: it is nearest to the mean of the others, which are at equal distances
        m = rng.integers(1, 3)
        row[rng.choice(at, m, replace=False)] = 1005 * rng.choice([-1, 1], m) + (rng.integers(-1, 2, m) if kind == "near" else 0)
    ref = oracle.Index(d, np.float32, R, L, alpha, n, batch_growth=1.0)
    g = jx.Index(d, jx.F32, R, L, alpha, capacity=n, max_batch=n, batch_growth=1.0)
    for lo, hi in ((0, 250), (250, n)):
        ref.insert(x[lo:hi])
        g.insert(dev(x[lo:hi]))
        assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), (lo, hi)
    gone = rng.choice(n, n // 5, replace=False).astype(np.uint32)
    ref.delete(gone); g.delete(dev(gone)); ref.consolidate(); g.consolidate()
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0]), "consolidated"


@pytest.mark.parametrize("R,L", [(16, 60), (16, 140), (24, 33), (64, 129)])
@pytest.mark.parametrize("d", [320, 960])
def test_long_rows_that_are_not_finite(jx, d, R, L):
    """As test_rows_that_are_not_finite, on rows that take two parts first.  A vector with an infinite coordinate cannot be told from
    the zeros that fill the last block of candidates; these have no id and no vector."""
    n = 600
    x = random_data(n, d, np.float32, seed=4)
    x[317, 3] = np.nan
    x[400, :] = np.inf
    x[401, 5] = -3.0e38
    x[np.arange(310, 340, 7), 9] = np.inf
    x[350:353, d - 1] = [3.0e38, -np.inf, np.inf]
    g = jx.Index(d, jx.F32, R, L, 1.2, capacity=n, max_batch=n)
    g.insert(dev(x[:300]))
    g.insert(dev(x[300:]))
    adj = u32(g.export_graph()[0])
    assert np.all((adj < n) | (adj == 0xFFFFFFFF))


@pytest.mark.parametrize("d", [320, 960])
def test_distances_of_long_rows_that_overflow(jx, d):
    """As test_distances_that_overflow, on rows that take two parts first: their squares are summed apart from the products."""
    n = 600
    x = datagen.dyadic_grid(n, d, seed=5).astype(np.float32)
    rng = np.random.default_rng(6)
    far = rng.choice(n, 40, replace=False)
    x[far] = (rng.uniform(1, 2, (40, d)) * 1e22).astype(np.float32)
    for R, L in ((16, 60), (32, 140)):
        gs = [jx.Index(d, jx.F32, R, L, 1.2, capacity=n, max_batch=n, batch_growth=1.0, flags=f) for f in (0, jx.FLAG_NO_GRAM)]
        for lo, hi in ((0, 200), (200, 350), (350, n)):
            for g in gs:
                g.insert(dev(x[lo:hi]))
            a, b = (u32(g.export_graph()[0]) for g in gs)
            assert np.array_equal(a, b), (R, lo, np.flatnonzero((a != b).any(1))[:5])
