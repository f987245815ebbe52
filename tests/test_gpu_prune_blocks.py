"""robustPrune as one Gram matrix per workgroup: candidate lists around the edges of its 32-row blocks and of its two
sizes (128, 256), with rows that end inside a 128-byte piece.  The data lie on a dyadic grid, where every partial sum is
exact in float32 (and in the three bfloat16 parts of a value), so the adjacency table is the oracle's, bit for bit."""
import numpy as np
import pytest

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
