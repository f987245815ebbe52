"""The sorts behind insertion and consolidation at the sizes where they change form: up to 8,192 edges in one workgroup, up
to 2^20 by merge passes, the radix sort beyond.  The same points inserted with batches of other sizes go through other
forms; every graph equals the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_common import dev, random_data, u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


# edges of the last internal batch = points x R: one workgroup (full and not), one merge, several, runs that end
# early; 2^20 edges exactly (merge passes) and just more (radix sort, six passes, and seven where ids have 17 bits)
@pytest.mark.parametrize("n0,batch,R", [(1500, 1, 16), (1500, 33, 31), (2100, 512, 16), (2100, 513, 16), (3000, 700, 24), (6000, 1400, 48),
                                        (16_400, 4096, 256), (16_400, 4097, 256), (66_000, 4097, 256)])
def test_insert_batches_equal_the_oracle(jx, n0, batch, R):
    x = random_data(n0 + batch, 32, np.uint8, 31)
    x[100:200] = x[0]  # equal distances
    g = jx.Index(32, jx.U8, R, 24, 1.2, capacity=n0 + batch, max_batch=max(4096, n0 // 4))
    g.insert(dev(x[:n0]))
    full = oracle.Index(32, np.uint8, R, 24, 1.2, n0 + batch)
    full.insert(x[:n0])
    full.insert(x[n0:])
    g.insert(dev(x[n0:]))
    assert np.array_equal(u32(g.export_graph()[0]), full.graph()[0])


# the widths of the one-workgroup network (64, 256, 1,024, 2,048, 4,096 edges), then chunks of 2,048 and a merge of two, of eight,
# a second pass of eight, a third, and chunks of 4,096: each size exactly, and one point more
@pytest.mark.parametrize("n0,batch,R", [(300, 4, 16), (300, 5, 16), (300, 16, 16), (300, 17, 16), (300, 64, 16), (300, 65, 16), (1100, 128, 16),
                                        (1100, 129, 16), (1100, 256, 16), (1100, 257, 16), (4200, 1024, 16), (4200, 1025, 16), (8300, 2048, 64),
                                        (8300, 2049, 64), (16_400, 4096, 64), (16_400, 4097, 64)])
def test_widths_of_the_sorts_equal_the_oracle(jx, n0, batch, R):
    test_insert_batches_equal_the_oracle(jx, n0, batch, R)


@pytest.mark.parametrize("drop", [3, 40, 700])
def test_consolidation_equals_the_oracle(jx, drop):
    n, R = 4000, 24
    x = random_data(n, 32, np.uint8, 32)
    ref = oracle.Index(32, np.uint8, R, 32, 1.2, n)
    ref.insert(x)
    g = jx.Index(32, jx.U8, R, 32, 1.2, capacity=n, max_batch=4096)
    g.insert(dev(x))
    ids = np.random.default_rng(4).choice(n, drop, replace=False).astype(np.uint32)
    ref.delete(ids)
    ref.consolidate()
    g.delete(dev(ids))
    g.consolidate()
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0])


@pytest.mark.parametrize("max_batch", [16_384, 20_000])
def test_consolidation_by_the_longest_sorts_equals_the_oracle(jx, max_batch):
    """1.6 M candidates in slices of at most max_batch x R: 2^20 (merge passes), and 1.28 M (radix sorts, the first of them
    without passes over digits that are zero)."""
    n, R = 20_000, 64
    x = random_data(n, 32, np.uint8, 33)
    ref = oracle.Index(32, np.uint8, R, 32, 1.2, n)
    ref.insert(x)
    g = jx.Index(32, jx.U8, R, 32, 1.2, capacity=n, max_batch=max_batch)
    g.insert(dev(x))
    ids = np.random.default_rng(4).choice(n, 4_000, replace=False).astype(np.uint32)
    rows = ref.graph()[0].astype(np.int64)
    live = ~np.isin(np.arange(n), ids)
    valid = rows != 0xFFFFFFFF
    dead = valid & ~live[np.where(valid, rows, 0)]
    kept = (valid & ~dead).sum(1)  # of a row of each vertex: what it hands on where it is deleted
    assert (np.where(dead, kept[np.where(valid, rows, 0)], 0).sum(1) + kept)[live & dead.any(1)].sum() > 1_500_000
    ref.delete(ids)
    ref.consolidate()
    g.delete(dev(ids))
    g.consolidate()
    assert np.array_equal(u32(g.export_graph()[0]), ref.graph()[0])
