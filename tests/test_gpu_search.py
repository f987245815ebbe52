"""GPU parity: beamSearch and brute force through the C ABI vs the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_07048_amd import datagen
from gpu_common import dev, u32, random_data, oracle_index, gpu_index_from_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


@pytest.fixture(scope="module")
def u8_case(jx):
    n = 20000
    x = datagen.base(2, n)
    q = datagen.queries(2, 203)  # not a multiple of the queries per workgroup
    ix = oracle_index(x, 64, 64)
    g = gpu_index_from_oracle(jx, x, ix, 64, 64)
    return x, q, ix, g


@pytest.fixture(scope="module")
def f32_case(jx):
    n = 10000
    x = datagen.base(1, n)[datagen.insertion_order(1, n)]
    q = datagen.queries(1, 200)
    ix = oracle_index(x, 32, 64)
    g = gpu_index_from_oracle(jx, x, ix, 32, 64)
    return x, q, ix, g


@pytest.mark.parametrize("L", [1, 10, 32, 64, 100, 128, 200, 256, 300, 512])
def test_beam_u8_bit_exact(jx, u8_case, L):
    """Integer distances: the whole frontier (ids and distances), the number of
    expansions and the bounds on distance evaluations must match the oracle."""
    x, q, ix, g = u8_case
    ref = ix.search(q, 1, L, want_frontier=True)
    ref_nofilter = ix.search(q, 1, L, filter=oracle.FILTER_NONE)
    ids, dist, st = g.beam_frontier(dev(q), L, stats=True)
    ids, dist = u32(ids), dist.cpu().numpy()
    assert np.array_equal(ids, ref["F_ids"])
    assert np.array_equal(dist.astype(np.float64), ref["F_dist"])
    assert st["hops"] == ref["hops"]
    assert ref["evals"] <= st["dist_evals"] <= ref_nofilter["evals"]
    assert st["adj_bytes"] == st["hops"] * 4 * 64 and st["vec_bytes"] == st["dist_evals"] * 128


def test_search_topk_is_frontier_prefix_and_deterministic(jx, u8_case):
    x, q, ix, g = u8_case
    dq = dev(q)
    a_ids, a_dist = g.search(dq, 10, 64)
    b_ids, b_dist = g.search(dq, 10, 64)
    f_ids, f_dist = g.beam_frontier(dq, 64)
    assert torch.equal(a_ids, b_ids) and torch.equal(a_dist, b_dist)
    assert torch.equal(a_ids, f_ids[:, :10]) and torch.equal(a_dist, f_dist[:, :10])
    ref = ix.search(q, 10, 64)
    assert np.array_equal(u32(a_ids), ref["ids"])


def test_exact_searches_in_flight_on_two_streams(jx, u8_case):
    """jx_search in JX_EXACT mode without statistics only reads the index and writes its own outputs: calls issued
    alternately on two streams, with a result buffer each, overlap on the device and every one returns the oracle's
    ids and distances."""
    x, q, ix, g = u8_case
    big = np.concatenate([q] * 40)   # 8,120 queries: long enough launches to overlap
    dq = dev(big)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [(torch.empty((big.shape[0], 10), dtype=torch.int32, device="cuda"),
             torch.empty((big.shape[0], 10), dtype=torch.float32, device="cuda")) for _ in range(4)]
    torch.cuda.synchronize()
    for i in range(8):
        with torch.cuda.stream(streams[i & 1]):
            g.search(dq, 10, 64 if i & 2 else 32, out=outs[i & 3])
    torch.cuda.synchronize()
    for L, pair in ((32, (0, 1)), (64, (2, 3))):
        ref = ix.search(q, 10, L)
        for o in pair:
            ids, dist = outs[o]
            assert np.array_equal(u32(ids)[:q.shape[0]], ref["ids"]) and np.array_equal(u32(ids)[-q.shape[0]:], ref["ids"])
            assert np.array_equal(dist.cpu().numpy().astype(np.float64)[:q.shape[0]], ref["dist"])


@pytest.mark.parametrize("L", [16, 64, 130])
def test_beam_f32_tolerance(jx, f32_case, L):
    """float32 distances: within 1e-4 relative of the oracle's double result;
    ids compared where the oracle's gap to both neighbours exceeds that."""
    x, q, ix, g = f32_case
    ref = ix.search(q, 1, L, want_frontier=True)
    ids, dist = g.beam_frontier(dev(q), L)
    ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
    rd, ri = ref["F_dist"], ref["F_ids"]
    assert np.allclose(dist, rd, rtol=1e-4, atol=0)
    gap_prev = np.abs(np.diff(rd, axis=1, prepend=-np.inf))
    gap_next = np.abs(np.diff(rd, axis=1, append=np.inf))
    safe = (gap_prev > 2e-4 * rd) & (gap_next > 2e-4 * rd)
    assert safe.mean() > 0.8
    assert np.array_equal(ids[safe], ri[safe])
    # recall against brute force within 0.002 of the oracle's
    gt, _ = oracle.bruteforce(x, q, min(10, L))
    k = min(10, L)
    assert abs(oracle.recall_at_k(ids[:, :k], gt) - oracle.recall_at_k(ri[:, :k], gt)) <= 0.002


def test_beam_f32_dyadic_grid_bit_exact(jx):
    """Points on a coarse dyadic grid make every float32 partial sum exact in
    any order, so the float path can be compared bit for bit."""
    x = datagen.dyadic_grid(4000, 64, seed=5)
    q = datagen.dyadic_grid(100, 64, seed=6)
    ix = oracle_index(x, 24, 48)
    g = gpu_index_from_oracle(jx, x, ix, 24, 48)
    for L in (20, 70):
        ref = ix.search(q, 1, L, want_frontier=True)
        ids, dist, st = g.beam_frontier(dev(q), L, stats=True)
        assert np.array_equal(u32(ids), ref["F_ids"])
        assert np.array_equal(dist.cpu().numpy().astype(np.float64), ref["F_dist"])
        assert st["hops"] == ref["hops"]


@pytest.mark.parametrize("dtype,d", [(np.uint8, 16), (np.uint8, 64), (np.uint8, 256), (np.uint8, 1024),
                                     (np.uint8, 2048), (np.uint8, 4096), (np.uint8, 6144),
                                     (np.float32, 4), (np.float32, 96), (np.float32, 200), (np.float32, 960),
                                     (np.float32, 1536)])
def test_beam_shapes(jx, dtype, d):
    """Every lanes-per-record / chunks-per-lane variant, ragged dimensions."""
    n = 1500
    x = random_data(n, d, dtype, seed=d)
    q = random_data(37, d, dtype, seed=d + 1)
    ix = oracle_index(x, 20, 40)
    g = gpu_index_from_oracle(jx, x, ix, 20, 40)
    ref = ix.search(q, 1, 50, want_frontier=True)
    ids, dist = g.beam_frontier(dev(q), 50)
    ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
    if dtype == np.uint8:
        # the order is decided on exact integers; the returned float32 is the
        # exact distance when it is below 2^24 (d <= 256), else its nearest float
        assert np.array_equal(ids, ref["F_ids"])
        assert np.array_equal(dist, ref["F_dist"].astype(np.float32).astype(np.float64))
    else:
        assert np.allclose(dist, ref["F_dist"], rtol=1e-4)
        assert (ids == ref["F_ids"]).mean() > 0.98


@pytest.mark.parametrize("R", [1, 7, 64, 100, 256])
def test_beam_degrees(jx, R):
    x = random_data(1200, 32, np.uint8, seed=R)
    q = random_data(21, 32, np.uint8, seed=R + 1)
    ix = oracle_index(x, R, 32)
    g = gpu_index_from_oracle(jx, x, ix, R, 32)
    ref = ix.search(q, 1, 40, want_frontier=True)
    ids, dist, st = g.beam_frontier(dev(q), 40, stats=True)
    assert np.array_equal(u32(ids), ref["F_ids"])
    assert st["hops"] == ref["hops"]


def test_beam_small_index_and_padding(jx):
    """N < L: the frontier never fills; unused slots are NONE / +inf.  An entry
    with no edges returns only itself."""
    x = random_data(9, 16, np.uint8, seed=1)
    ix = oracle_index(x, 4, 8)
    g = gpu_index_from_oracle(jx, x, ix, 4, 8)
    q = random_data(5, 16, np.uint8, seed=2)
    ref = ix.search(q, 1, 32, want_frontier=True)
    ids, dist = g.beam_frontier(dev(q), 32)
    assert np.array_equal(u32(ids), ref["F_ids"])
    d = dist.cpu().numpy()
    assert np.isinf(d[u32(ids) == jx.NONE]).all() and (u32(ids) == jx.NONE).any()
    adj = np.full((9, 4), jx.NONE, np.uint32)
    g.import_graph(dev(x), dev(adj), 3)
    ids, dist = g.search(dev(q), 2, 4)
    assert (u32(ids)[:, 0] == 3).all() and (u32(ids)[:, 1] == jx.NONE).all()


def test_search_argument_errors(jx, u8_case):
    x, q, ix, g = u8_case
    dq = dev(q)
    with pytest.raises(jx.JxError):
        g.search(dq, 11, 10)            # k > L
    with pytest.raises(jx.JxError):
        g.search(dq, 10, jx.MAX_L + 1)  # L too large
    with pytest.raises(jx.JxError):
        g.search(dq, 10, 64, mode=jx.RABITQ)  # not quantised
    e = jx.Index(128, jx.U8, 8, 8, 1.2, capacity=16)
    with pytest.raises(jx.JxError):
        e.search(dq, 1, 8)              # empty index
    ids, dist = g.search(dq[:0], 10, 64)  # empty batch is fine
    assert ids.shape == (0, 10)
    with pytest.raises(jx.JxError):
        jx.Index(100, jx.U8, 8, 8, 1.2, capacity=16)  # bad dim


@pytest.mark.parametrize("dtype,n,d,k", [(np.uint8, 5000, 128, 10), (np.uint8, 777, 32, 1), (np.float32, 3000, 96, 100),
                                         (np.float32, 1000, 960, 10), (np.uint8, 100, 16, 128)])
def test_bruteforce_parity(jx, dtype, n, d, k):
    x = random_data(n, d, dtype, seed=n)
    q = random_data(70, d, dtype, seed=n + 1)
    g = jx.Index(d, jx.U8 if dtype == np.uint8 else jx.F32, 8, 8, 1.2, capacity=n)
    adj = np.full((n, 8), jx.NONE, np.uint32)
    g.import_graph(dev(x), dev(adj), 0)
    ids, dist = g.bruteforce(dev(q), k)
    ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
    rid, rd = oracle.bruteforce(x, q, k)
    if dtype == np.uint8:
        assert np.array_equal(ids, rid) and np.array_equal(dist, rd)
    else:
        fin = np.isfinite(rd)
        assert np.allclose(dist[fin], rd[fin], rtol=1e-4)
        assert np.array_equal(np.isfinite(dist), fin)
        assert (ids == rid).mean() > 0.99


def test_import_graph_rejects_a_bad_table(jx):
    """Ids out of range, a row with a gap or a row that names a vertex twice would send the kernels out of bounds:
    refused before any kernel runs on the table, index unchanged."""
    x = random_data(300, 32, np.uint8, seed=1)
    ix = oracle_index(x, 8, 16)
    g = gpu_index_from_oracle(jx, x, ix, 8, 16)
    adj, _ = ix.graph()
    for bad in ("range", "gap", "repeat", "repeat-far"):
        a = adj.copy()
        if bad == "range":
            a[7, 0] = 300
        elif bad == "repeat":
            a[11, :] = [4, 5, 4, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF]
        elif bad == "repeat-far":
            a[299, :] = [1, 2, 3, 4, 5, 6, 7, 1]
        else:
            a[9, :] = [5, 0xFFFFFFFF, 6, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF, 0xFFFFFFFF]
        with pytest.raises(jx.JxError) as e:
            g.import_graph(dev(x), dev(a), ix.entry)
        assert e.value.code == -1
    got, _ = g.export_graph()
    assert np.array_equal(u32(got), adj)


def test_ablation_variants_uint8_bit_exact(jx, u8_case):
    """The kernel variants of the ablation (jx_set_flags) on 128-byte uint8 vectors: every visited-filter, lane,
    load and workgroup variant returns the oracle's frontier (ids, distances) and expansion count."""
    x, q, ix, g = u8_case
    variants = [0, jx.FLAG_NO_PAIR, jx.FLAG_VISITED_IDS, jx.FLAG_VISITED_NONE, jx.FLAG_LANES_WIDE, jx.FLAG_LANES_NARROW,
                jx.FLAG_TILED_LOADS, jx.FLAG_QPW_2, jx.FLAG_QPW_4, jx.FLAG_QPW_4 | jx.FLAG_VISITED_NONE,
                jx.FLAG_TILED_LOADS | jx.FLAG_VISITED_IDS]
    names = set()
    try:
        for L in (10, 64, 100, 200):
            ref = ix.search(q, 1, L, want_frontier=True)
            nof = ix.search(q, 1, L, filter=oracle.FILTER_NONE)
            for fl in variants:
                g.set_flags(fl)
                ids, dist, st = g.beam_frontier(dev(q), L, stats=True)
                names.add(st["beam_kernel"].split("<")[0] + "<" + ",".join(st["beam_kernel"].split("<")[1].split(",")[:3]))
                # two expansions per round: with one and two frontier registers on a table of full ids, with four on either
                if fl in (0, jx.FLAG_VISITED_IDS):
                    assert ("pair" in st["beam_kernel"]) == (L == 200 or (L >= 64 and fl == jx.FLAG_VISITED_IDS)), (fl, L)
                assert np.array_equal(u32(ids), ref["F_ids"]), (fl, L)
                assert np.array_equal(dist.cpu().numpy().astype(np.float64), ref["F_dist"]), (fl, L)
                assert st["hops"] == ref["hops"], (fl, L)
                if fl & jx.FLAG_VISITED_NONE:
                    assert st["dist_evals"] == nof["evals"], (fl, L)   # Alg. 2 as printed
                else:
                    assert ref["evals"] <= st["dist_evals"] <= nof["evals"], (fl, L)
        # a combination without an instance fails loudly instead of running something else
        g.set_flags(jx.FLAG_TILED_LOADS | jx.FLAG_QPW_2)
        with pytest.raises(jx.JxError):
            g.beam_frontier(dev(q), 64)
    finally:
        g.set_flags(0)
    assert {"beam_search_pair_kernel<0,4,2", "beam_search_kernel<0,4,2", "beam_search_kernel<0,8,1", "beam_search_kernel<0,2,4",
            "beam_search_variant_kernel<0,4,2"} <= names, names


@pytest.mark.parametrize("d", [96, 960, 1536])
def test_ablation_variants_float32_bit_exact(jx, d):
    """Tiled loads and wavefront teams on float32 vectors of the sizes the ablation measures.  Points on a dyadic grid
    make every partial sum exact, so each variant must give the oracle's frontier bit for bit."""
    n = 1200
    x = datagen.dyadic_grid(n, d, seed=d, step=0.25, lim=2.0)
    q = datagen.dyadic_grid(33, d, seed=d + 1, step=0.25, lim=2.0)
    ix = oracle_index(x, 20, 40)
    g = gpu_index_from_oracle(jx, x, ix, 20, 40)
    variants = [0, jx.FLAG_TILED_LOADS, jx.FLAG_VISITED_NONE] + ([jx.FLAG_WAVES_2, jx.FLAG_WAVES_4, jx.FLAG_WAVES_4 | jx.FLAG_VISITED_NONE] if d >= 960 else [])
    if d == 1536:
        variants.remove(jx.FLAG_TILED_LOADS)   # no tiled instance for 384-chunk records
    for L in (8, 64, 150):
        ref = ix.search(q, 1, L, want_frontier=True)
        for fl in variants:
            g.set_flags(fl)
            ids, dist, st = g.beam_frontier(dev(q), L, stats=True)
            assert np.array_equal(u32(ids), ref["F_ids"]), (fl, L, st["beam_kernel"])
            assert np.array_equal(dist.cpu().numpy().astype(np.float64), ref["F_dist"]), (fl, L)
            assert st["hops"] == ref["hops"], (fl, L)
            if fl & (jx.FLAG_WAVES_2 | jx.FLAG_WAVES_4):
                assert st["beam_kernel"].startswith("beam_search_team_kernel<1,64,")
