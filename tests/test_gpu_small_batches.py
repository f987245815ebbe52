"""Small batches run on kernels of their own (more records in flight, a team of wavefronts per query that reads ahead),
larger ones on one wavefront per query.  All of them are the same search: ids, distances (to the last bit) and expansion
counts equal those of the general kernel, which a full-id visited table selects, on both sides of every size limit."""
import numpy as np
import pytest
import torch

from gpu_common import dev, jx_dtype, random_data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


def _compare(jx, g, q, L, **kw):
    g.set_flags(0)
    ids, dist, st = g.search(q, min(10, L), L, stats=True, **kw)
    g.set_flags(jx.FLAG_VISITED_IDS | jx.FLAG_NO_PAIR)
    ids0, dist0, st0 = g.search(q, min(10, L), L, stats=True, **kw)
    g.set_flags(0)
    assert st0["beam_kernel"].startswith("beam_search_kernel<") and st0["beam_kernel"].endswith(",0>"), st0["beam_kernel"]
    assert torch.equal(ids, ids0), st["beam_kernel"]
    assert torch.equal(dist, dist0), st["beam_kernel"]
    assert st["hops"] == st0["hops"], st["beam_kernel"]
    return st["beam_kernel"].split("<")[0]


@pytest.mark.parametrize("dtype,d,R", [("uint8", 128, 64), ("uint8", 96, 33), ("uint8", 256, 64), ("uint8", 128, 80),
                                       ("float32", 128, 64), ("float32", 100, 17), ("float32", 200, 64), ("float32", 960, 64),
                                       ("float32", 1536, 40), ("float16", 128, 64), ("float16", 960, 64)])
def test_small_batches_equal_the_general_kernel(jx, dtype, d, R):
    n = 3000
    x = random_data(n, d, np.uint8 if dtype == "uint8" else np.float32, 5).astype(dtype)
    q = random_data(2100, d, np.uint8 if dtype == "uint8" else np.float32, 6).astype(dtype)
    g = jx.Index(d, jx_dtype(jx, x), R, 64, 1.2, capacity=n, max_batch=4096)
    g.insert(dev(x))
    names = set()
    for L in (1, 16, 64, 65, 128, 200):
        for nq in (1, 3, 256, 257, 513, 2049):
            if nq > 513 and L not in (16, 65):
                continue
            names.add(_compare(jx, g, dev(q[:nq]), L))
    assert ("beam_search_ahead_kernel" in names) == (d >= 200 and dtype != "uint8" and R <= 64), names


@pytest.mark.parametrize("d,bits,qbits", [(960, 4, 8), (960, 4, 4), (960, 8, 8), (1536, 1, 4), (1536, 2, 4), (960, 1, 8), (128, 4, 8)])
def test_small_batches_of_code_searches(jx, d, bits, qbits):
    n = 2000
    x = random_data(n, d, np.float32, 7)
    q = random_data(600, d, np.float32, 8)
    g = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n, max_batch=4096, quant_bits=bits)
    g.insert(dev(x))
    rot = np.linalg.qr(np.random.default_rng(9).standard_normal((d, d)))[0].astype(np.float32)
    g.quantize(bits, dev(rot), query_bits=qbits, rule=jx.RULE_MAXABS)
    names = set()
    for L in (16, 100, 192):
        for nq in (1, 255, 600):
            names.add(_compare(jx, g, dev(q[:nq]), L, mode=jx.RABITQ))
    assert ("beam_search_ahead_kernel" in names) == (d >= 960), names


@pytest.mark.parametrize("d", [128, 960])
def test_expansion_list_builds_equal_the_general_kernel(jx, d):
    """The candidate search of insertion that returns the expansion list, one wavefront per point: a graph built from small
    internal batches (wide instances among them) is the graph of the general kernel."""
    x = random_data(2500, d, np.float32, 11)
    adj = []
    for flags in (0, jx.FLAG_VISITED_IDS):
        g = jx.Index(d, jx.F32, 64, 96, 1.2, capacity=2500, max_batch=4096, cand_mode=jx.CAND_VISITED, flags=flags)
        g.insert(dev(x))
        adj.append(g.export_graph()[0])
    assert torch.equal(adj[0], adj[1])


@pytest.mark.parametrize("d,n,bits", [(200, 40_000, 0), (960, 20_000, 0), (960, 30_000, 4)])
def test_teams_evaluate_what_the_table_forgot(jx, d, n, bits):
    """On enough vertices sets of the visited table overflow: neighbours it held when a team read their row ahead and has
    forgotten by the expansion (d = 200, 64 queries: 265 of them at L = 64, 1,618 at 256) are evaluated there.  The
    one-wavefront kernel with the same table (a switch that concerns other records leaves the teams out) does the same."""
    x, q = random_data(n, d, np.float32, 5), random_data(64, d, np.float32, 6)
    g = jx.Index(d, jx.F32, 64, 64, 1.2, capacity=n, max_batch=n, quant_bits=bits)
    g.insert(dev(x))
    kw = {}
    if bits:
        rot = np.linalg.qr(np.random.default_rng(9).standard_normal((d, d)))[0].astype(np.float32)
        g.quantize(bits, dev(rot), query_bits=8, rule=jx.RULE_MAXABS)
        kw["mode"] = jx.RABITQ
    for L in (64, 128, 256):
        got = []
        for flags, kernel in ((0, "beam_search_ahead_kernel<"), (jx.FLAG_NO_PAIR, "beam_search_kernel<")):
            g.set_flags(flags)
            ids, dist, st = g.search(dev(q), 10, L, stats=True, **kw)
            assert st["beam_kernel"].startswith(kernel), st["beam_kernel"]
            got.append((ids, dist, st["hops"], st["dist_evals"]))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        assert got[0][2:] == got[1][2:]


@pytest.mark.parametrize("dtype,d,L,most", [("float32", 200, 128, 1536), ("float32", 200, 200, 1024), ("float16", 960, 200, 1024),
                                            ("float32", 960, 128, 1280), ("float32", 960, 32, 1536), ("float32", 1536, 33, 1024)])
def test_wide_instances_end_where_they_lose(jx, dtype, d, L, most):
    """The instance with more records in flight runs up to the batch that its registers and the bandwidth allow, the usual
    one from there on; both return the same."""
    x = random_data(2000, d, np.float32, 15).astype(dtype)
    q = dev(random_data(most + 1, d, np.float32, 16).astype(dtype))
    g = jx.Index(d, jx_dtype(jx, x), 32, 48, 1.2, capacity=2000, max_batch=2048)
    g.insert(dev(x))
    ids, dist, st = g.search(q[:most], 10, L, stats=True)
    ids1, dist1, st1 = g.search(q, 10, L, stats=True)
    assert st["beam_kernel"].endswith(",2>") and st1["beam_kernel"].endswith(",1>"), (st["beam_kernel"], st1["beam_kernel"])
    assert torch.equal(ids, ids1[:most]) and torch.equal(dist, dist1[:most])


@pytest.mark.parametrize("dtype,d,R,L,form", [
    ("float16", 128, 64, 200, {1000: 2, 4096: 1, 4097: 0}), ("uint8", 256, 16, 150, {1000: 1, 4097: 0}), ("float32", 200, 64, 200, {4097: 1}),
    ("float32", 96, 16, 200, {1000: 1}), ("float32", 96, 17, 200, {1000: 2}), ("float32", 96, 32, 300, {1000: 0}), ("float32", 96, 33, 300, {1000: 2, 1025: 2, 1537: 0}),
    ("float32", 960, 16, 300, {1000: 2, 1025: 0}), ("float32", 960, 16, 64, {1000: 2})])
def test_forms_end_where_they_lose(jx, dtype, d, R, L, form):
    """Rows that the usual form covers, frontiers of six registers and more, short records beyond four wavefronts per SIMD:
    each batch runs in the form that is the fastest there, and all return the same."""
    n = 1500
    x = random_data(n, d, np.uint8 if dtype == "uint8" else np.float32, 17).astype(dtype)
    q = dev(random_data(4097, d, np.uint8 if dtype == "uint8" else np.float32, 18).astype(dtype))
    g = jx.Index(d, jx_dtype(jx, x), R, 48, 1.2, capacity=n, max_batch=4097)
    g.insert(dev(x))
    g.set_flags(jx.FLAG_VISITED_IDS)
    ids0, dist0, st0 = g.search(q, 10, L, stats=True)
    assert st0["beam_kernel"].endswith(",0>")
    g.set_flags(0)
    for nq, mode in form.items():
        ids, dist, st = g.search(q[:nq], 10, L, stats=True)
        assert st["beam_kernel"].startswith("beam_search_kernel<") and st["beam_kernel"].endswith(f",{mode}>"), (nq, st["beam_kernel"])
        assert torch.equal(ids, ids0[:nq]) and torch.equal(dist, dist0[:nq])


@pytest.mark.parametrize("R,L,team", [(64, 200, True), (33, 200, True), (32, 200, False), (32, 128, True), (16, 64, False)])
def test_teams_need_rows_to_read_ahead(jx, R, L, team):
    n, d = 1500, 960
    x, q = random_data(n, d, np.float32, 19), random_data(64, d, np.float32, 20)
    g = jx.Index(d, jx.F32, R, 48, 1.2, capacity=n, max_batch=4096, quant_bits=4)
    g.insert(dev(x))
    rot = np.linalg.qr(np.random.default_rng(9).standard_normal((d, d)))[0].astype(np.float32)
    g.quantize(4, dev(rot), query_bits=8, rule=jx.RULE_MAXABS)
    assert _compare(jx, g, dev(q), L, mode=jx.RABITQ) == ("beam_search_ahead_kernel" if team else "beam_search_kernel")
