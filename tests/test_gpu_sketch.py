"""float32 searches that read byte copies of the vectors first leave out what cannot enter a frontier: ids, distances (to the
last bit), expansion lists and expansion counts are those of the general kernel, which a full-id visited table selects."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import dev, random_data, u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


def _same(jx, g, q, L, want_sketch=True):
    g.set_flags(0)
    ids, dist, st = g.search(q, min(10, L), L, stats=True)
    g.set_flags(jx.FLAG_VISITED_IDS)
    ids0, dist0, st0 = g.search(q, min(10, L), L, stats=True)
    g.set_flags(0)
    assert st["beam_kernel"].startswith("beam_search_sketch_kernel<") == want_sketch, st["beam_kernel"]
    assert st0["beam_kernel"].startswith("beam_search_kernel<"), st0["beam_kernel"]
    assert torch.equal(ids, ids0), (L, st["beam_kernel"])
    assert torch.equal(dist.view(torch.int32), dist0.view(torch.int32)), (L, st["beam_kernel"])
    assert st["hops"] == st0["hops"], (L, st["beam_kernel"])


def _mixed(n, d, seed, extremes=True):
    """Clusters near and far from the origin, long and short vectors, copies, one-sided rows, constant and single-spike rows,
    rows without a byte copy (beyond 1e17, infinities, NaN) and rows whose squares are subnormal."""
    x = random_data(n, d, np.float32, seed)
    rng = np.random.default_rng(seed + 1)
    part = np.array_split(rng.permutation(n)[:n // 2], 10)
    x[part[0]] += np.float32(300)
    x[part[1]] *= np.float32(1e-3)
    x[part[2]] = x[part[2][0]]
    x[part[3]] = np.abs(x[part[3]])
    x[part[4]] = rng.standard_normal((len(part[4]), 1)).astype(np.float32)
    x[part[5]] = 0
    x[part[5], rng.integers(0, d, len(part[5]))] = 50
    x[part[6]] *= np.float32(1e-25)
    x[part[7]] += rng.integers(0, 2, (len(part[7]), d)).astype(np.float32) * np.float32(1e4)
    if not extremes:
        return x
    odd = part[8][:12]
    x[odd[:4], 3] = [np.inf, -np.inf, np.nan, 3e38]
    x[odd[4:8]] *= np.float32(1e18)
    x[odd[8:12]] *= np.float32(5e16)
    return x


@pytest.mark.parametrize("d,R,n", [(132, 64, 9000), (200, 33, 6000), (256, 64, 5000), (260, 64, 5000), (516, 64, 9000), (960, 64, 5000),
                                   (1024, 17, 5000), (1028, 64, 5000), (1536, 64, 3000)])
def test_searches_equal_the_general_kernel(jx, d, R, n):
    q = np.concatenate([random_data(1500, d, np.float32, 32), _mixed(1200, d, 33)])
    x = random_data(n, d, np.float32, 31)
    g = jx.Index(d, jx.F32, R, 48, 1.2, capacity=n, max_batch=n)
    g.insert(dev(x))
    adj, entry = g.export_graph()[0], g.size()[1]
    for y in (x, _mixed(n, d, 31)):
        g.import_graph(dev(y), adj, entry)
        for L in (1, 10, 64, 65, 128, 129, 256):
            for nq in (513, 2700):
                _same(jx, g, dev(q[:nq]), L, want_sketch=d > 256 or L <= 128)


@pytest.mark.parametrize("d,R,L_build,visited", [(200, 64, 128, False), (300, 40, 64, False), (960, 64, 128, True), (960, 64, 64, True),
                                                 (1536, 64, 100, True)])
def test_builds_equal_the_general_kernel(jx, d, R, L_build, visited):
    n = 8000
    for x in (random_data(n, d, np.float32, 41), _mixed(n, d, 42, extremes=False)):
        adj = []
        for flags in (0, jx.FLAG_VISITED_IDS):
            g = jx.Index(d, jx.F32, R, L_build, 1.2, capacity=n, max_batch=n, flags=flags,
                         cand_mode=jx.CAND_VISITED if visited else jx.CAND_FRONTIER)
            g.insert(dev(x))
            adj.append(g.export_graph()[0])
        assert torch.equal(adj[0], adj[1])


def test_copies_follow_imports_inserts_and_compaction(jx):
    d, n = 300, 9000
    x, q = random_data(n, d, np.float32, 51), dev(random_data(700, d, np.float32, 52))
    g = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n, max_batch=n)
    g.insert(dev(x[:6000]))
    h = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n, max_batch=n)
    h.import_graph(dev(x[:6000]), g.export_graph()[0], g.size()[1])
    _same(jx, h, q, 64)
    h.insert(dev(x[6000:]))
    _same(jx, h, q, 64)
    h.delete(dev(np.random.default_rng(5).permutation(n)[:3000].astype(np.int32)))
    _same(jx, h, q, 64)
    h.consolidate()
    h.compact()
    _same(jx, h, q, 64)


@pytest.mark.parametrize("d,n", [(288, 9000), (512, 9000), (960, 5000), (1536, 3000)])
def test_rerank_reads_what_may_be_among_the_first(jx, d, n):
    """The re-rank that reads byte copies first returns, bit for bit, what the one on whole vectors returns, which keeps batches
    of fewer than 2,048 queries with at most 48 candidates; with more candidates its ids are those of 64-bit distances.  Copies
    of one row and rows without a byte copy are among the candidates."""
    x = random_data(n, d, np.float32, 61)
    y = _mixed(n, d, 61, extremes=False)
    y[np.random.default_rng(64).permutation(n)[:9]] *= np.float32(1e17)
    q = dev(np.concatenate([random_data(1400, d, np.float32, 62), _mixed(700, d, 63)]))
    g = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n, max_batch=n, quant_bits=1)
    g.insert(dev(x))
    adj, entry = g.export_graph()[0], g.size()[1]
    rot = np.linalg.qr(np.random.default_rng(9).standard_normal((d, d)))[0].astype(np.float32)
    for z in (x, y):
        g.import_graph(dev(z), adj, entry)
        g.quantize(1, dev(rot), dev(x.mean(0, dtype=np.float64).astype(np.float32)), query_bits=4)
        for k, L, rr in ((1, 8, 3), (3, 40, 16), (10, 64, 32), (13, 64, 40), (16, 64, 48)):
            ids, dist = g.search(q, k, L, mode=jx.RABITQ, rerank=rr)
            few = [g.search(part.contiguous(), k, L, mode=jx.RABITQ, rerank=rr) for part in q.split(700)]
            assert torch.equal(ids, torch.cat([f[0] for f in few])), (k, rr)
            assert torch.equal(dist.view(torch.int32), torch.cat([f[1] for f in few]).view(torch.int32)), (k, rr)
    g.import_graph(dev(x), adj, entry)
    g.quantize(1, dev(rot), query_bits=4)
    x64, q = dev(x).double(), q[:300].contiguous()
    for k, rr in ((10, 49), (21, 64)):
        cand = g.search(q, rr, 70, mode=jx.RABITQ)[0].long()
        far = torch.stack([(x64[c] - v.double()).square().sum(1) for c, v in zip(cand, q)])
        want = cand.gather(1, far.sort(dim=1)[1][:, :k]).to(torch.int32)
        assert torch.equal(g.search(q, k, 70, mode=jx.RABITQ, rerank=rr)[0], want), (k, rr)


def test_counters_count_what_is_read(jx):
    """dist_evals lies between an exact visited set's count and that of no filter; vec_bytes and rerank_bytes are those of the
    vectors that were read and of the byte copies, not of every neighbour and candidate.  Integer data: the oracle's walk."""
    d, n, L, nq = 960, 5000, 64, 4200
    rng = np.random.default_rng(71)
    c = rng.integers(-20, 21, (8, d))
    x, q = ((c[rng.integers(0, 8, m)] + rng.integers(-12, 13, (m, d))).astype(np.float32) for m in (n, nq))
    g = jx.Index(d, jx.F32, 48, L, 1.2, capacity=n, max_batch=n, quant_bits=1)
    g.insert(dev(x))
    ref = oracle.Index(d, np.float32, 48, L, 1.2, n)
    ref.set_graph(x, u32(g.export_graph()[0]), g.size()[1])
    few = q[:600]
    st = g.search(dev(few), 10, L, stats=True)[2]
    assert st["beam_kernel"].startswith("beam_search_sketch_kernel<")
    exact, none = ref.search(few, 10, L), ref.search(few, 10, L, filter=oracle.FILTER_NONE)
    assert st["hops"] == exact["hops"]
    assert exact["evals"] <= st["dist_evals"] <= none["evals"]
    copy = d + 16  # bytes
    # most were looked at through their copies: not those before the frontier was full, nor the few new ones of an expansion
    assert 600 * L * 4 * d + (st["dist_evals"] - 600 * (L + 48)) * copy <= st["vec_bytes"] <= 0.9 * st["dist_evals"] * 4 * d
    g.quantize(1, dev(np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32)), query_bits=4)
    st = g.search(dev(q), 10, L, mode=jx.RABITQ, rerank=40, stats=True)[2]
    assert nq * (10 * 4 * d + 40 * copy) <= st["rerank_bytes"] <= nq * (30 * 4 * d + 40 * copy)
    st = g.search(dev(few), 10, L, mode=jx.RABITQ, rerank=40, stats=True)[2]
    assert st["rerank_bytes"] == 600 * 40 * 4 * d


@pytest.mark.parametrize("d,L", [(132, 128), (200, 65), (256, 100)])
def test_short_vectors_forget_no_more_than_without_copies(jx, d, L):
    """The visited table of a full batch is the one that searches of whole vectors have (another lane mapping asks for these)."""
    n = 10_000
    x, q = (dev(np.rint(4 * random_data(m, d, np.float32, s))) for m, s in ((n, 83), (4200, 84)))  # exact in every order of sums
    g = jx.Index(d, jx.F32, 64, 64, 1.2, capacity=n, max_batch=n)
    g.insert(x)
    ids0, dist0, st0 = g.search(q, 10, L, stats=True)
    g.set_flags(jx.FLAG_LANES_WIDE)
    ids, dist, st = g.search(q, 10, L, stats=True)
    assert st0["beam_kernel"].startswith("beam_search_sketch_kernel<") and st["beam_kernel"].startswith("beam_search_kernel<")
    assert torch.equal(ids, ids0) and torch.equal(dist, dist0)
    assert (st["hops"], st["dist_evals"]) == (st0["hops"], st0["dist_evals"])


@pytest.mark.parametrize("d,L", [(960, 256), (1536, 129)])
def test_batches_that_are_all_resident_forget_no_more(jx, d, L):
    """Wide frontiers: the visited table is halved for batches of 1,793 to 2,048 queries only, which all fit beside each other then."""
    n = 6000
    x, q = (dev(np.rint(4 * random_data(m, d, np.float32, s))) for m, s in ((n, 85), (2100, 86)))  # exact in every order of sums
    g = jx.Index(d, jx.F32, 64, 64, 1.2, capacity=n, max_batch=n)
    g.insert(x)
    ids, dist, st = g.search(q, 10, L, stats=True)
    assert st["beam_kernel"].startswith("beam_search_sketch_kernel<")
    for at in (1050, 1792, 1793, 2048):
        parts = [g.search(part.contiguous(), 10, L, stats=True) for part in (q[:at], q[at:])]
        assert all(torch.equal(torch.cat([p[i] for p in parts]), (ids, dist)[i]) for i in (0, 1)), at
        assert sum(p[2]["hops"] for p in parts) == st["hops"], at
        if at == 1050:
            assert all(p[2]["beam_kernel"].startswith("beam_search_sketch_kernel<") for p in parts)
            assert sum(p[2]["dist_evals"] for p in parts) == st["dist_evals"]


@pytest.mark.parametrize("d", [200, 960])
def test_switches_of_other_kernels_leave_the_copies_in_use(jx, d):
    """Two expansions per round and half the lanes per record are no forms of these searches, twice the lanes none of vectors of
    more than 256 dimensions: such a switch changes nothing.  Those that ask for another kernel get it, as do all of them in
    the batches of teams, and the results are the same."""
    n = 20_000 if d == 200 else 5000
    x, q = (dev(np.rint(4 * random_data(m, d, np.float32, s))) for m, s in ((n, 81), (600, 82)))  # exact in every order of sums
    g = jx.Index(d, jx.F32, 64, 64, 1.2, capacity=n, max_batch=n)
    g.insert(x)
    ids0, dist0, st0 = g.search(q, 10, 64, stats=True)
    assert st0["beam_kernel"].startswith("beam_search_sketch_kernel<")
    none = (jx.FLAG_NO_PAIR, jx.FLAG_LANES_NARROW, jx.FLAG_NO_GRAM | jx.FLAG_NO_PAIR, jx.FLAG_NO_INCR_PRUNE)
    other = (jx.FLAG_VISITED_IDS, jx.FLAG_VISITED_NONE | jx.FLAG_NO_PAIR) + ((jx.FLAG_WAVES_2,) if d == 960 else ())
    for fl in none + other + (jx.FLAG_LANES_WIDE,):
        g.set_flags(fl)
        ids, dist, st = g.search(q, 10, 64, stats=True)
        kept = fl in none or (fl == jx.FLAG_LANES_WIDE and d == 960)
        assert st["beam_kernel"].startswith("beam_search_sketch_kernel<") == kept, (fl, st["beam_kernel"])
        assert torch.equal(ids, ids0) and torch.equal(dist, dist0) and st["hops"] == st0["hops"], fl
        if fl in none:
            assert st["dist_evals"] == st0["dist_evals"], fl
            st = g.search(q[:64], 10, 64, stats=True)[2]
            assert st["beam_kernel"].startswith("beam_search_ahead_kernel<" if not fl & (jx.FLAG_NO_PAIR | jx.FLAG_LANES_NARROW) else "beam_search_kernel<"), fl


@pytest.mark.parametrize("d", [960, 1536])
def test_insertion_of_expansion_lists_reads_copies_under_switches(jx, d):
    """Expansion lists have one kernel per visited table: graphs built under the other switches are the same."""
    n = 6000
    x = dev(random_data(n, d, np.float32, 91))
    adj = []
    for flags in (0, jx.FLAG_NO_PAIR, jx.FLAG_TILED_LOADS, jx.FLAG_WAVES_2, jx.FLAG_VISITED_IDS):
        g = jx.Index(d, jx.F32, 64, 64, 1.2, capacity=n, max_batch=n, flags=flags, cand_mode=jx.CAND_VISITED)
        g.insert(x)
        adj.append(g.export_graph()[0])
    assert all(torch.equal(a, adj[0]) for a in adj)


def test_arenas_without_room_for_copies(jx):
    """An arena that lacks the bytes of the byte copies, and no others, is accepted: whole vectors are read and the results are the
    same."""
    d, n = 960, 6000
    x, q = dev(random_data(n, d, np.float32, 101)), dev(random_data(700, d, np.float32, 102))
    rot = dev(np.linalg.qr(np.random.default_rng(9).standard_normal((d, d)))[0].astype(np.float32))

    def index(lean):
        kw = dict(capacity=n, max_batch=n, quant_bits=1, cand_mode=jx.CAND_VISITED)
        full = jx.Index(d, jx.F32, 64, 64, 1.2, **kw)
        copies = n * 1024
        if lean == 0:
            return full
        size = full.arena.numel() - copies + (0 if lean == 1 else copies - 256)
        full.close()
        with pytest.raises(jx.JxError) as e:
            jx.Index(d, jx.F32, 64, 64, 1.2, arena_bytes=full.arena.numel() - copies - 256, **kw)
        assert e.value.code == -2
        return jx.Index(d, jx.F32, 64, 64, 1.2, arena_bytes=size, **kw)

    out = []
    for lean in (0, 1, 2):
        g = index(lean)
        g.insert(x[:5000])
        g.insert(x[5000:])
        g.delete(torch.arange(0, n, 7, dtype=torch.int32, device="cuda"))
        g.consolidate()
        g.compact()
        ids, dist, st = g.search(q, 10, 64, stats=True)
        assert st["beam_kernel"].startswith("beam_search_sketch_kernel<" if lean == 0 else "beam_search_kernel<")
        g.quantize(1, rot, query_bits=4)
        many = q.repeat(6, 1)  # 4,200 queries: the re-rank that reads copies
        out.append((g.export_graph()[0], ids, dist, *g.search(many, 10, 64, mode=jx.RABITQ, rerank=40)))
    assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(o, out[0]))


@pytest.mark.parametrize("d", [200, 960])
@pytest.mark.parametrize("kind,useful", [("near", True), ("far", False), ("shifted", False), ("odd first rows", True), ("one vector", True)])
def test_sets_of_which_copies_say_nothing_do_without(jx, d, kind, useful):
    """Far from the origin, or with an offset per coordinate, every neighbour is kept: whole vectors are read.  Decided by the first
    insert and by an import, whatever a few rows are; the results are those of an index without room for copies."""
    n = 8000
    x, q = random_data(n + 500, d, np.float32, 111), random_data(600, d, np.float32, 112)
    move = {"far": np.float32(200), "shifted": 100 * np.random.default_rng(3).standard_normal(d).astype(np.float32)}.get(kind, np.float32(0))
    x, q = x + move, q + move
    if kind == "odd first rows":
        x[:30] += 1000
        x[30], x[31], x[32] = 1e20, -1e18, 1e18
    if kind == "one vector":
        x[:] = x[0]
    x, q = dev(x), dev(q)
    copies = (n + 500) * ((d + 15) // 16 * 16 + 16 + 63 >> 6 << 6)

    def searched(g):
        ids, dist, st = g.search(q, 10, 64, stats=True)
        return st["beam_kernel"].startswith("beam_search_sketch_kernel<"), ids, dist.view(torch.int32)

    g = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n + 500, max_batch=n)
    lean = jx.Index(d, jx.F32, 48, 64, 1.2, capacity=n + 500, max_batch=n, arena_bytes=g.arena.numel() - (copies + 255 >> 8 << 8))
    for part in (x[:n], x[n:]):
        out = []
        for ix in (g, lean):
            ix.insert(part)
            out.append((ix.export_graph()[0], *searched(ix)))
        assert out[0][1] == useful and not out[1][1]
        assert all(torch.equal(out[0][i], out[1][i]) for i in (0, 2, 3))
    adj, entry = g.export_graph()[0], g.size()[1]
    for moved, use in ((x, useful), (dev(random_data(n + 500, d, np.float32, 113)), True), (x, useful)):
        for ix in (g, lean):
            ix.import_graph(moved, adj, entry)
        a, b = searched(g), searched(lean)
        assert a[0] == use and all(torch.equal(a[i], b[i]) for i in (1, 2))


@pytest.mark.parametrize("d,bits", [(288, 4), (512, 2), (960, 4), (1536, 1)])
@pytest.mark.parametrize("kind,spread", [("clusters", True), ("powers", False)])
def test_rerank_reads_copies_where_the_estimates_are_spread(jx, d, bits, kind, spread):
    """Candidates whose estimates lie farther apart than the bounds are wide are left out by their copies; of others the vectors are
    read at once.  Either way the result is that of an index without copies, bit for bit."""
    n, nq = 6000, 4500
    rng = np.random.default_rng(d)
    if kind == "clusters":  # a decaying spectrum around many centres: neighbours at very different distances
        c = rng.standard_normal((400, d)) * 1.3
        mix = rng.standard_normal((d, d)) * np.arange(1, d + 1)[:, None] ** -1.0
        make = lambda m: (c[rng.integers(0, 400, m)] + rng.standard_normal((m, d)) @ mix * 0.7).astype(np.float32)
    else:
        make = lambda m: (rng.standard_normal((m, d)) ** 5).astype(np.float32)
    x, q = dev(make(n)), dev(make(nq))
    rot = dev(np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32))
    kw = dict(capacity=n, max_batch=n, quant_bits=bits)
    g = jx.Index(d, jx.F32, 48, 64, 1.2, **kw)
    g.insert(x)
    stride = (d + 15) // 16 * 16 + 16 + 63 >> 6 << 6
    lean = jx.Index(d, jx.F32, 48, 64, 1.2, arena_bytes=g.arena.numel() - (n * stride + 255 >> 8 << 8), **kw)
    lean.import_graph(x, g.export_graph()[0], g.size()[1])
    read = []
    for ix in (g, lean):
        ix.quantize(bits, rot, query_bits=4)
    for k, rr in ((10, 40), (1, 3), (13, 40), (16, 48), (10, 64), (21, 64)):
        out = [ix.search(q, k, 64, mode=jx.RABITQ, rerank=rr, stats=True) for ix in (g, lean)]
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32)), (k, rr)
        assert out[1][2]["rerank_bytes"] == rr * nq * 4 * d
        read.append(out[0][2]["rerank_bytes"] / out[1][2]["rerank_bytes"])
    # A query that takes copies reads all m of them and k vectors at least.  Where the estimates are close fewer than half of the
    # queries do, with a third of the candidates asked for
    least = lambda k, m: 1 - 0.5 * (1 - k / m - stride / (4 * d))
    assert (min(read[0], read[4]) < 0.8) if spread else (least(13, 40) < read[2] <= 1 and least(21, 64) < read[5] <= 1), read
