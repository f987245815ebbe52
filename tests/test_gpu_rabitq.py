"""GPU parity of the RaBitQ pipeline (rotation GEMM, encoder, query records,
estimated-distance beamSearch, exact re-rank) vs the CPU oracle, stage by stage
with injected inputs and end to end."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_07048_amd import datagen
from gpu_common import dev, u32, oracle_index, gpu_index_from_oracle, jx_dtype, random_data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jx():
    from paper_2601_07048_amd import jx as m
    return m


def _clustered(n, d, seed, comps=8):
    rng = np.random.default_rng(seed)
    cent = rng.standard_normal((comps, d)) * 0.5
    lam = np.sqrt(np.arange(1, d + 1, dtype=np.float64) ** -0.5)
    x = cent[rng.integers(0, comps, n)] + 0.3 * rng.standard_normal((n, d)) * lam
    return x.astype(np.float32)


def _signed_permutation(d, seed):
    rng = np.random.default_rng(seed)
    P = np.zeros((d, d), np.float32)
    P[np.arange(d), rng.permutation(d)] = rng.choice([-1.0, 1.0], d)
    return P


@pytest.mark.parametrize("d,n", [(96, 300), (960, 257), (1536, 130)])
def test_rotation_gemm(jx, d, n):
    """(in - c) P^T on the matrix cores vs the double-precision rotation."""
    rng = np.random.default_rng(d)
    x = _clustered(n, d, d)
    P = datagen.random_orthogonal(d, d + 1).astype(np.float32)
    c = x.astype(np.float64).mean(0).astype(np.float32)
    g = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=n, quant_bits=1)
    g.import_graph(dev(x), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(1, dev(P), dev(c))
    got = g.rotate(dev(x)).cpu().numpy().astype(np.float64)
    _, want = oracle.rabitq_rotate(x, P, c)
    scale = np.abs(want).max()
    assert np.abs(got - want).max() <= 2e-6 * scale * np.sqrt(d)
    # a signed permutation with c = 0 must be reproduced exactly
    Q = _signed_permutation(d, 3)
    g.quantize(1, dev(Q), dev(np.zeros(d, np.float32)))
    got = g.rotate(dev(x)).cpu().numpy()
    assert np.array_equal(got, x @ Q.T)


@pytest.mark.parametrize("bits,d", [(1, 1536), (4, 960), (1, 96), (4, 32), (4, 1536), (1, 960), (2, 960), (2, 32), (2, 1536),
                                    (8, 96), (8, 960), (8, 1536)])
def test_encoder_on_injected_rotated_vectors(jx, bits, d):
    """Encoder stage alone: fed with the oracle's float32 rotated vectors it must
    emit the oracle's codes bit for bit (the decisions are float32 on both
    sides) and the two floats to float rounding."""
    n = 400
    r32 = (_clustered(n, d, bits * 1000 + d) * np.float32(1.7)).astype(np.float32)
    r32[3] = 0.0  # degenerate vector
    r32[5, :7] = [0.0, -0.0, 1e-30, -1e-30, 5.0, -5.0, 0.25]
    g = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=n, quant_bits=bits)
    g.import_graph(dev(r32), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(bits, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXABS)
    codes, meta = g.encode_rotated(dev(r32))
    wc, wm, _ = oracle.rabitq_encode(r32, bits, oracle.RULE_MAXABS)
    assert np.array_equal(codes.cpu().numpy(), wc)
    assert np.allclose(meta.cpu().numpy(), wm, rtol=2e-7, atol=0)
    # with P = I and c = 0 the whole quantise call is the same computation
    ec, em, cen = g.export_codes()
    assert np.array_equal(ec.cpu().numpy(), wc) and np.allclose(em.cpu().numpy(), wm, rtol=2e-7, atol=0)
    assert (cen.cpu().numpy() == 0).all()


@pytest.mark.parametrize("d", [960, 96, 1536])
def test_max_cosine_encoder_two_bit(jx, d):
    """The same sweep for 2-bit codes (one breakpoint per coordinate)."""
    n = 300
    r32 = (_clustered(n, d, 78 + d) * np.float32(2.3)).astype(np.float32)
    r32[3] = 0.0
    r32[7] = np.float32(0.5)
    r32[9, ::2] = r32[9, 1::2]
    g = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=n, quant_bits=2)
    g.import_graph(dev(r32), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(2, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXCOS)
    codes, meta = g.encode_rotated(dev(r32))
    wc, wm, _ = oracle.rabitq_encode(r32, 2, oracle.RULE_MAXCOS)
    assert np.array_equal(codes.cpu().numpy(), wc)
    assert np.allclose(meta.cpu().numpy(), wm, rtol=2e-7, atol=0)
    ec, em, _ = g.export_codes()   # through the two-plane record and back
    assert np.array_equal(ec.cpu().numpy(), wc)


@pytest.mark.parametrize("d", [960, 96, 32, 1152])
def test_max_cosine_encoder_on_injected_rotated_vectors(jx, d):
    """The "extended" 4-bit rule: the GPU sorts the grid-scale breakpoints and
    sweeps them exactly like the oracle, in double, so the codes must be equal
    (the sweep's argmax could only differ if two cosines agreed to ~1e-15)."""
    n = 300
    r32 = (_clustered(n, d, 77 + d) * np.float32(2.3)).astype(np.float32)
    r32[3] = 0.0
    r32[5, :7] = [0.0, -0.0, 1e-30, -1e-30, 5.0, -5.0, 0.25]
    r32[7] = np.float32(0.5)          # every coordinate equal: all breakpoints tie
    r32[9, ::2] = r32[9, 1::2]        # many exact ties between coordinates
    g = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=n, quant_bits=4)
    g.import_graph(dev(r32), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(4, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXCOS)
    codes, meta = g.encode_rotated(dev(r32))
    wc, wm, wcos = oracle.rabitq_encode(r32, 4, oracle.RULE_MAXCOS)
    same = (codes.cpu().numpy() == wc).all(axis=1)
    assert same.all(), np.nonzero(~same)[0][:10]
    assert np.allclose(meta.cpu().numpy(), wm, rtol=2e-7, atol=0)
    ec, em, _ = g.export_codes()
    assert np.array_equal(ec.cpu().numpy(), wc)
    # and it is a better code than max-abs scaling
    _, _, cos_abs = oracle.rabitq_encode(r32, 4, oracle.RULE_MAXABS)
    assert (wcos >= cos_abs - 1e-12).all()


def test_max_cosine_rule_limits(jx):
    g = jx.Index(1536, jx.F32, 8, 8, 1.2, capacity=4, quant_bits=4)
    x = _clustered(4, 1536, 1)
    g.import_graph(dev(x), dev(np.full((4, 8), jx.NONE, np.uint32)), 0)
    with pytest.raises(jx.JxError):
        g.quantize(4, dev(np.eye(1536, dtype=np.float32)), rule=jx.RULE_MAXCOS)  # 7*dim breakpoints exceed the LDS sort


def _quantized_pair(jx, x, P, bits, qbits, R=24, L=48, centroid=None, inject=False, rule=1):
    ix = oracle_index(x, R, L)
    ix.quantize(bits, P, centroid=centroid, qbits=qbits, rule=rule)
    g = gpu_index_from_oracle(jx, x, ix, R, L, quant_bits=bits)
    if inject:
        codes, meta, cen = ix.codes()
        g.import_codes(bits, dev(P), dev(cen), dev(codes), dev(meta), query_bits=qbits)
    else:
        g.quantize(bits, dev(P), None if centroid is None else dev(centroid), query_bits=qbits, rule=rule)
    return ix, g


@pytest.mark.parametrize("bits,qbits,d", [(4, 8, 960), (1, 8, 1536), (4, 4, 128), (1, 4, 256), (1, 8, 96), (4, 8, 1536),
                                          (2, 4, 960), (2, 8, 96), (2, 4, 1536), (8, 8, 96), (8, 8, 960), (8, 4, 1536),
                                          # 9 to 12 code chunks with B_q = 4: four lanes x three code chunks, meta chunk apart
                                          (1, 4, 1536), (1, 4, 1280), (2, 4, 768), (1, 4, 1152)])
def test_estimated_beam_bit_exact_on_injected_codes(jx, bits, qbits, d):
    """beamSearch + estimator stage: oracle codes injected, rotation a signed
    permutation and c = 0 (so both sides see identical rotated queries).  The
    integer inner products are exact and the five float operations are ordered
    identically, so frontier ids AND estimated distances must be identical."""
    n = 1500
    x = _clustered(n, d, d + bits)
    q = _clustered(60, d, d + bits + 1)
    P = _signed_permutation(d, 5)
    ix, g = _quantized_pair(jx, x, P, bits, qbits, centroid=np.zeros(d, np.float32), inject=True)
    for L in (10, 50, 130):
        ref = ix.search(q, 1, L, mode=1, want_frontier=True)
        ids, dist, st = g.beam_frontier(dev(q), L, mode=jx.RABITQ, stats=True)
        assert np.array_equal(u32(ids), ref["F_ids"])
        assert np.array_equal(dist.cpu().numpy().astype(np.float64), ref["F_dist"])
        assert st["hops"] == ref["hops"]


@pytest.mark.parametrize("bits,d,n,rule", [(4, 960, 3000, 1), (4, 960, 3000, 0), (1, 1536, 2000, 1)])
def test_quantize_end_to_end(jx, bits, d, n, rule):
    """Whole path with a random orthogonal P and the mean as centroid.  The GPU
    rotates in float32 on the matrix cores, the oracle in double, so a code may
    differ where a coordinate sits on a rounding boundary."""
    wl = 3 if bits == 4 else 4
    x = datagen.base(wl, n)
    q = datagen.queries(wl, 2000)
    P = datagen.rotation(wl)
    ix, g = _quantized_pair(jx, x, P, bits, 8, R=32, L=64, rule=rule)
    wc, wm, wcen = ix.codes()
    gc, gm, gcen = [t.cpu().numpy() for t in g.export_codes()]
    assert np.allclose(gcen, wcen, rtol=0, atol=1e-6)
    r32, r64 = oracle.rabitq_rotate(x, P, wcen)
    U = np.stack([oracle.rabitq_unpack(wc[i], bits, d) for i in range(0, n, 7)])
    G = np.stack([oracle.rabitq_unpack(gc[i], bits, d) for i in range(0, n, 7)])
    diff = U != G
    if bits == 1:
        # codes agree except where the rotated value is within 1e-6 of zero
        assert (np.abs(r64[::7][diff]) < 1e-6).all()
    else:
        # at most one level apart, and rare (max-cosine: a different sweep optimum on a near
        # tie changes a whole vector's scale, so the bound is on vectors there)
        assert diff.mean() < (2e-3 if rule == 1 else 2e-2)
        assert (np.abs(U.astype(int) - G.astype(int))[diff] <= (1 if rule == 1 else 2)).all()
    same = ~diff.any(axis=1)
    assert np.allclose(gm[::7][same], wm[::7][same], rtol=1e-4)
    # search: estimates within 1e-4 relative where the same vertex sits at the same rank
    ref = ix.search(q, 10, 64, mode=1, want_frontier=True)
    ids, dist = g.beam_frontier(dev(q), 64, mode=jx.RABITQ)
    ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
    m = ids == ref["F_ids"]
    assert m.mean() > 0.9
    assert np.allclose(dist[m], ref["F_dist"][m], rtol=1e-3, atol=1e-3 * np.abs(ref["F_dist"]).mean())
    # The chain behind an estimate, on the GPU's own intermediate results: the oracle's query preparation fed with
    # the GPU's float32 rotation of the query, and the oracle's integer estimator on the GPU's codes, must give the
    # GPU's estimate bit for bit.  And where the oracle's own chain (double rotation) arrives at the same integer
    # query and the same code, the two estimates agree to 1e-4 relative (only lo and delta differ, by rounding).
    qs = 60
    qr_gpu = g.rotate(dev(q[:qs])).cpu().numpy()
    qr_ref, _ = oracle.rabitq_rotate(q[:qs], P, wcen)
    scale = np.abs(ref["F_dist"]).mean()
    n_bit, n_tol = 0, 0
    for i in range(qs):
        qint_g, m4_g = oracle.rabitq_query_prep(qr_gpu[i], bits, 8)
        qint_o, m4_o = oracle.rabitq_query_prep(qr_ref[i], bits, 8)
        for j in (0, 3, 17, 40, 63):
            v = int(ids[i, j])
            if v == 0xFFFFFFFF:
                continue
            e_chain = oracle.rabitq_est_int(gc[v], bits, d, gm[v, 0], gm[v, 1], qint_g, m4_g)
            assert np.float32(e_chain) == np.float32(dist[i, j]), (i, j)
            n_bit += 1
            if np.array_equal(qint_g, qint_o) and np.array_equal(gc[v], wc[v]):
                e_ref = oracle.rabitq_est_int(wc[v], bits, d, wm[v, 0], wm[v, 1], qint_o, m4_o)
                assert abs(e_ref - dist[i, j]) <= 1e-4 * abs(e_ref) + 1e-6 * scale, (i, j, e_ref, dist[i, j])
                n_tol += 1
    assert n_bit >= 4 * qs and n_tol >= qs // 2, (n_bit, n_tol)
    # re-ranked results: exact distances, recall within 0.002 of the oracle's (2,000 queries)
    gt, gd = oracle.bruteforce(x, q, 10)
    rr = ix.search(q, 10, 64, mode=1, rerank=40)
    gi, gdist, st = g.search(dev(q), 10, 64, mode=jx.RABITQ, rerank=40, stats=True)
    gi, gdist = u32(gi), gdist.cpu().numpy().astype(np.float64)
    r_gpu, r_ref = oracle.recall_at_k(gi, gt), oracle.recall_at_k(rr["ids"], gt)
    assert abs(r_gpu - r_ref) <= 0.002, (r_gpu, r_ref)
    assert st["rerank_bytes"] == 40 * len(q) * d * 4
    for i in range(0, len(q), 97):
        for j in range(10):
            assert abs(gdist[i, j] - oracle.l2sq(q[i], x[gi[i, j]])) <= 1e-4 * gdist[i, j]
        keys = list(zip(gdist[i].tolist(), gi[i].tolist()))
        assert keys == sorted(keys)


def test_rerank_stage_exact_on_injected_codes(jx):
    """Re-rank stage: with injected codes and an exact rotation the candidate
    lists are identical, so the re-ranked ids must equal the oracle's wherever
    the exact distances are not within float rounding of each other."""
    d, n = 128, 2000
    x = _clustered(n, d, 1)
    q = _clustered(80, d, 2)
    P = _signed_permutation(d, 9)
    ix, g = _quantized_pair(jx, x, P, 4, 8, centroid=np.zeros(d, np.float32), inject=True)
    for rr_n, k in ((40, 10), (64, 64), (10, 1)):
        want = ix.search(q, k, 64, mode=1, rerank=rr_n)
        ids, dist = g.search(dev(q), k, 64, mode=jx.RABITQ, rerank=rr_n)
        ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
        assert np.allclose(dist, want["dist"], rtol=1e-5)
        gaps = np.abs(np.diff(want["dist"], axis=1))
        safe = np.ones_like(ids, bool)
        tight = gaps < 1e-5 * want["dist"][:, 1:]
        safe[:, 1:] &= ~tight
        safe[:, :-1] &= ~tight
        assert np.array_equal(ids[safe], want["ids"][safe])


def test_insert_after_quantize_encodes_new_points(jx):
    d, n = 96, 1200
    x = _clustered(n, d, 4)
    P = datagen.random_orthogonal(d, 8).astype(np.float32)
    c = x[:800].astype(np.float64).mean(0).astype(np.float32)
    g = jx.Index(d, jx.F32, 16, 32, 1.2, capacity=n, max_batch=n, quant_bits=4)
    g.insert(dev(x[:800]))
    g.quantize(4, dev(P), dev(c), rule=jx.RULE_MAXABS)
    g.insert(dev(x[800:]))
    codes, meta, _ = [t.cpu().numpy() for t in g.export_codes()]
    h = jx.Index(d, jx.F32, 16, 32, 1.2, capacity=n, max_batch=n, quant_bits=4)
    h.insert(dev(x))
    h.quantize(4, dev(P), dev(c), rule=jx.RULE_MAXABS)
    c2, m2, _ = [t.cpu().numpy() for t in h.export_codes()]
    assert codes.shape == (n, d // 2) and np.array_equal(codes, c2) and np.array_equal(meta, m2)


def test_rabitq_argument_errors(jx):
    d, n = 64, 50
    x = _clustered(n, d, 1)
    g = jx.Index(d, jx.F32, 8, 16, 1.2, capacity=n, quant_bits=4)
    P = dev(np.eye(d, dtype=np.float32))
    with pytest.raises(jx.JxError):
        g.quantize(4, P)                      # empty index
    g.insert(dev(x))
    with pytest.raises(jx.JxError):
        g.quantize(1, P)                      # bits differ from quant_bits
    with pytest.raises(jx.JxError):
        g.quantize(4, P, query_bits=5)
    with pytest.raises(jx.JxError):
        g.search(dev(x[:4]), 1, 8, mode=jx.RABITQ)  # not quantised yet
    g.quantize(4, P)
    with pytest.raises(jx.JxError):
        g.search(dev(x[:4]), 5, 8, mode=jx.RABITQ, rerank=3)  # rerank < k
    with pytest.raises(jx.JxError):
        jx.Index(48, jx.U8, 8, 16, 1.2, capacity=n, quant_bits=4)  # RaBitQ needs dim % 32 == 0
    with pytest.raises(jx.JxError):
        jx.Index(d, jx.F32, 8, 16, 1.2, capacity=n, quant_bits=3)  # widths are 1, 2, 4, 8
    g8 = jx.Index(d, jx.F32, 8, 16, 1.2, capacity=n, quant_bits=8)
    g8.import_graph(dev(x), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    with pytest.raises(jx.JxError):
        g8.quantize(8, P, rule=jx.RULE_MAXCOS)  # the breakpoint sweep is offered for 2- and 4-bit codes


def test_rabitq_on_uint8_data(jx):
    """4-bit codes of uint8 vectors (the 2x compression case of Sec. 5.1).  uint8 -> float32 is exact, so an index
    on the same values held as float32 must give identical codes, and with injected oracle codes and an exact
    rotation the estimated-distance frontier equals the oracle's bit for bit; re-rank distances are exact integers."""
    n, d, R, L = 3000, 128, 32, 64
    x = random_data(n, d, np.uint8, seed=17)
    q = random_data(2000, d, np.uint8, seed=18)
    ix = oracle_index(x, R, L)
    P = datagen.random_orthogonal(d, seed=4).astype(np.float32)
    g = gpu_index_from_oracle(jx, x, ix, R, L, quant_bits=4)
    g.quantize(4, dev(P))
    gf = gpu_index_from_oracle(jx, x.astype(np.float32), ix, R, L, quant_bits=4)
    gf.quantize(4, dev(P))
    c8, m8, cen8 = [t.cpu().numpy() for t in g.export_codes()]
    cf, mf, cenf = [t.cpu().numpy() for t in gf.export_codes()]
    assert np.array_equal(c8, cf) and np.array_equal(m8, mf) and np.array_equal(cen8, cenf)
    # end to end against the oracle (its rotation is in double: recall, not bits)
    ix.quantize(4, P)
    gt = oracle.bruteforce(x, q, 10)[0]
    ids, dist = g.search(dev(q), 10, L, mode=jx.RABITQ, rerank=40)
    want = ix.search(q, 10, L, mode=1, rerank=40)
    r_g, r_o = oracle.recall_at_k(u32(ids), gt), oracle.recall_at_k(want["ids"], gt)
    assert abs(r_g - r_o) <= 0.002 and r_g > 0.6, (r_g, r_o)
    same = (u32(ids) == want["ids"]).all(axis=1)
    assert same.mean() > 0.95
    assert np.array_equal(dist.cpu().numpy().astype(np.float64)[same], want["dist"][same])  # exact integers
    # injected codes + signed permutation + zero centroid: bit-exact frontier
    Pp = _signed_permutation(d, 6)
    zero = np.zeros(d, np.float32)
    ix.quantize(4, Pp, centroid=zero)
    oc, om, _ = ix.codes()
    g.import_codes(4, dev(Pp), dev(zero), dev(oc), dev(om))
    q = q[:100]
    ref = ix.search(q, 1, 50, mode=1, want_frontier=True)
    fi, fd = g.beam_frontier(dev(q), 50, mode=jx.RABITQ)
    assert np.array_equal(u32(fi), ref["F_ids"])
    assert np.array_equal(fd.cpu().numpy().astype(np.float64), ref["F_dist"])


@pytest.mark.parametrize("bits,d,n", [(2, 960, 3000), (8, 960, 3000), (2, 1536, 2000), (8, 128, 3000)])
def test_quantize_end_to_end_other_widths(jx, bits, d, n):
    """2- and 8-bit codes, whole path (rotation on the GPU in float32, oracle in double): codes at most one level
    apart on rare coordinates, re-ranked recall within 0.002 of the oracle's (2,000 queries), estimates close where
    ranks agree."""
    wl = 3 if d == 960 else (4 if d == 1536 else 1)
    x = datagen.base(wl, n)
    q = datagen.queries(wl, 2000)
    P = datagen.rotation(wl)
    ix, g = _quantized_pair(jx, x, P, bits, 8, R=32, L=64, rule=1)
    wc, wm, wcen = ix.codes()
    gc, gm, gcen = [t.cpu().numpy() for t in g.export_codes()]
    assert gc.shape == wc.shape == (n, d * bits // 8)
    U = np.stack([oracle.rabitq_unpack(wc[i], bits, d) for i in range(0, n, 7)]).astype(int)
    G = np.stack([oracle.rabitq_unpack(gc[i], bits, d) for i in range(0, n, 7)]).astype(int)
    diff = U != G
    assert diff.mean() < (2e-3 if bits == 2 else 2e-2) and (np.abs(U - G)[diff] <= 1).all()
    gt = oracle.bruteforce(x, q, 10)[0]
    rr = ix.search(q, 10, 64, mode=1, rerank=40)
    gi, _ = g.search(dev(q), 10, 64, mode=jx.RABITQ, rerank=40)
    r_gpu, r_ref = oracle.recall_at_k(u32(gi), gt), oracle.recall_at_k(rr["ids"], gt)
    assert abs(r_gpu - r_ref) <= 0.002, (r_gpu, r_ref)
    ref = ix.search(q, 10, 64, mode=1, want_frontier=True)
    ids, dist = g.beam_frontier(dev(q), 64, mode=jx.RABITQ)
    ids, dist = u32(ids), dist.cpu().numpy().astype(np.float64)
    m = ids == ref["F_ids"]
    assert m.mean() > 0.8
    # a code that differs by one (coarse) level moves that vector's estimate; everything else agrees to rounding
    err = np.abs(dist[m] - ref["F_dist"][m]) / np.abs(ref["F_dist"]).mean()
    assert np.quantile(err, 0.98) < 1e-3 and err.max() < 0.05, (np.quantile(err, 0.98), err.max())


@pytest.mark.parametrize("dtype,bits", [(np.float32, 1), (np.float32, 4), (np.float16, 8), (np.uint8, 2)])
@pytest.mark.parametrize("d,n", [(32, 1), (96, 127), (128, 128), (160, 129), (960, 300), (960, 2945), (160, 16001)])
def test_rotation_of_every_tile_edge(jx, d, n, dtype, bits):
    """One row to just over a tile of them, dimensions that end inside one, tiles of 64 and (the last two) of 128 columns: products of three bfloat16 parts (queries, 1-bit codes)
    and the float32 form (codes of more bits) against double sums, 1e-6 of a row's norm (sums of 32 coordinates leave 2e-7)."""
    x = random_data(n, d, np.uint8 if dtype == np.uint8 else np.float32, seed=d + n).astype(dtype)
    P = datagen.random_orthogonal(d, d).astype(np.float32)
    g = jx.Index(d, jx_dtype(jx, x), 8, 16, 1.2, capacity=max(n, 16), max_batch=max(n, 1024), quant_bits=bits)
    g.insert(dev(x))
    g.quantize(bits, dev(P), query_bits=4)
    x = x.astype(np.float32)
    c = g.export_codes()[2].cpu().numpy().astype(np.float64)
    want = (x.astype(np.float64) - c) @ P.astype(np.float64).T
    norm = np.linalg.norm(want, axis=1, keepdims=True)
    for got in (g.rotate(dev(x)), g.rotate_points(dev(x.astype(dtype)))):
        assert (np.abs(got.cpu().numpy().astype(np.float64) - want) <= 1e-6 * norm + 1e-7 * np.abs(x).max()).all()


@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.uint8])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_stages_make_the_codes_of_an_index(jx, bits, dtype):
    """jx_rotate_points and jx_encode_rotated are what jx_quantize does, bit for bit.  Of two forms of the rotation that differ in the
    last bits only, some ten of these 2.9 M codes and most of the floats beside them would not agree."""
    n, d = 3_000, 960
    x = random_data(n, d, np.uint8, bits) if dtype == np.uint8 else _clustered(n, d, bits).astype(dtype)
    g = jx.Index(d, jx_dtype(jx, x), 8, 8, 1.2, capacity=n, max_batch=1024, quant_bits=bits)
    g.import_graph(dev(x), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(bits, dev(datagen.random_orthogonal(d, 5).astype(np.float32)))
    codes, meta = g.encode_rotated(g.rotate_points(dev(x)))
    want_codes, want_meta, _ = g.export_codes()
    assert torch.equal(codes, want_codes)
    assert torch.equal(meta.view(torch.int32), want_meta.view(torch.int32))


def test_rotation_of_values_that_are_hardly_finite(jx):
    """The largest float32 values round to an infinite bfloat16 part, infinities and NaN have no parts: such elements come out
    as plain float32 sums give them."""
    d = 64
    P = np.eye(d, dtype=np.float32)[::-1].copy()
    x = random_data(40, d, np.float32, seed=2)
    g = jx.Index(d, jx.F32, 8, 16, 1.2, capacity=64, max_batch=1024, quant_bits=1)
    g.insert(dev(x))
    g.quantize(1, dev(P), dev(np.zeros(d, np.float32)), query_bits=4)
    top = np.finfo(np.float32).max
    q = x[:6].copy()
    q[0, 3], q[1, 60], q[2, 5], q[3, 7], q[4, 9] = top, -top, 3.395e38, np.inf, np.nan
    got = g.rotate(dev(q)).cpu().numpy()
    assert np.array_equal(got[[0, 1, 2, 5]], q[[0, 1, 2, 5], ::-1])
    for r, at in ((3, 7), (4, 9)):  # infinity and NaN times zero: the whole row, as the float32 sums have it
        assert not np.isfinite(got[r]).any()


@pytest.mark.parametrize("bits,d", [(4, 64), (4, 256), (4, 288), (4, 512), (4, 544), (4, 1024), (4, 1056), (2, 256), (2, 544), (2, 1024), (2, 2048), (2, 2080), (2, 4096)])
def test_max_cosine_of_every_spread(jx, bits, d):
    """Where the largest cosine lies depends on how the magnitudes are spread; the encoder evaluates what bounds leave of the
    breakpoints.  Normal, heavy-tailed, few different values (ties between levels), sparse, one outlier, subnormal and huge
    magnitudes, at both sides of every number of magnitudes per thread, against the oracle's sweep over all of them."""
    rng = np.random.default_rng(d)
    base = rng.standard_normal((24, d))
    tails = base / (np.abs(rng.standard_normal((24, d))) + 1e-3)
    rows = [base, base ** 3, tails, np.round(base * 1.5), np.round(base * 6), base * (rng.random((24, d)) < 0.04), base * 1e-39, base * 1e35,
            rng.random((24, d)), np.where(rng.random((24, d)) < 2 / d, 60.0, base), np.tile(np.arange(1, 9), (24, d // 8)).astype(float)]
    r32 = np.concatenate(rows).astype(np.float32)
    g = jx.Index(d, jx.U8 if d > 1536 else jx.F32, 8, 8, 1.2, capacity=64, quant_bits=bits)
    x = np.ones((64, d), np.uint8 if d > 1536 else np.float32)
    g.import_graph(dev(x), dev(np.full((64, 8), jx.NONE, np.uint32)), 0)
    g.quantize(bits, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXCOS)
    codes, meta = g.encode_rotated(dev(r32))
    wc, wm, _ = oracle.rabitq_encode(r32, bits, oracle.RULE_MAXCOS)
    bad = np.nonzero((codes.cpu().numpy() != wc).any(axis=1))[0]
    assert bad.size == 0, (bad[:8], bad.size)
    assert np.allclose(meta.cpu().numpy(), wm, rtol=2e-7, atol=1e-45)
