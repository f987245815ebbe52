"""Measured cases: what a program that uses this library has it do, through jx.py.

Six kinds of pass, each over the sizes at which it is used in earnest:

  search    beamSearch on stored vectors (uint8, float32, binary16), from one query to a 10,000-query batch
  codes     beamSearch on RaBitQ codes of 1, 2, 4 or 8 bits with exact re-rank
  build     an index made from nothing and filled with one insert call
  update    a stored graph taken in, then a stream of insert calls
  delete    a stored graph taken in, vertices deleted, the graph consolidated and compacted
  quantize  rotation and encoding of a whole base set, codes read back
  knn       exhaustive k nearest neighbours, the ground truth of every recall figure

Inputs are Gaussian mixtures with a decaying spectrum, as real descriptor sets have, drawn on the GPU from the seed.
"""
import math

import torch

from paper_2601_07048_amd import jx

TYPES = {"u8": torch.uint8, "f32": torch.float32, "f16": torch.float16}
KINDS = {"u8": jx.U8, "f32": jx.F32, "f16": jx.F16}
SIZES = {"u8": 1, "f32": 4, "f16": 2}


def listed():
    return [
        # one user's query against a served index: latency
        _search("search_u8_one_query", "u8", 200_000, 128, 64, 128, nq=1, L=32),
        # the headline: a full batch at the beam width that gives recall@10 >= 0.95
        _search("search_u8_batch", "u8", 1_000_000, 128, 64, 128, nq=10_000, L=16),
        # an ordinary float index and an ordinary batch
        _search("search_f32_1000_queries", "f32", 10_000, 128, 32, 64, nq=1_000, L=32),
        # 960-dimensional float descriptors, searched on 4-bit codes, 40 candidates re-ranked
        _codes("search_4bit_d960", "f32", 100_000, 960, bits=4, qbits=8, nq=10_000, L=128),
        # 1536-dimensional text embeddings, searched on 1-bit codes
        _codes("search_1bit_d1536", "f32", 50_000, 1536, bits=1, qbits=4, nq=5_000, L=192),
        # an index built in one call, uint8
        _build("build_u8", "u8", 200_000, 128, 64, 128),
        # the same of 960-dimensional floats
        _build("build_f32_d960", "f32", 20_000, 960, 64, 128),
        # online updates: a stored index, then small batches as they arrive
        dict(name="update_u8_small_batches", path="update", dtype="u8", n=50_000, dim=128, R=64, L_build=128, visited=True, batch=32, calls=16),
        # a tenth of an index deleted, repaired and compacted
        dict(name="delete_u8_tenth", path="delete", dtype="u8", n=200_000, dim=128, R=64, L_build=128, visited=True, drop=20_000),
        # codes of a whole base set
        dict(name="quantize_4bit_d960", path="quantize", dtype="f32", n=50_000, dim=960, bits=4, qbits=8),
        # ground truth for a recall figure: uint8, the full query batch
        dict(name="knn_u8_10000_queries", path="knn", dtype="u8", n=1_000_000, dim=128, nq=10_000, k=10, static=True),
        # ground truth on floats, an odd number of points, a long list of neighbours
        dict(name="knn_f32_d960_k100", path="knn", dtype="f32", n=100_003, dim=960, nq=1_000, k=100, static=False),
    ]


def _search(name, dtype, n, dim, R, L_build, nq, L):
    return dict(name=name, path="search", dtype=dtype, n=n, dim=dim, R=R, L_build=L_build, visited=dtype != "f16", nq=nq, k=min(10, L), L=L)


def _codes(name, dtype, n, dim, bits, qbits, nq, L):
    return dict(name=name, path="codes", dtype=dtype, n=n, dim=dim, R=64, L_build=128, visited=_visited(dtype, dim, 128), bits=bits, qbits=qbits,
                nq=nq, k=10, L=L, rerank=min(40, L))


def _build(name, dtype, n, dim, R, L_build):
    return dict(name=name, path="build", dtype=dtype, n=n, dim=dim, R=R, L_build=L_build, visited=_visited(dtype, dim, L_build))


def _visited(dtype, dim, L_build):
    """Whether expansion lists are offered as insertion candidates (see JX_CAND_VISITED)."""
    size = dim * SIZES[dtype]
    return L_build <= 128 and ((dtype == "u8" and size <= 128) or (dtype == "f32" and (size <= 512 or 2048 < size <= 6144)))


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["search", "search", "search", "codes", "codes", "build", "build", "update", "update", "delete", "quantize", "knn", "knn"])
    dtype = rng.choice(["u8", "u8", "f32", "f32", "f16"])
    if path == "search":
        dim = {"u8": rng.choice([96, 128, 128, 256]), "f32": rng.choice([96, 128, 200, 960]), "f16": rng.choice([96, 128, 960])}[dtype]
        n = log(5_000, 300_000 if dim <= 256 else 30_000)
        L = log(10, 256)
        L_build = rng.choice([64, 96, 128])
        nq = log(1, 10_000 if dim <= 256 else 2_000)
        return dict(path=path, dtype=dtype, n=n, dim=dim, R=rng.choice([32, 48, 64]), L_build=L_build, visited=_visited(dtype, dim, L_build), nq=nq, k=min(10, L), L=L)
    if path == "codes":
        dtype = rng.choice(["f32", "f32", "f16", "u8"])
        dim = {"f32": rng.choice([128, 960, 1536]), "f16": rng.choice([960, 1536]), "u8": 128}[dtype]
        L = log(40, 256)
        return dict(path=path, dtype=dtype, n=log(5_000, 50_000), dim=dim, R=64, L_build=128, visited=_visited(dtype, dim, 128), bits=rng.choice([1, 1, 2, 4, 4, 8]),
                    qbits=rng.choice([4, 8]), nq=log(1, 5_000), k=10, L=L, rerank=min(40, L))
    if path == "build":
        dim = {"u8": rng.choice([96, 128, 128, 256]), "f32": rng.choice([96, 128, 960]), "f16": rng.choice([128, 960])}[dtype]
        n = log(2_000, 200_000 if dtype == "u8" else 60_000 if dim <= 256 else 20_000)
        L_build = rng.choice([64, 96, 128])
        return dict(path=path, dtype=dtype, n=n, dim=dim, R=rng.choice([32, 48, 64]), L_build=L_build, visited=rng.random() < 0.7 and _visited(dtype, dim, L_build))
    if path == "update":
        dim = {"u8": 128, "f32": rng.choice([96, 128]), "f16": 128}[dtype]
        n = log(5_000, 100_000)
        batch = log(1, n // 10)
        calls = max(1, min(16, 20_000 // batch))
        return dict(path=path, dtype=dtype, n=n, dim=dim, R=rng.choice([32, 64]), L_build=128, visited=_visited(dtype, dim, 128), batch=batch, calls=calls)
    if path == "delete":
        dim = {"u8": 128, "f32": rng.choice([96, 128]), "f16": 128}[dtype]
        n = log(5_000, 200_000 if dtype == "u8" else 50_000)
        return dict(path=path, dtype=dtype, n=n, dim=dim, R=rng.choice([32, 64]), L_build=128, visited=_visited(dtype, dim, 128), drop=max(1, int(n * rng.uniform(0.005, 0.1))))
    if path == "quantize":
        dim = {"u8": 128, "f32": rng.choice([128, 960, 1536]), "f16": 960}[dtype]
        bits = rng.choice([1, 2, 4, 4, 8])
        return dict(path=path, dtype=dtype, n=log(3_000, 50_000), dim=dim if bits != 4 or dim <= 960 else 960, bits=bits, qbits=rng.choice([4, 8]))
    dim = {"u8": rng.choice([96, 128, 256]), "f32": rng.choice([96, 128, 200, 960]), "f16": rng.choice([128, 960])}[dtype]
    k = rng.choice([1, 10, 10, 50, 100])
    most = {"u8": 2e12, "f32": 1e11, "f16": 2e11}[dtype]
    nq = log(1, 10_000)
    n = log(2_000, max(2_001, min(1_000_000 if dim <= 256 else 200_000, int(most / dim / nq))))
    return dict(path=path, dtype=dtype, n=n, dim=dim, nq=nq, k=k, static=nq * k <= 32_768)


# ------------------------------------------------------------------ inputs


def _points(gen, n, dim, dtype, mixture):
    """n rows of a mixture; unit-variance noise with a decaying spectrum around 256 centres."""
    centres, mix = mixture
    out = torch.empty((n, dim), dtype=TYPES[dtype], device="cuda")
    for i in range(0, n, 131_072):
        m = min(131_072, n - i)
        which = torch.randint(0, centres.shape[0], (m,), device="cuda", generator=gen)
        z = torch.randn((m, dim), device="cuda", generator=gen)
        x = centres[which] + z @ mix
        out[i:i + m] = (64 + 18 * x).round_().clamp_(0, 255).to(torch.uint8) if dtype == "u8" else x.to(TYPES[dtype])
    return out


def _mixture(gen, dim):
    spectrum = torch.arange(1, dim + 1, device="cuda", dtype=torch.float32).pow(-1.25)
    spectrum *= dim / spectrum.sum()
    mix = torch.randn((dim, dim), device="cuda", generator=gen) * (spectrum.sqrt() / math.sqrt(dim))[:, None]
    return 1.3 * torch.randn((256, dim), device="cuda", generator=gen), mix


def _rotation(seed, dim):
    """A random orthogonal matrix, the same bits on every run: a product of reflections in 64 bits."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 3)
    p = torch.diag(torch.randint(0, 2, (dim,), device="cuda", generator=gen).double() * 2 - 1)
    v = torch.randn((16, 4, dim), device="cuda", generator=gen, dtype=torch.float64)
    v /= v.norm(dim=2, keepdim=True)
    for block in v:  # dense reflections, then a stride through the coordinates
        for u in block:
            p -= 2 * torch.outer(p @ u, u)
        p = p[:, torch.randperm(dim, device="cuda", generator=gen)]
    return p.float().contiguous()


def _inputs(case, seed):
    """(base, further points or queries) of a case."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    mixture = _mixture(gen, case["dim"])
    base = _points(gen, case["n"], case["dim"], case["dtype"], mixture)
    more = case["nq"] if "nq" in case else case.get("batch", 0) * case.get("calls", 0)
    return base, _points(gen, more, case["dim"], case["dtype"], mixture)


def _index(case, n, max_batch, bits=0):
    return jx.Index(case["dim"], KINDS[case["dtype"]], case.get("R", 32), case.get("L_build", 64), 1.2, capacity=n, max_batch=max_batch, quant_bits=bits,
                    cand_mode=jx.CAND_VISITED if case.get("visited") else jx.CAND_FRONTIER)


def _batch_for(n):
    """max_batch that lets n points be inserted in one call: internal batches are a quarter of the points linked."""
    return max(n // 4 + 1, 1024)


def _bare(index, base):
    """Vectors without a graph: for calls that only read vectors."""
    index.import_graph(base, torch.full((base.shape[0], index.R), -1, dtype=torch.int32, device="cuda"), 0)
    return index


def prepare(case, seed):
    base, more = _inputs(case, seed)
    path, n = case["path"], case["n"]
    state = {"case": case, "base": base, "more": more}
    if path in ("search", "codes"):
        index = _index(case, n, max(_batch_for(n), case["nq"]), case.get("bits", 0))
        index.insert(base)
        if path == "codes":
            index.quantize(case["bits"], _rotation(seed, case["dim"]), query_bits=case["qbits"])
        state["index"] = index
    elif path in ("update", "delete"):
        index = _index(case, n, _batch_for(n))
        index.insert(base)
        state["adj"], state["entry"] = index.export_graph()[0], index.size()[1]
        index.close()
        total = n + more.shape[0]
        state["index"] = _index(case, total, _batch_for(total))
        if path == "update":
            state["more"] = [b.contiguous() for b in more.split(case["batch"])]
        else:
            gen = torch.Generator(device="cuda").manual_seed(seed + 1)
            state["drop"] = torch.randperm(n, device="cuda", generator=gen)[:case["drop"]].to(torch.int32)
    elif path == "quantize":
        state["rotation"] = _rotation(seed, case["dim"])
        state["index"] = _bare(_index(case, n, 4096, case["bits"]), base)
    elif path == "knn" and not case["static"]:
        state["index"] = _bare(_index(case, n, max(4096, case["nq"])), base)
    return state


def run(state):
    case = state["case"]
    path, index = case["path"], state.get("index")
    if path == "search":
        return index.search(state["more"], case["k"], case["L"])
    if path == "codes":
        return index.search(state["more"], case["k"], case["L"], mode=jx.RABITQ, rerank=case["rerank"])
    if path == "build":
        index = _index(case, case["n"], _batch_for(case["n"]))
        index.insert(state["base"])
        return index.export_graph()
    if path == "update":
        index.import_graph(state["base"], state["adj"], state["entry"])
        for batch in state["more"]:
            index.insert(batch)
        return index.export_graph()
    if path == "delete":
        index.import_graph(state["base"], state["adj"], state["entry"])
        index.delete(state["drop"])
        index.consolidate()
        renamed = index.compact()
        return (*index.export_graph(), renamed)
    if path == "quantize":
        index.quantize(case["bits"], state["rotation"], query_bits=case["qbits"])
        return index.export_codes()
    if case["static"]:
        return jx.bruteforce_static(state["base"], state["more"], case["k"])
    return index.bruteforce(state["more"], case["k"])


# ------------------------------------------------------------------ what a pass cannot do without


def work(case):
    n, dim, size = case["n"], case["dim"], case["dim"] * SIZES[case["dtype"]]
    path = case["path"]
    if path in ("search", "codes"):
        # every entry of the final beam is expanded: its row is read and about half of its neighbours are new
        hops = case["nq"] * min(case["L"], n)
        record = size if path == "search" else dim * case["bits"] // 8 + 12
        index = n * (4 * case["R"] + record)
        b = min(hops * (4 * case["R"] + case["R"] // 2 * record), index) + case["nq"] * (size + 8 * case["k"])
        f = hops * (case["R"] // 2) * 2.0 * dim
        if path == "codes":
            b += 4 * dim * dim + min(case["nq"] * case["rerank"], n) * size
            f += 2.0 * case["nq"] * dim * dim + 3.0 * case["nq"] * case["rerank"] * dim
        return {"bytes": b, "flops": f}
    if path in ("build", "update"):
        new = n if path == "build" else case["batch"] * case["calls"]
        # the search of each new point, and one row's pairs tested for it
        f = new * (case["L_build"] * (case["R"] // 2) + case["R"] * case["R"] / 2) * 2.0 * dim
        return {"bytes": (n + (new if path == "update" else 0)) * (size + 4 * case["R"]), "flops": f}
    if path == "delete":
        touched = min(n, case["drop"] * case["R"] / 2)
        return {"bytes": 2 * n * (size + 4 * case["R"]), "flops": touched * case["R"] * case["R"] / 2 * 2.0 * dim}
    if path == "quantize":
        return {"bytes": n * (size + dim * case["bits"] // 8 + 8) + 4 * dim * dim, "flops": 2.0 * n * dim * dim}
    return {"bytes": (n + case["nq"]) * size + case["nq"] * case["k"] * 8, "flops": 2.0 * n * case["nq"] * dim}


# ------------------------------------------------------------------ how far outputs may be off


def tolerance(case):
    """About four times what the path shows when its inputs move by half a unit in the last place, or against 64 bits."""
    path, dtype = case["path"], case["dtype"]
    if dtype == "u8" and path not in ("codes", "quantize"):
        return "exact"  # integers throughout
    if path in ("build", "update", "delete"):
        return {"differ": 1e-3}  # a near-tie of the pruning rule changes a row, and the searches that cross it
    if path == "quantize":
        return {"rel": 2e-6, "max": 1e-5, "differ": 2e-5}
    if path == "codes":  # the distances are those of the exact re-rank
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    # squared distances in 32 bits; binary16 rows take the form |a|^2 - 2ab + |b|^2
    return {"rel": 7e-6, "max": 3e-5, "differ": 1e-3} if dtype == "f16" else {"rel": 2e-6, "max": 6e-6, "differ": 1e-3}


# ------------------------------------------------------------------ the same in 64 bits


def exact(case, seed):
    if case["path"] == "knn":
        return _exact_knn(case, seed)
    if case["path"] == "quantize":
        return _exact_codes(case, seed)
    return None  # results on a graph that the library itself has built


def _exact_knn(case, seed):
    base, queries = _inputs(case, seed)
    k = min(case["k"], case["n"])
    ids = torch.full((case["nq"], case["k"]), -1, dtype=torch.int64, device="cuda")
    dist = torch.full((case["nq"], case["k"]), math.inf, dtype=torch.float64, device="cuda")
    q = queries.double()
    for i in range(0, case["nq"], 1024):
        part = q[i:i + 1024]
        best_d = best_i = None
        for j in range(0, case["n"], 131_072):
            b = base[j:j + 131_072].double()
            d = (b * b).sum(1)[None, :] - 2 * (part @ b.T)
            near_d, near = d.topk(min(k + 8, d.shape[1]), dim=1, largest=False)
            near = near + j
            best_d, best_i = (near_d, near) if best_d is None else (torch.cat([best_d, near_d], 1), torch.cat([best_i, near], 1))
        few = best_d.topk(min(k + 8, best_d.shape[1]), dim=1, largest=False)[1]
        best_i = best_i.gather(1, few).sort(1)[0]  # ties go to the smaller id
        d = torch.stack([(base[row].double() - one).square().sum(1) for row, one in zip(best_i, part)])
        order = d.sort(dim=1, stable=True)[1][:, :k]
        ids[i:i + part.shape[0], :k] = best_i.gather(1, order)
        dist[i:i + part.shape[0], :k] = d.gather(1, order)
    return None, dist


def _exact_codes(case, seed):
    """Squared norm and rescaling factor of every centred row, and the centroid; the codes themselves have no 64-bit form."""
    base = _inputs(case, seed)[0].double()
    centroid = base.mean(0)
    bits, half = case["bits"], 1 << (case["bits"] - 1)
    rotation = _rotation(seed, case["dim"]).double()
    meta = torch.empty((case["n"], 2), dtype=torch.float64, device="cuda")
    dim, levels = case["dim"], half - 1
    sweep = bits in (2, 4) and dim * levels <= 8192
    for i in range(0, case["n"], 2048):
        r = (base[i:i + 2048] - centroid.float().double()) @ rotation.T
        a = r.abs()
        if bits == 1:
            level = torch.zeros_like(a)
        elif not sweep:
            level = (a * ((half - 0.5) / a.amax(1, keepdim=True))).floor().clamp(max=levels)
        else:  # the grid scale with the largest cosine, over all scales at which a coordinate steps to its next level
            steps = torch.arange(1, half, device="cuda", dtype=torch.float64)
            t, order = (steps[None, None, :] / a[:, :, None]).flatten(1).sort(1)
            j = order % levels + 1
            up = a.gather(1, order // levels)
            cosine = (0.5 * a.sum(1, keepdim=True) + up.cumsum(1)) / (0.25 * dim + (2.0 * j).cumsum(1)).sqrt()
            best = t.gather(1, cosine.argmax(1, keepdim=True))
            level = (steps[None, None, :] / a[:, :, None] <= best[:, :, None]).sum(2).double()
        norm = a.square().sum(1)
        meta[i:i + 2048, 0] = norm
        meta[i:i + 2048, 1] = -2 * norm / ((level + 0.5) * a).sum(1)
    return None, meta, centroid
