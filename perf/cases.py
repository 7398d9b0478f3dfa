"""The calls whose speed matters to a user of this library, as cases a timing program can run.

A case is one pass through a public entry point of `paper_1905_06900_amd.binding` at one size: a two-pass
search over a flat code array, the same over an inverted index, encoding of vectors, and training of the
quantizers.  `listed()` names twelve of them, from a single query on a small array to the largest batch;
`draw(rng)` gives further ones of the same ranges.  Inputs are seeded synthetic data with the shapes and
distributions of the workloads in `paper_1905_06900_amd.synth`.

Codes of the encoded data sets (SIFT- and GIST-like) are drawn instead of encoded one by one: the vectors
are an isotropic Gaussian mixture, so within a component the sub-vectors, and hence the sub-codes, are
independent.  A few hundred vectors per component are encoded and every sub-code of the array is then drawn
from those of its component.
"""
from __future__ import annotations

import math

import torch

from paper_1905_06900_amd import binding, synth

DEV = "cuda:0"


def listed():
    return [
        # One query at a time on a database of a million: what an interactive caller waits for.
        {"name": "flat_zipf_1m_one_query", "op": "flat", "data": "zipf", "m": 4, "dsub": 32, "N": 1_000_000, "Q": 1, "r": 1000, "k": 100},
        # The smallest benchmark workload: 64-bit codes, a hundred queries, skewed codes (many equal distances).
        {"name": "flat_zipf_1m", "op": "flat", "data": "zipf", "m": 4, "dsub": 32, "N": 1_000_000, "Q": 100, "r": 1000, "k": 100},
        # The paper's usual candidate set of about 10 K on a million 128-d vectors, at an odd size and batch.
        {"name": "flat_sift_1m_many_candidates", "op": "flat", "data": "sift", "m": 8, "dsub": 16, "N": 1_000_003, "Q": 251, "r": 10_000, "k": 100},
        # An ordinary batch over ten million encoded vectors.
        {"name": "flat_sift_10m", "op": "flat", "data": "sift", "m": 8, "dsub": 16, "N": 10_000_000, "Q": 1000, "r": 2000, "k": 100},
        # Online serving: the few queries that arrived together against the largest flat array.
        {"name": "flat_deep_100m_few_queries", "op": "flat", "data": "deep", "m": 8, "dsub": 12, "N": 100_000_000, "Q": 16, "r": 4000, "k": 100},
        # The headline workload: the largest batch over the largest flat array.
        {"name": "flat_deep_100m", "op": "flat", "data": "deep", "m": 8, "dsub": 12, "N": 100_000_000, "Q": 4096, "r": 4000, "k": 100},
        # Long vectors: 960-d descriptors, 16 sub-quantizers.
        {"name": "flat_gist_10m", "op": "flat", "data": "gist", "m": 16, "dsub": 60, "N": 10_000_000, "Q": 512, "r": 5000, "k": 100},
        # 8-bit quantizers with 4-bit derived codebooks (one byte per sub-code), odd size and batch.
        {"name": "flat_bits_8_4", "op": "flat", "data": "bits", "m": 16, "dsub": 8, "N": 9_999_991, "Q": 333, "r": 2000, "k": 100, "bbar": 4},
        # One query through an inverted index of ten million, scanned from the codes themselves.
        {"name": "ivf_10m_one_query", "op": "ivf", "m": 8, "dsub": 16, "N": 10_000_000, "nlist": 4096, "nprobe": 16, "Q": 1, "r": 1000, "k": 100, "plane": False},
        # The billion-scale inverted index, scanned from the low-byte plane.
        {"name": "ivf_1b", "op": "ivf", "m": 8, "dsub": 16, "N": 1_000_000_000, "nlist": 65536, "nprobe": 64, "Q": 1024, "r": 1000, "k": 100, "plane": True},
        # Adding vectors to a database: encoding at PQ 8x16, odd count.
        {"name": "encode_sift_250k", "op": "encode", "data": "sift", "m": 8, "dsub": 16, "b": 16, "n": 250_007},
        # Training all quantizers of a database (k-means, same-size k-means, final order).
        {"name": "train_sift_131k", "op": "train", "m": 8, "dsub": 16, "b": 16, "bbar": 8, "n": 131_072, "iters": 2, "iters_same": 1},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; most are odd sizes that no tile divides."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choices(("flat", "ivf", "encode", "train"), weights=(7, 3, 1, 1))[0]
    if op == "flat":
        data = rng.choice(("zipf", "sift", "deep", "gist", "bits"))
        top_n = {"zipf": 4_000_000, "sift": 10_000_000, "deep": 100_000_000, "gist": 10_000_000, "bits": 10_000_000}[data]
        top_q = {"zipf": 1000, "sift": 1000, "deep": 4096, "gist": 512, "bits": 512}[data]
        case = {"op": "flat", "data": data, "m": 8, "dsub": 16, "N": _log(rng, 100_000, top_n), "Q": _log(rng, 1, top_q),
                "r": _log(rng, 500, 12_000), "k": rng.choice((1, 10, 50, 100, 100, 100))}
        if data == "zipf":
            case.update(m=4, dsub=32)
        elif data == "deep":
            case.update(dsub=12)
        elif data == "gist":
            case.update(m=16, dsub=60)
        elif data == "bits":
            m = rng.choice((8, 16))
            case.update(m=m, dsub=128 // m, bbar=rng.choice((4, 5, 6)))
        return case
    if op == "ivf":
        nlist = _log(rng, 1024, 65536)
        nprobe = _log(rng, 8, 128)
        n = min(1_000_000_000, _log(rng, 200, 15_000) * nlist)
        q = _log(rng, 1, 1024)
        # no more probed codes than the largest listed case
        q = max(1, min(q, int(1e9 * nlist / (float(n) * nprobe))))
        return {"op": "ivf", "m": 8, "dsub": 16, "N": n, "nlist": nlist, "nprobe": nprobe, "Q": q, "r": _log(rng, 500, 4000),
                "k": rng.choice((10, 100)), "plane": rng.random() < 0.6}
    if op == "encode":
        data = rng.choice(("sift", "deep", "gist", "zipf", "bits"))
        m, dsub = {"sift": (8, 16), "deep": (8, 12), "gist": (16, 60), "zipf": (4, 32), "bits": (16, 8)}[data]
        n = _log(rng, 2000, 20_000 if data == "gist" else 250_000)
        return {"op": "encode", "data": data, "m": m, "dsub": dsub, "b": 8 if data == "bits" else 16, "n": n}
    m, dsub = rng.choice(((4, 32), (8, 16), (16, 8)))
    return {"op": "train", "m": m, "dsub": dsub, "b": 16, "bbar": rng.choice((6, 8)), "n": _log(rng, 66_000, 131_072),
            "iters": 1, "iters_same": 1}


# ---- inputs --------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _codebooks(data, m, dsub, b, seed, pbits=4):
    """Hierarchical codebooks with the scales of the workload that `data` names."""
    parents, sigma_c = {
        "zipf": (lambda s, g: 128.0 * torch.rand(s, generator=g, device=DEV), 4.0),
        "sift": (lambda s, g: 160.0 * torch.rand(s, generator=g, device=DEV), 12.0),
        "deep": (lambda s, g: 96 ** -0.5 * torch.randn(s, generator=g, device=DEV), 0.03),
        "gist": (lambda s, g: 0.3 * torch.rand(s, generator=g, device=DEV), 0.03),
        "bits": (lambda s, g: 0.3 * torch.randn(s, generator=g, device=DEV), 0.05),
        "residual": (lambda s, g: 20.0 * torch.randn(s, generator=g, device=DEV), 6.0),
    }[data]
    return synth.hierarchical_codebooks(m, dsub, b, pbits, parents, sigma_c, DEV, seed)


def _mixture_codes(n, sampler, means_rows, cb, per_component, seed):
    """Codes of n mixture vectors: sub-codes drawn from those of encoded vectors of the same component."""
    m = cb.shape[0]
    base = binding.encode(sampler(means_rows.repeat_interleave(per_component, 0)), cb).view(torch.int16)
    g = _gen(seed)
    comp = torch.randint(0, means_rows.shape[0], (n,), generator=g, device=DEV) * per_component
    codes = torch.empty((n, m), dtype=torch.int16, device=DEV)
    for j in range(m):
        pick = comp + torch.randint(0, per_component, (n,), generator=g, device=DEV)
        codes[:, j] = base[:, j].contiguous()[pick]
    return codes.view(torch.uint16)


def _sift_from(means, g):
    return (means + 12.0 * torch.randn(means.shape, generator=g, device=DEV)).clamp_(0.0, 255.0).round_()


def _vectors(data, n, D, seed, means_seed):
    if data == "sift":
        means = 160.0 * torch.rand((1024, D), generator=_gen(means_seed), device=DEV)
        g = _gen(seed)
        return _sift_from(means[torch.randint(0, 1024, (n,), generator=g, device=DEV)], g)
    if data == "deep":
        return synth.deep_like(n, DEV, seed, means_seed)
    if data == "gist":
        return synth.gist_like(n, DEV, seed, means_seed)
    scale = 128.0 if data == "zipf" else 0.3
    g = _gen(seed)
    if data == "zipf":
        return scale * torch.rand((n, D), generator=g, device=DEV)
    return scale * torch.randn((n, D), generator=g, device=DEV)


def _flat_inputs(c, seed):
    data, m, dsub, n, q = c["data"], c["m"], c["dsub"], c["N"], c["Q"]
    b = 8 if data == "bits" else 16
    cb = _codebooks(data, m, dsub, b, seed + 1)
    if data == "zipf":
        codes = synth.zipf_codes(n, m, 16, 4, DEV, seed + 2)
        g = _gen(seed + 3)
        y = synth.decode(codes[torch.randint(0, n, (q,), generator=g, device=DEV)], cb)
        queries = (y + 8.0 * torch.randn(y.shape, generator=g, device=DEV)).clamp_(0.0, 255.0)
        codes = codes.view(torch.uint16)
    elif data == "sift":
        means = 160.0 * torch.rand((1024, m * dsub), generator=_gen(seed + 7), device=DEV)
        g = _gen(seed + 4)
        codes = _mixture_codes(n, lambda x: _sift_from(x, g), means, cb, 256, seed + 2)
        queries = _vectors("sift", q, m * dsub, seed + 3, seed + 7)
    elif data == "gist":
        means = 0.3 * torch.rand((1024, m * dsub), generator=_gen(seed + 7), device=DEV)
        g = _gen(seed + 4)
        codes = _mixture_codes(n, lambda x: x + 0.03 * torch.randn(x.shape, generator=g, device=DEV), means, cb, 64, seed + 2)
        queries = _vectors("gist", q, m * dsub, seed + 3, seed + 7)
    elif data == "deep":
        codes = synth.random_codes(n, m, DEV, seed + 2).view(torch.uint16)
        queries = _vectors("deep", q, m * dsub, seed + 3, seed + 7)
    else:
        codes = torch.randint(0, 256, (n, m), generator=_gen(seed + 2), device=DEV, dtype=torch.uint8)
        queries = _vectors("bits", q, m * dsub, seed + 3, seed + 7)
    return cb, codes.contiguous(), queries.contiguous(), b


def prepare(case, seed):
    seed = 1000 * int(seed) + 190506900
    op = case["op"]
    if op == "flat":
        cb, codes, queries, b = _flat_inputs(case, seed)
        q, k = case["Q"], case["k"]
        # a serving program holds the derived codebooks (index build), one workspace and its output buffers
        ws = binding.search_workspace_bytes(case["N"], case["m"], q, case["r"], 0, b)
        return {"op": op, "queries": queries, "codebooks": cb, "derived": binding.derive_codebooks(cb, case.get("bbar", 8)),
                "codes": codes, "r": case["r"], "k": k, "ws": torch.empty(ws, dtype=torch.uint8, device=DEV),
                "ids": torch.empty((q, k), dtype=torch.uint32, device=DEV),
                "dist": torch.empty((q, k), dtype=torch.float32, device=DEV)}
    if op == "ivf":
        m, dsub, n, nlist, q, k = case["m"], case["dsub"], case["N"], case["nlist"], case["Q"], case["k"]
        cb = _codebooks("residual", m, dsub, 16, seed + 1)
        codes = synth.random_codes(n, m, DEV, seed + 2).view(torch.uint16)
        ws = binding.ivf_search_workspace_bytes(q, nlist, case["nprobe"], m, case["r"])
        return {"op": op, "queries": _vectors("sift", q, m * dsub, seed + 3, seed + 7), "codebooks": cb,
                "coarse": _vectors("sift", nlist, m * dsub, seed + 11, seed + 7),
                "derived": binding.derive_codebooks(cb), "codes": codes,
                "plane": binding.pack_low_bytes(codes) if case["plane"] else None,
                "offsets": synth.zipf_list_offsets(nlist, n, DEV, seed + 12), "nprobe": case["nprobe"], "r": case["r"], "k": k,
                "ws": torch.empty(ws, dtype=torch.uint8, device=DEV),
                "ids": torch.empty((q, k), dtype=torch.uint32, device=DEV),
                "dist": torch.empty((q, k), dtype=torch.float32, device=DEV)}
    m, dsub = case["m"], case["dsub"]
    if op == "encode":
        return {"op": op, "vectors": _vectors(case["data"], case["n"], m * dsub, seed + 3, seed + 7),
                "codebooks": _codebooks(case["data"], m, dsub, case["b"], seed + 1)}
    # training starts from vectors of the training set, a different choice per sub-quantizer
    x = _vectors("sift", case["n"], m * dsub, seed + 3, seed + 7)
    g = _gen(seed + 5)
    init = torch.stack([x[torch.randperm(case["n"], generator=g, device=DEV)[:1 << case["b"]], j * dsub:(j + 1) * dsub]
                        for j in range(m)]).contiguous()
    return {"op": op, "train": x, "init": init, "bbar": case["bbar"], "iters": case["iters"], "iters_same": case["iters_same"]}


# ---- one pass ------------------------------------------------------------------------------------------------

def run(s):
    if s["op"] == "flat":
        return binding.search(s["queries"], s["codebooks"], s["derived"], s["codes"], s["r"], s["k"], workspace=s["ws"],
                              ids=s["ids"], dist=s["dist"])
    if s["op"] == "ivf":
        return binding.ivf_search(s["queries"], s["coarse"], s["codebooks"], s["derived"], s["codes"], s["offsets"], s["nprobe"],
                                  s["r"], s["k"], plane=s["plane"], workspace=s["ws"], ids=s["ids"], dist=s["dist"])
    if s["op"] == "encode":
        return binding.encode(s["vectors"], s["codebooks"])
    return binding.build_quantizers(s["train"], s["init"], s["bbar"], s["iters"], s["iters_same"])


def work(case):
    m, dsub = case["m"], case["dsub"]
    D = m * dsub
    if case["op"] == "flat":
        b = 8 if case["data"] == "bits" else 16
        n, q, r, k = case["N"], case["Q"], case["r"], case["k"]
        rows = min(1 << b, q * r)          # centroids per sub-quantizer that a candidate can name
        nbytes = n * m * b // 8 + 4 * q * D + 4 * m * rows * dsub + 4 * D * (1 << case.get("bbar", 8)) + 8 * q * k
        # small tables, one addition per (query, code, sub-quantizer), table entries of the candidates
        return {"bytes": nbytes, "flops": 3 * q * D * (1 << case.get("bbar", 8)) + q * n * m + 3 * q * r * D}
    if case["op"] == "ivf":
        n, q, r, k, nlist, nprobe = (case[x] for x in ("N", "Q", "r", "k", "nlist", "nprobe"))
        # every query scans lists of its own; distinct codes cannot exceed the array
        lists = nlist * (1.0 - (1.0 - nprobe / nlist) ** q)
        probed = q * nprobe * n / nlist
        width = m if case["plane"] else 2 * m
        nbytes = int(n * lists / nlist * width) + 4 * q * D + 4 * nlist * D + 4 * m * min(65536, q * r) * dsub + 8 * q * k
        return {"bytes": nbytes, "flops": 2 * q * nlist * D + 3 * q * nprobe * D * 256 + int(probed * m) + 3 * q * r * D}
    n, kc = case["n"], 1 << case["b"]
    if case["op"] == "encode":
        return {"bytes": 4 * n * D + 4 * kc * D + n * m * case["b"] // 8, "flops": 2 * n * kc * D}
    # every k-means iteration and the last assignment compare all points with all centroids; the same-size
    # iterations compare all centroids with all groups
    kbar = 1 << case["bbar"]
    return {"bytes": 4 * n * D + 2 * 4 * kc * D + 4 * kbar * D,
            "flops": 2 * n * kc * D * (case["iters"] + 1) + 2 * kc * kbar * D * case["iters_same"]}


def tolerance(case):
    if case["op"] == "encode":
        return "exact"                     # the nearest centroid in double precision; equal distances: smaller index
    if case["op"] == "train":
        # the training vectors are whole numbers below 256: sums of them in double precision are exact in any
        # order, so every correct implementation rounds the same means to fp32
        return "exact"
    # fp32 distances against the same sums in 64 bits differ by 7e-8 (2-norm) and 3e-7 (largest); at most 1.2e-3 of
    # the ids (the 960-d vectors) are in another order there, where distances agree to the last bits
    return {"rel": 3e-7, "max": 1.5e-6, "differ": 5e-3}
