"""The performance cases of the query library: the calls a program makes through the public entry points of
paper_1702_05911_amd, with the sizes, distributions, formats and options they are made with.

A case is a dict of plain values.  Its "call" says which entry point is timed:
  query   pqt_query_batch on an index the program keeps (the online phase)
  exact   pqt_query_batch_exact: the same, then the exact distances of a short list
  brute   pqt_brute_force over the attached vectors (ground truth, small collections)
  train   pqt_train: codebooks and line table from a sample
  build   pqt_builder_create / add / finish: a collection binned, encoded and sorted into lists
Symbols follow include/pqt.h: D dimensions, P tree parts, k1/k2 centroids per level, M sub-parts of a code,
H bin slots, T tuples and C candidates per query, w refined clusters, k results.
"""
import math

import torch

DEVICE = 0
CLUSTERS = 1000
LATENT = 24


def listed():
    return [
        # one user's query against a million descriptors: latency, launches and host work count
        {"name": "one-query", "call": "query", "data": "bytes", "N": 1_000_000, "D": 128, "P": 2, "k1": 16, "k2": 8, "M": 8,
         "H": 16384, "T": 1024, "C": 4096, "codes": "table", "order": "summed", "nq": 1, "k": 10, "w": 8},
        # what a server collects in a few milliseconds, on a collection with long lists (odd batch size)
        {"name": "serve-67", "call": "query", "data": "bytes", "N": 4_000_000, "D": 128, "P": 2, "k1": 32, "k2": 16, "M": 8,
         "H": 262144, "T": 1024, "C": 10_000, "codes": "table", "order": "summed", "nq": 67, "k": 100, "w": 8},
        # the benchmark's headline: 10,000 queries on the SIFT1M shape, an index that fits the caches
        {"name": "batch-1M", "call": "query", "data": "bytes", "N": 1_000_000, "D": 128, "P": 2, "k1": 16, "k2": 8, "M": 8,
         "H": 16384, "T": 1024, "C": 4096, "codes": "table", "order": "summed", "nq": 10_000, "k": 100, "w": 8},
        # the same batch on the 100M benchmark's index, which does not fit them
        {"name": "batch-100M", "call": "query", "data": "bytes", "N": 100_000_000, "D": 128, "P": 2, "k1": 32, "k2": 16, "M": 8,
         "H": 262144, "T": 1024, "C": 10_000, "codes": "table", "order": "summed", "nq": 10_000, "k": 100, "w": 8},
        # (pair, lambda) codes of an odd number of sub-parts, odd sizes throughout
        {"name": "ragged-pairs", "call": "query", "data": "bytes", "N": 300_007, "D": 96, "P": 2, "k1": 20, "k2": 7, "M": 12,
         "H": 19600, "T": 500, "C": 3001, "codes": "pair", "order": "summed", "nq": 3217, "k": 37, "w": 5},
        # GIST1M shape: long float vectors, four tree parts, sparse bins
        {"name": "gist-1000", "call": "query", "data": "unit", "N": 1_000_000, "D": 960, "P": 4, "k1": 16, "k2": 8, "M": 16,
         "H": 268_435_456, "T": 4096, "C": 4096, "codes": "table", "order": "summed", "nq": 1000, "k": 100, "w": 4},
        # the tree the paper uses at its largest scale: four parts, bin numbers hashed to a prime near N/10
        {"name": "four-hashed", "call": "query", "data": "bytes", "N": 8_000_000, "D": 128, "P": 4, "k1": 32, "k2": 16, "M": 8,
         "H": 800_011, "T": 1024, "C": 10_000, "codes": "table", "order": "summed", "nq": 5003, "k": 100, "w": 8},
        # short lists re-ranked by exact distances to byte vectors
        {"name": "exact-1000", "call": "exact", "data": "bytes", "N": 1_000_000, "D": 128, "P": 2, "k1": 16, "k2": 8, "M": 8,
         "H": 16384, "T": 1024, "C": 4096, "codes": "table", "order": "summed", "nq": 10_000, "k": 100, "w": 8, "k_short": 1000,
         "vectors": "u8"},
        # ground truth of the benchmark's queries over byte vectors
        {"name": "brute-u8", "call": "brute", "data": "bytes", "N": 1_000_000, "D": 128, "nq": 10_000, "k": 100, "vectors": "u8"},
        # a smaller float collection searched exactly (odd sizes)
        {"name": "brute-f32", "call": "brute", "data": "unit", "N": 150_001, "D": 960, "nq": 777, "k": 10, "vectors": "f32"},
        # the offline phase: codebooks and line table from 100,000 vectors, as the benchmark trains them ...
        {"name": "train-100k", "call": "train", "data": "bytes", "n": 100_000, "D": 128, "P": 2, "k1": 16, "k2": 8, "M": 8,
         "iters": 20, "n_table": 100_000},
        # ... and a collection streamed through the builder
        {"name": "build-2M", "call": "build", "data": "bytes", "N": 2_000_003, "D": 128, "P": 2, "k1": 16, "k2": 8, "M": 8,
         "H": 16384, "T": 1024, "C": 4096, "codes": "table"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tree(rng, case):
    """Dimensions, tree and code length of a drawn case."""
    if case["data"] == "bytes":
        case["P"] = rng.choice((1, 2, 2, 2, 4))
        case["M"] = rng.choice((4, 8, 8, 8, 12, 16, 32))
        case["D"] = rng.choice((96, 128, 128)) if case["M"] != 12 else 96
        case["k1"] = rng.choice((16, 16, 20, 32, 48))
        case["k2"] = rng.choice((5, 7, 8, 16))
    else:
        case["P"] = rng.choice((2, 4))
        case["M"] = rng.choice((8, 16))
        case["D"] = rng.choice((192, 320, 960))
        case["k1"] = 16
        case["k2"] = rng.choice((7, 8))


def draw(rng):
    call = rng.choice(("query",) * 6 + ("exact", "brute", "train", "build"))
    case = {"call": call, "data": rng.choice(("bytes", "bytes", "bytes", "unit"))}
    if call == "brute":
        case["D"] = rng.choice((96, 128, 200)) if case["data"] == "bytes" else rng.choice((192, 320, 960))
        case["N"] = _log_int(rng, 20_000, 1_000_000 if case["data"] == "bytes" else 150_000)
        case["nq"] = _log_int(rng, 1, 10_000 if case["data"] == "bytes" else 1_000)
        case["k"] = rng.randint(1, 150)
        case["vectors"] = rng.choice(("u8", "f32")) if case["data"] == "bytes" and case["D"] % 16 == 0 else "f32"
        return case
    _tree(rng, case)
    if call == "train":
        case["n"] = _log_int(rng, 20_000, 100_000)
        case["iters"] = rng.randint(8, 20)
        case["n_table"] = case["n"] if rng.random() < 0.7 else 0
        return case
    big = case["data"] == "bytes"
    case["N"] = _log_int(rng, 100_000, 4_000_000 if big else 500_000)
    case["codes"] = "pair" if case["k1"] <= 20 and rng.random() < 0.3 else "table"
    bins = (case["k1"] * case["k2"]) ** case["P"]
    case["H"] = bins if bins <= (1 << 24) and (case["P"] < 4 or rng.random() < 0.5) else max(101, case["N"] // 10) | 1
    case["T"] = rng.randint(200, 1024) if case["P"] == 2 or rng.random() < 0.5 else rng.randint(1024, 4096)
    case["C"] = _log_int(rng, 1000, 10_000)
    if call == "build":
        case["N"] = min(case["N"], 16_000_000 // case["M"])
        return case
    case["order"] = "static" if case["P"] == 2 and case["H"] == bins and rng.random() < 0.15 else "summed"
    case["nq"] = _log_int(rng, 1, 10_000 if big else 1_000)
    if case["P"] == 4:
        case["nq"] = max(1, case["nq"] // 4)
    case["w"] = rng.randint(2, 8)
    case["k"] = rng.randint(1, 100)
    if call == "exact":
        case["k_short"] = max(case["k"], _log_int(rng, 100, 1000))
        case["vectors"] = rng.choice(("u8", "f32")) if big else "f32"
    return case


# ---- inputs --------------------------------------------------------------------------------------------------------
def _generator(seed, stream, part=0):
    g = torch.Generator(device=torch.device("cuda", DEVICE))
    g.manual_seed((int(seed) * 0x9E3779B1 + stream * 0x85EBCA6B + part * 0xC2B2AE35 + 0x165667B1) & 0x7FFFFFFFFFFFFFFF)
    return g


class _Source:
    """The vectors of one seed, drawn on the GPU piece by piece: clusters with Zipf-like weights, 24 latent
    directions and noise.  "bytes": whole numbers 0..255 with heavy tails and many zeros, as image descriptors
    are; "unit": floats in [0, 1] of unit length."""

    def __init__(self, data, D, seed):
        self.data, self.D, self.seed = data, D, seed
        dev = torch.device("cuda", DEVICE)
        g = _generator(seed, 1)
        rnd = dict(generator=g, device=dev)
        if data == "bytes":
            centres = torch.empty((CLUSTERS, D), device=dev).exponential_(1.0 / 28.0, generator=g)
            centres *= torch.exp(0.6 * torch.randn((1, D), **rnd))
            self.centres = (centres * (torch.rand((CLUSTERS, D), **rnd) < 0.8)).clamp_(0, 255)
            self.basis = 14.0 * torch.randn((LATENT, D), **rnd) * (torch.rand((LATENT, D), **rnd) < 0.5)
            self.noise = 6.0
        else:
            self.centres = torch.rand((CLUSTERS, D), **rnd) * (torch.rand((CLUSTERS, D), **rnd) < 0.7)
            self.basis = 0.08 * torch.randn((LATENT, D), **rnd)
            self.noise = 0.02
        wts = 1.0 / (torch.arange(CLUSTERS, device=dev, dtype=torch.float32) + 10.0) ** 0.9
        self.cdf = torch.cumsum(wts / wts.sum(), 0)

    def take(self, stream, part, count):
        g = _generator(self.seed, stream, part)
        rnd = dict(generator=g, device=self.centres.device)
        cl = torch.searchsorted(self.cdf, torch.rand((count,), **rnd)).clamp_(max=CLUSTERS - 1)
        x = torch.randn((count, self.D), **rnd).mul_(self.noise)
        x.addmm_(torch.randn((count, LATENT), **rnd), self.basis)
        if self.data == "bytes":
            gain = torch.rand((count, 1), **rnd).mul_(0.5).add_(0.81)
            return x.add_(self.centres[cl].mul_(gain)).round_().clamp_(0, 255)
        x.add_(self.centres[cl]).clamp_(0.0, 1.0)
        return x.div_(x.norm(dim=1, keepdim=True).clamp_min_(1e-12))


def _rows(case):
    """Vectors per piece that goes through the builder."""
    return 1 << 20 if case["D"] <= 256 else 1 << 18


def _pieces(case, source, n):
    step = _rows(case)
    return [(s, min(step, n - s), i) for i, s in enumerate(range(0, n, step))]


def _database(case, source):
    """All vectors as the program holds them beside the index."""
    dtype = torch.uint8 if case["vectors"] == "u8" else torch.float32
    X = torch.empty((case["N"], case["D"]), dtype=dtype, device=torch.device("cuda", DEVICE))
    for s, n, i in _pieces(case, source, case["N"]):
        X[s:s + n] = source.take(2, i, n)
    return X


def _index(case, source):
    from paper_1702_05911_amd import binding, builder
    step = _rows(case)

    def chunks(start, count):
        return source.take(2, start // step, min(step, case["N"] - start))[:count]
    index = builder.build_index_native(chunks=chunks, N=case["N"], D=case["D"], P=case["P"], k1=case["k1"], k2=case["k2"],
                                       M=case["M"], H=case["H"], T=case["T"], C=case["C"], train_n=min(case["N"], 100_000),
                                       chunk_rows=step, device=DEVICE, code_format=int(case["codes"] == "pair"))
    if case["order"] == "static":
        binding.pqt_set_bin_order(index, binding.PQT_ORDER_STATIC_SLOPES)
    return index


def prepare(case, seed):
    from paper_1702_05911_amd import binding
    source = _Source(case["data"], case["D"], seed)
    state = {"case": case}
    if case["call"] == "train":
        state["sample"] = source.take(2, 0, case["n"])
        return state
    if case["call"] == "build":
        state["pieces"] = [source.take(2, i, n) for _, n, i in _pieces(case, source, case["N"])]
        params = binding.pqt_train(state["pieces"][0][:100_000], P=case["P"], k1=case["k1"], k2=case["k2"], M=case["M"])
        params.update({n: case[n] for n in ("N", "D", "P", "k1", "k2", "M", "H", "T", "C")})
        params["code_format"] = int(case["codes"] == "pair")
        state["params"] = params
        return state
    if case["call"] == "brute":
        # the collection only: one bin holds everything, the tree is as small as it may be
        tree = dict(case, P=1, k1=2, k2=1, M=1, H=2, T=1, C=1024, codes="table", order="summed")
        index = _index(tree, source)
    else:
        index = _index(case, source)
    if "vectors" in case:
        state["vectors"] = _database(case, source)
        binding.pqt_index_set_vectors(index, state["vectors"])
    state["index"] = index
    state["queries"] = source.take(3, 0, case["nq"])
    state["ids"] = torch.empty((case["nq"], case["k"]), dtype=torch.int64, device=state["queries"].device)
    state["dists"] = torch.empty((case["nq"], case["k"]), dtype=torch.float32, device=state["queries"].device)
    return state


def run(state):
    from paper_1702_05911_amd import binding
    case = state["case"]
    call = case["call"]
    if call == "train":
        return binding.pqt_train(state["sample"], P=case["P"], k1=case["k1"], k2=case["k2"], M=case["M"], iters=case["iters"],
                                 n_table=case["n_table"])
    if call == "build":
        b = binding.pqt_builder_create(state["params"], DEVICE)
        for piece in state["pieces"]:
            binding.pqt_builder_add(b, piece)
        index = binding.pqt_builder_finish(b)
        binding.pqt_builder_free(b)
        lists = binding.pqt_index_export(index, ("offsets", "ids", "codes"))
        binding.pqt_index_free(index)
        return lists
    if call == "query":
        return binding.pqt_query_batch(state["index"], state["queries"], case["k"], case["w"], state["ids"], state["dists"])
    if call == "exact":
        return binding.pqt_query_batch_exact(state["index"], state["queries"], case["k_short"], case["k"], case["w"], state["ids"],
                                             state["dists"])
    return binding.pqt_brute_force(state["index"], state["queries"], case["k"], state["ids"], state["dists"])


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _code_bytes(case):
    return case["M"] * (2 if case["codes"] == "pair" else 1)


def work(case):
    D = case["D"]
    call = case["call"]
    if call == "train":
        # every Lloyd iteration reads the sample once per level and compares it with k1, then k2 centroids;
        # the last assignments once more; the line votes (a distance from three numbers) per sub-part and pair
        pairs = case["k1"] * (case["k1"] - 1) // 2
        return {"bytes": 4.0 * case["n"] * D * (2 * case["iters"] + 1) + 4.0 * case["n_table"] * D,
                "flops": 3.0 * case["n"] * D * (case["k1"] + case["k2"]) * case["iters"] + 8.0 * case["n_table"] * case["M"] * pairs}
    if call == "build":
        return {"bytes": case["N"] * (4.0 * D + 4.0 + _code_bytes(case)) + 4.0 * case["H"],
                "flops": case["N"] * (2.0 * D * (case["k1"] + case["k2"] * case["P"]) + 3.0 * 256 * case["M"])}
    out = 12.0 * case["nq"] * case["k"]
    if call == "brute":
        elem = 1 if case["vectors"] == "u8" else 4
        return {"bytes": float(elem) * case["N"] * D + 4.0 * case["nq"] * D + out, "flops": 2.0 * case["nq"] * case["N"] * D}
    # candidates: the budget where bins are filled; a bin of a sparse tree near a query holds about a tenth
    cand = min(case["C"], case["N"]) if case["N"] > case["H"] else min(case["C"], case["T"] // 10)
    per_query = 4.0 * D + cand * _code_bytes(case) + 4.0 * case.get("k_short", case["k"])
    flops = 2.0 * D * (case["k1"] + case["w"] * case["k2"]) + 1.0 * cand * case["M"]
    if call == "exact":
        per_query += case["k_short"] * D * (1.0 if case["vectors"] == "u8" else 4.0)
        flops += 3.0 * case["k_short"] * D
    return {"bytes": case["nq"] * per_query + out, "flops": case["nq"] * flops}


def tolerance(case):
    """About four times what the path differs from itself by when its sums are taken in another order (the dimensions
    permuted within the sub-parts) and, for floats searched exactly, from 64-bit arithmetic."""
    call = case["call"]
    if call == "build":
        return "exact"         # bins, ids and codes: one vector in another bin moves every list behind it
    if call == "brute":
        # whole numbers below 2^24 are exact in any order; floats: 5.0e-6, 1.8e-5 at most, and of the ids (near ties) 2.6e-4
        # with ten results, 1.6e-3 with 84
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3} if case["data"] == "bytes" else {"rel": 2e-5, "max": 1e-4, "differ": 6e-3}
    if call == "train":
        # one vector that changes its cell moves two centroids: 2.0e-4, 6.5e-3 at most on whole-number vectors; on floats
        # the iterations amplify it (0.29), so that only equal assignments can be compared
        return {"rel": 1e-3, "max": 0.03, "differ": 1e-3} if case["data"] == "bytes" else {"rel": 0.03, "max": 0.9, "differ": 0.01}
    # distances 1.8e-7; where two bins are a near tie at the end of the budget other candidates are scored: 1.3e-4 over
    # a batch, 0.026 for one distance, 3.0e-4 of the ids
    return {"rel": 5e-4, "max": 0.1, "differ": 1.2e-3}
