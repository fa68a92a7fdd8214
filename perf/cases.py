"""Workloads for timing the search engine and the index construction on one GPU.

A case is a dict of plain values: the entry point it takes (``kind``), the collection (documents,
mean and largest document length, centroids, Zipf exponent of the cluster sizes, bits per residual
component) and the call (queries, tokens per query, probes, t', k). The collections follow the
recipe of ``synth/`` (the tiny, small, mid, long and full workloads of this repository), drawn on
the GPU so that even the largest is ready in seconds: cluster popularity is Zipf, documents take
their tokens' clusters independently, residual codes are uniform (they come from quantile
buckets), and the tokens that the queries copy carry the codes of their own residuals.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2501_17788_amd as warp

DIM = 128
TOKEN_NOISE = 0.1   # a token is normalize(centroid + 0.1 n)
QUERY_NOISE = 0.05  # a query token is normalize(token + 0.05 n)
LEN_SIGMA = 0.6     # document lengths: lognormal with this sigma, clamped to [1, cap]
# standard deviation of a residual component of such a token: x - c = c (1/L - 1) + 0.1 n / L with
# L^2 = 1 + 128 * 0.1^2
_L = math.sqrt(1.0 + DIM * TOKEN_NOISE ** 2)
RESIDUAL_STD = math.sqrt((1.0 / _L - 1.0) ** 2 / DIM + (TOKEN_NOISE / _L) ** 2)


def _case(name, kind, docs, mean, cap, n_c, zipf, nbits, queries, qtok, nprobe, t_prime, k):
    c = {"kind": kind, "docs": docs, "mean": mean, "cap": cap, "n_c": n_c, "zipf": zipf, "nbits": nbits,
         "queries": queries, "qtok": qtok, "nprobe": nprobe, "t_prime": t_prime, "k": k, "literal": False}
    if name:
        c["name"] = name
    return c


def _build_case(name, tokens, docs, n_c, sample, steps, nbits, quant):
    c = {"kind": "build", "tokens": tokens, "docs": docs, "n_c": n_c, "sample": sample, "steps": steps,
         "nbits": nbits, "quant": quant}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one query against a few thousand documents (one tenant's collection): launches and latency
        _case("tiny_q1", "async", 4096, 32, 48, 1024, 1.1, 4, 1, 32, 16, 10_000, 10),
        # interactive search of a small collection (100k documents, 6.3M embeddings, b = 4)
        _case("small_q1", "async", 100_000, 64, 180, 1 << 15, 1.1, 4, 1, 32, 32, 40_000, 100),
        # a batch of queries against the small collection (an evaluation run)
        _case("small_q256", "async", 100_000, 64, 180, 1 << 15, 1.1, 4, 256, 32, 32, 40_000, 100),
        # host arrays in and out through the blocking call; 8-bit codes, ragged sizes throughout
        _case("host_b8_q77", "host", 99_991, 64, 180, 32_003, 1.1, 8, 77, 23, 32, 40_000, 100),
        # the allocation-free call of a serving loop; 1-bit codes, waves of a dozen queries
        _case("noalloc_b1_q40", "noalloc", 60_013, 64, 180, 20_001, 1.1, 1, 40, 32, 32, 30_000, 50),
        # wide probing and deep result lists (candidates for a reranker): the whole-list sorts
        _case("deep_q8", "async", 100_000, 64, 180, 1 << 15, 1.1, 4, 8, 32, 400, 40_000, 5000),
        # interactive search of a million documents (70M embeddings, b = 2)
        _case("mid_q1", "async", 1_000_000, 70, 512, 1 << 17, 1.1, 2, 1, 32, 32, 100_000, 100),
        # a batch against the million documents
        _case("mid_q256", "async", 1_000_000, 70, 512, 1 << 17, 1.1, 2, 256, 32, 32, 100_000, 100),
        # long documents, heavily skewed clusters (240M embeddings, b = 4), long result lists
        _case("long_q64", "async", 2_000_000, 120, 512, 1 << 18, 1.3, 4, 64, 32, 32, 100_000, 1000),
        # interactive search at passage-collection scale (8.8M documents, 600M embeddings, b = 2)
        _case("full_q1", "async", 8_800_000, 68, 512, 1 << 18, 1.1, 2, 1, 32, 32, 100_000, 1000),
        # a batch at that scale
        _case("full_q48", "async", 8_800_000, 68, 512, 1 << 18, 1.1, 2, 48, 32, 32, 100_000, 1000),
        # index construction: a million tokens into 2^14 clusters, four k-means steps, 4-bit codes
        _build_case("build_1m", 1_000_000, 15_000, 1 << 14, 125_000, 4, 4, 65_536),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    u = rng.random()
    if u < 0.12:
        tokens = _log_int(rng, 20_000, 1_000_000)
        n_c = 1 << int(math.log2(16 * math.sqrt(tokens)))  # clusters grow with the square root of the tokens
        if rng.random() < 0.5:
            n_c = rng.randint(n_c // 2 + 1, n_c)
        sample = rng.randint(max(n_c, tokens // 10), max(n_c + 1, tokens // 8))
        return _build_case(None, tokens, max(1, tokens // 64), n_c, sample, rng.randint(1, 4),
                           rng.choice([1, 2, 4, 4, 8]), min(tokens, rng.randint(20_000, 65_536)))
    kind = "async" if u < 0.75 else "host" if u < 0.83 else "noalloc" if u < 0.91 else "deep"
    most = {"async": 8_800_000, "host": 1_000_000, "noalloc": 300_000, "deep": 200_000}[kind]
    docs = _log_int(rng, 4096, most)
    mean = rng.randint(32, 120)
    nbits = rng.choice([1, 2, 2, 4, 4, 4, 8])
    while docs * mean * (2 * nbits * 8 + 4) > 24e9:  # the codes of the largest listed collection
        mean, nbits = max(32, mean - 16), max(1, nbits // 2)
    n = docs * mean
    n_c = min(1 << 18, 1 << int(math.log2(16 * math.sqrt(n))))
    if rng.random() < 0.4:
        n_c = rng.randint(n_c // 2 + 1, n_c)
    zipf = rng.choice([1.1, 1.1, 1.2, 1.3])
    qtok = 32 if rng.random() < 0.7 else rng.randint(1, 31)
    queries = 1 if rng.random() < 0.4 else _log_int(rng, 2, 256)
    nprobe = _log_int(rng, 4, 64)
    k = _log_int(rng, 10, 1000)
    literal = rng.random() < 0.1
    if kind == "deep":
        kind, queries = "async", min(queries, 8)
        nprobe, k = rng.randint(257, 512), rng.randint(4097, 10_000)
    c = _case(None, kind, docs, mean, 512, n_c, zipf, nbits, queries, qtok, min(nprobe, n_c), int(min(100_000, 15.8 * math.sqrt(n))), k)
    c["literal"] = literal
    top = next(x for x in listed() if x["name"] == "full_q48")
    per = 8 if literal else 4
    while c["queries"] > 1 and (_pairs(c) > _pairs(top) or c["queries"] * qtok * docs * per > 54e9):
        c["queries"] -= max(1, c["queries"] // 8)
    return c


# ---------------------------------------------------------------------------- inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _lengths(case, g):
    mu = math.log(case["mean"]) - LEN_SIGMA ** 2 / 2
    z = torch.randn(case["docs"], generator=g, device="cuda")
    return torch.exp(mu + LEN_SIGMA * z).round().clamp(1, case["cap"]).to(torch.int64)


def _zipf(n_c, s):
    p = torch.arange(1, n_c + 1, dtype=torch.float64, device="cuda") ** (-s)
    return p / p.sum()


def _bucket_tables(nbits):
    """Bucket weights (float32) and cutoffs (float64) of the residual components' quantiles."""
    nb = 1 << nbits
    q = (torch.arange(nb, dtype=torch.float64, device="cuda") + 0.5) / nb
    cut = torch.arange(1, nb, dtype=torch.float64, device="cuda") / nb
    return (RESIDUAL_STD * torch.special.ndtri(q)).float(), RESIDUAL_STD * torch.special.ndtri(cut)


def _pack(codes, nbits):
    """Codes [n, 128] packed 8 / nbits to a byte, the first dimension in the top bits."""
    per = 8 // nbits
    c = codes.to(torch.int32).reshape(codes.shape[0], DIM // per, per)
    shift = torch.tensor([8 - nbits * (p + 1) for p in range(per)], dtype=torch.int32, device=codes.device)
    return (c << shift).sum(-1).to(torch.uint8)


def _collection(case, seed):
    """The index arrays and the query tokens of a search case, on the GPU."""
    g = _generator(seed)
    n_c, nbits = case["n_c"], case["nbits"]
    C = _unit(torch.randn(n_c, DIM, generator=g, device="cuda"))
    lens = _lengths(case, g)
    ends = lens.cumsum(0)
    n = int(ends[-1])
    perm = torch.randperm(n_c, generator=g, device="cuda").to(torch.int32)
    cdf = _zipf(n_c, case["zipf"]).cumsum(0)
    cl = torch.empty(n, dtype=torch.int32, device="cuda")
    step = 1 << 26
    for a in range(0, n, step):
        u = torch.rand(min(step, n - a), generator=g, device="cuda", dtype=torch.float64)
        cl[a:a + step] = perm[torch.searchsorted(cdf, u, right=True).clamp_(max=n_c - 1)]
    sizes = torch.zeros(n_c, dtype=torch.int64, device="cuda")
    for a in range(0, n, step):
        sizes += torch.bincount(cl[a:a + step], minlength=n_c)
    offsets = torch.zeros(n_c + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = sizes.cumsum(0)
    # the tokens that the queries copy: nq documents, qtok of the tokens of each with replacement
    nq, T = case["queries"], case["qtok"]
    target = torch.randint(case["docs"], (nq,), generator=g, device="cuda")
    pos = (torch.rand(nq, T, generator=g, device="cuda", dtype=torch.float64) * lens[target][:, None]).long()
    want = (ends[target] - lens[target])[:, None] + torch.minimum(pos, lens[target][:, None] - 1)
    ids, back = want.reshape(-1).unique(return_inverse=True)
    own = cl[ids].long()
    x = _unit(C[own] + TOKEN_NOISE * torch.randn(len(ids), DIM, generator=g, device="cuda"))
    # clusters in order, documents ascending inside each (a stable sort of the tokens)
    cl, order = cl.sort(stable=True)
    del cl
    docs = torch.repeat_interleave(torch.arange(case["docs"], dtype=torch.int32, device="cuda"), lens, output_size=n)
    docs = docs[order]
    mark = torch.zeros(n, dtype=torch.bool, device="cuda")
    mark[ids] = True
    at = mark[order].nonzero().reshape(-1)  # rows of the wanted tokens in cluster order
    row = torch.empty_like(at)
    row[torch.searchsorted(ids, order[at])] = at
    del order, mark
    weights, cut = _bucket_tables(nbits)
    codes = torch.empty(n, DIM * nbits // 8, dtype=torch.uint8, device="cuda")
    words = codes.view(torch.int32).reshape(-1)
    for a in range(0, words.numel(), 1 << 29):
        words[a:a + (1 << 29)].random_(-(1 << 31), (1 << 31), generator=g)
    codes[row] = _pack(torch.searchsorted(cut, (x - C[own]).double(), right=True), nbits)
    q = _unit(x[back] + QUERY_NOISE * torch.randn(nq * T, DIM, generator=g, device="cuda")).reshape(nq, T, DIM)
    return {"centroids": C, "offsets": offsets, "doc_ids": docs, "codes": codes, "weights": weights, "queries": q.contiguous()}


def _tokens(case, seed):
    """The inputs of an index construction, on the GPU: tokens around Zipf-popular centres, as in a
    collection, their documents, the sampled tokens and the starting vectors."""
    g = _generator(seed)
    n, n_c = case["tokens"], case["n_c"]
    centres = _unit(torch.randn(n_c, DIM, generator=g, device="cuda"))
    cdf = _zipf(n_c, 1.1).cumsum(0)
    z = torch.searchsorted(cdf, torch.rand(n, generator=g, device="cuda", dtype=torch.float64)).clamp_(max=n_c - 1)
    x = _unit(centres[z] + TOKEN_NOISE * torch.randn(n, DIM, generator=g, device="cuda"))
    docs = (torch.arange(n, device="cuda") * case["docs"] // n).to(torch.int32)
    sample = torch.randperm(n, generator=g, device="cuda")[:case["sample"]].sort().values
    start = x[sample[torch.randperm(case["sample"], generator=g, device="cuda")[:n_c]]]
    return {"tokens": x.contiguous(), "docs": docs, "sample": sample, "start": start.contiguous()}


def prepare(case, seed):
    if case["kind"] == "build":
        return {"case": case, **_tokens(case, seed)}
    d = _collection(case, seed)
    ix = warp.Index.from_device(d["centroids"], d["offsets"], d["doc_ids"], d["codes"], case["nbits"], d["weights"],
                                case["docs"])
    if case["literal"]:
        ix.set_scoring(warp.SCORING_EQ1_LITERAL)
    q = d["queries"]
    del d
    torch.cuda.empty_cache()  # the index holds its own copies; the engine's scratch needs the room
    return {"case": case, "index": ix, "queries": q.cpu().numpy() if case["kind"] == "host" else q}


def run(state):
    case = state["case"]
    if case["kind"] == "build":
        return warp.build_index(state["tokens"], state["docs"], case["docs"], state["start"], state["sample"],
                                case["steps"], case["nbits"], case["quant"])
    ix = state["index"]
    search = {"async": ix.search_async, "host": ix.search, "noalloc": ix.search_noalloc}[case["kind"]]
    return search(state["queries"], case["nprobe"], case["t_prime"], case["k"])


# ---------------------------------------------------------------------------- work and tolerance

def _probabilities(case):
    p = np.arange(1, case["n_c"] + 1, dtype=np.float64) ** (-case["zipf"])
    return p / p.sum()


def _pairs(case):
    """Expected (query token, embedding) pairs scored: a token probes its own cluster (as popular
    as the cluster is large) and nprobe - 1 others, which lie anywhere."""
    p = _probabilities(case)
    n = case["docs"] * case["mean"]
    return case["queries"] * case["qtok"] * n * (float((p * p).sum()) + (case["nprobe"] - 1) / case["n_c"])


def work(case):
    if case["kind"] == "build":
        n, n_c = case["tokens"], case["n_c"]
        moved = n * (4 * DIM + 4) + n * (DIM * case["nbits"] // 8 + 8) + 2 * n_c * 4 * DIM + 8 * case["sample"]
        return {"bytes": float(moved), "flops": 2.0 * DIM * n_c * (n + case["steps"] * case["sample"])}
    p = _probabilities(case)
    tokens = case["queries"] * case["qtok"]
    n, n_c = case["docs"] * case["mean"], case["n_c"]
    seen = 1.0 - np.exp(tokens * (np.log1p(-np.minimum(p, 1 - 1e-12)) + math.log1p(-min(1 - 1e-12, (case["nprobe"] - 1) / n_c))))
    distinct = n * float((p * seen).sum())
    moved = distinct * (DIM * case["nbits"] // 8 + 4) + 4 * DIM * (n_c + tokens) + case["queries"] * (16 * case["k"] + 4)
    return {"bytes": moved, "flops": 2.0 * DIM * (_pairs(case) + tokens * n_c)}


def tolerance(case):
    """Results are defined in fixed point (scores) and exact sums (construction): the same bits
    whatever the order of evaluation."""
    return "exact"


# ---------------------------------------------------------------------------- 64-bit references

def _unpack(codes, nbits):
    per = 8 // nbits
    shift = torch.tensor([8 - nbits * (p + 1) for p in range(per)], dtype=torch.int32, device=codes.device)
    c = (codes.to(torch.int32)[:, :, None] >> shift) & ((1 << nbits) - 1)
    return c.reshape(codes.shape[0], DIM).long()


def _exact_search(case, seed):
    if _pairs(case) > 3e9 or case["docs"] * case["mean"] > 80e6:
        return None
    d = _collection(case, seed)
    nq, T, P, k = case["queries"], case["qtok"], case["nprobe"], case["k"]
    if nq * T * case["docs"] * 8 * (2 if case["literal"] else 1) > 40e9:
        return None
    C, w = d["centroids"].double(), d["weights"].double()
    q = d["queries"].double().reshape(nq * T, DIM)
    sizes = d["offsets"].diff()
    sel = torch.empty(nq * T, P, dtype=torch.int64, device="cuda")
    m = torch.empty(nq * T, dtype=torch.float64, device="cuda")
    for a in range(0, nq * T, 256):
        s, order = (q[a:a + 256] @ C.T).sort(dim=1, descending=True, stable=True)
        sel[a:a + 256] = order[:, :P]
        over = sizes[order].cumsum(1) > case["t_prime"]
        first = torch.where(over.any(1), over.int().argmax(1), s.shape[1] - 1)
        m[a:a + 256] = s.gather(1, first[:, None])[:, 0]
    # cluster by cluster: its embeddings decompressed, against the tokens that probe it
    best = torch.full((nq * T * case["docs"],), -math.inf, dtype=torch.float64, device="cuda")
    found = torch.zeros(nq * T * case["docs"], dtype=torch.float64, device="cuda") if case["literal"] else None
    cl, by = sel.reshape(-1).sort()
    tok = by // P
    off = d["offsets"].tolist()
    ids, start = cl.unique_consecutive(return_counts=True)
    at = 0
    for c, cnt in zip(ids.tolist(), start.tolist()):
        t = tok[at:at + cnt]
        at += cnt
        for a in range(off[c], off[c + 1], 1 << 21):
            b = min(off[c + 1], a + (1 << 21))
            docs = d["doc_ids"][a:b].long()
            x = C[c] + w[_unpack(d["codes"][a:b], case["nbits"])]
            for t0 in range(0, cnt, 64):
                tt = t[t0:t0 + 64]
                place = (tt[:, None] * case["docs"] + docs).reshape(-1)
                best.scatter_reduce_(0, place, (q[tt] @ x.T).reshape(-1), "amax")
                if found is not None:
                    found.scatter_add_(0, place, torch.ones_like(place, dtype=torch.float64))
    best = best.reshape(nq, T, case["docs"])
    scores = torch.full((nq, k), -math.inf, dtype=torch.float64, device="cuda")
    length = torch.bincount(d["doc_ids"], minlength=case["docs"]).double()
    m = m.reshape(nq, T)
    for i in range(nq):
        got = best[i] > -math.inf
        v = best[i]
        if found is not None:
            part = got & (found.reshape(nq, T, -1)[i] < length)
            v = torch.where(part, torch.maximum(v, m[i][:, None]), v)
        total = torch.where(got, v, m[i][:, None]).sum(0)
        total = torch.where(got.any(0), total, -math.inf)
        top = total.topk(min(k, case["docs"])).values
        scores[i, :len(top)] = top
    if case["kind"] == "host":
        return None, scores.cpu().numpy(), None
    return None, scores, None, None


def _exact_build(case, seed):
    if 2.0 * DIM * case["n_c"] * (case["tokens"] + case["steps"] * case["sample"]) > 1e13:
        return None
    d = _tokens(case, seed)
    x, nb = d["tokens"], 1 << case["nbits"]
    C = (d["start"].double() / d["start"].double().norm(dim=1, keepdim=True)).float()

    def nearest(rows):
        return torch.cat([(r.double() @ C.double().T).argmax(1) for r in rows.split(8192)])

    xs = x[d["sample"]]
    fixed = (xs.double() * 2.0 ** 30).round().long()
    for _ in range(case["steps"]):
        a = nearest(xs)
        sums = torch.zeros(case["n_c"], DIM, dtype=torch.int64, device="cuda").index_add_(0, a, fixed).double()
        norm = sums.norm(dim=1, keepdim=True)
        C = torch.where(norm > 0, sums / norm.clamp(min=1.0), C.double()).float()
    a = nearest(x[:case["quant"]])
    r = (x[:case["quant"]] - C[a]).reshape(-1).sort().values.double()
    n = r.numel()
    cut = [r[max(1, -(-n * j // nb)) - 1] for j in range(1, nb)]
    mid = [r[max(1, -(-n * (2 * j + 1) // (2 * nb))) - 1] for j in range(nb)]
    return {"centroids": C.double(), "offsets": None, "doc_ids": None, "codes": None, "weights": torch.stack(mid),
            "cutoffs": torch.stack(cut), "assign": None}


def exact(case, seed):
    return _exact_build(case, seed) if case["kind"] == "build" else _exact_search(case, seed)
