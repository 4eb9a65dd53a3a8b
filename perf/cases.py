"""The work that a user of the retrieval library has it do, as cases to be timed and compared.

A case is a plain dict.  ``op`` names the entry point of ``paper_2608_08340_amd.Index``:

dense        ``search_dense``: exact top-k of a query batch
hybrid       ``search_hybrid``: dense list and BM25 list, reciprocal rank fusion
dense_first  ``search_hybrid_dense_first``: BM25 of the dense candidates, fused with their order
weighted     ``search_hybrid_weighted``: min-max weighted sum of both scores over the corpus
ingest       a new ``Index``, ``upsert`` of ready fp32 vectors and ``upsert_pooled`` of chunks
             straight from the embedder's hidden states

Rows are unit vectors of a Gaussian mixture (about 128 rows a cluster, sigma 0.3), queries
noisy copies of rows (0.1 per coordinate), the sparse corpus Poisson-long chunks of Zipf(1.1)
terms over a 30,000-term vocabulary: the distributions of the repository's own workloads,
drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_08340_amd as oprag

DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ELEM = {"f32": 4, "bf16": 2, "f16": 2}
VOCAB, ZIPF, CHUNK_TOKENS = 30000, 1.1, 256
K1, B = 1.2, 0.75
RRF_K = 60


def listed():
    return [
        # the smallest call: a test-sized fp32 index, a handful of queries (launches and latency)
        {"name": "tiny_f32_b16_k5", "op": "dense", "rows": 1024, "dim": 384, "dtype": "f32", "batch": 16, "k": 5},
        # one interactive user on the 32K-chunk index: a pass over the index per query
        {"name": "serve_b1_k5", "op": "dense", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 1, "k": 5},
        # a few concurrent users, a longer list
        {"name": "serve_b16_k10", "op": "dense", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 16, "k": 10},
        # the headline workload: batched retrieval at the paper's corpus size
        {"name": "batch256_k5", "op": "dense", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 256, "k": 5},
        # one evaluation scenario's query set at once
        {"name": "batch1024_k5", "op": "dense", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 1024, "k": 5},
        # sizes as they come: rows and batch that fill no tile, fp16
        {"name": "ragged_f16_b333_k10", "op": "dense", "rows": 99991, "dim": 768, "dtype": "f16", "batch": 333, "k": 10},
        # a large corpus, one evaluation set
        {"name": "large_1m_b1024_k10", "op": "dense", "rows": 1048576, "dim": 768, "dtype": "bf16", "batch": 1024,
         "k": 10},
        # the streaming workload's search: millions of rows, thousands of queries, deep lists
        {"name": "stream_8m_b4096_k100", "op": "dense", "rows": 8454144, "dim": 384, "dtype": "f16", "batch": 4096,
         "k": 100},
        # full hybrid retrieval of a batch: dense top-100, BM25 top-100, rank fusion
        {"name": "hybrid_b256", "op": "hybrid", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 256, "k": 5,
         "k_dense": 100, "k_sparse": 100, "terms": 8},
        # the serving schedule: 128 dense candidates, lexical rerank
        {"name": "dense_first_b256", "op": "dense_first", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 256,
         "k": 5, "k_dense": 128, "terms": 8},
        # weighted score fusion for a small batch
        {"name": "weighted_b64", "op": "weighted", "rows": 32768, "dim": 1024, "dtype": "bf16", "batch": 64, "k": 5,
         "terms": 8},
        # an ingest step: 65,536 ready vectors and 256 chunks of up to 512 tokens from the embedder
        {"name": "ingest_64k", "op": "ingest", "rows": 65536, "dim": 1024, "dtype": "bf16", "chunks": 256,
         "tokens": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["dense", "dense", "dense", "dense", "f32", "hybrid", "dense_first", "weighted", "ingest"])
    dim = 128 * rng.randint(3, 8)  # embedders of 384 to 1,024 dimensions
    dtype = rng.choice(["bf16", "f16"])
    if op == "f32":
        return {"op": "dense", "rows": _log_int(rng, 1000, 32768), "dim": 4 * rng.randint(96, 256), "dtype": "f32",
                "batch": _log_int(rng, 1, 64), "k": rng.randint(1, 16)}
    if op == "dense":
        rows = _log_int(rng, 5000, 4000000)
        # at most a tenth of the largest listed case's products, and 12 GB of rows
        batch = min(_log_int(rng, 1, 4096), max(1, int(1.3e12 / (rows * dim))))
        k = rng.randint(1, 16) if rng.random() < 0.7 else rng.randint(17, 128)
        return {"op": "dense", "rows": rows, "dim": dim, "dtype": dtype, "batch": batch, "k": k}
    if op == "ingest":
        return {"op": "ingest", "rows": _log_int(rng, 1000, 200000), "dim": dim, "dtype": dtype,
                "chunks": _log_int(rng, 16, 512), "tokens": _log_int(rng, 32, 512)}
    case = {"op": op, "rows": _log_int(rng, 4096, 65536), "dim": dim, "dtype": dtype, "batch": _log_int(rng, 1, 512),
            "k": rng.randint(1, 16), "terms": rng.randint(2, 24)}
    if op == "hybrid":
        case["k_dense"], case["k_sparse"] = rng.randint(50, 128), rng.randint(50, 128)
    if op == "dense_first":
        case["k_dense"] = rng.randint(50, 128)
    return case


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + stream)


def _rows(case, seed, dtype):
    """[rows x dim] unit vectors of the mixture, rounded to dtype, drawn in pieces."""
    n, d = case["rows"], case["dim"]
    g = _gen(seed, 1)
    centres = torch.randn((max(8, n // 128), d), generator=g, device="cuda")
    out = torch.empty((n, d), dtype=dtype, device="cuda")
    step = 1 << 19
    for lo in range(0, n, step):
        m = min(step, n - lo)
        x = torch.randn((m, d), generator=g, device="cuda").mul_(0.3)
        x += centres[torch.randint(centres.shape[0], (m,), generator=g, device="cuda")]
        x /= x.norm(dim=1, keepdim=True)
        out[lo:lo + m] = x
    return out


def _queries(case, seed, rows):
    g = _gen(seed, 2)
    src = torch.randint(case["rows"], (case["batch"],), generator=g, device="cuda")
    q = rows[src].float() + 0.1 * torch.randn((case["batch"], case["dim"]), generator=g, device="cuda")
    return (q / q.norm(dim=1, keepdim=True)).to(rows.dtype).contiguous()


def _pmf():
    w = np.arange(1, VOCAB + 1, dtype=np.float64) ** -ZIPF
    return w / w.sum()


def _terms(n, g):
    cdf = torch.from_numpy(np.cumsum(_pmf())).cuda()
    u = torch.rand((n,), generator=g, device="cuda", dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=VOCAB - 1)


def _corpus(case, seed):
    """CSR postings (term -> ascending chunks, term frequencies) and chunk lengths."""
    n, g = case["rows"], _gen(seed, 3)
    length = torch.poisson(torch.full((n,), float(CHUNK_TOKENS), device="cuda"), generator=g).clamp_(min=1).long()
    chunk = torch.repeat_interleave(torch.arange(n, device="cuda"), length)
    key, tf = torch.unique(_terms(chunk.numel(), g) * n + chunk, return_counts=True)
    term = torch.div(key, n, rounding_mode="floor")
    indptr = torch.zeros(VOCAB + 1, dtype=torch.int64, device="cuda")
    indptr[1:] = torch.bincount(term, minlength=VOCAB).cumsum(0)
    return indptr, (key - term * n).int(), tf.int(), length.int()


def _query_terms(case, seed):
    nt, b = case["terms"], case["batch"]
    terms = _terms(b * nt, _gen(seed, 4)).int()
    return torch.arange(0, b * nt + 1, nt, dtype=torch.int32, device="cuda"), terms


def _hidden(case, seed):
    g = _gen(seed, 5)
    m, T, d = case["chunks"], case["tokens"], case["dim"]
    hidden = torch.randn((m, T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    lengths = torch.randint(max(1, T // 16), T + 1, (m,), generator=g, device="cuda", dtype=torch.int32)
    return hidden, lengths


def prepare(case, seed):
    if case["op"] == "ingest":
        hidden, lengths = _hidden(case, seed)
        return {"case": case, "rows": _rows(case, seed, torch.float32), "hidden": hidden, "lengths": lengths}
    rows = _rows(case, seed, DTYPE[case["dtype"]])
    idx = oprag.Index(case["dim"], case["rows"], DTYPE[case["dtype"]])
    idx.upsert(rows)
    st = {"case": case, "idx": idx, "q": _queries(case, seed, rows)}
    if case["op"] != "dense":
        idx.attach_sparse(*_corpus(case, seed), K1, B)
        st["qi"], st["qt"] = _query_terms(case, seed)
    return st


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def run(st):
    c, op = st["case"], st["case"]["op"]
    if op == "dense":
        return st["idx"].search_dense(st["q"], c["k"])
    if op == "hybrid":
        return st["idx"].search_hybrid(st["q"], st["qi"], st["qt"], c["k_dense"], c["k_sparse"], RRF_K, c["k"])
    if op == "dense_first":
        return st["idx"].search_hybrid_dense_first(st["q"], st["qi"], st["qt"], c["k_dense"], RRF_K, c["k"])
    if op == "weighted":
        return st["idx"].search_hybrid_weighted(st["q"], st["qi"], st["qt"], 0.5, 0.5, c["k"])
    idx = oprag.Index(c["dim"], c["rows"] + c["chunks"], DTYPE[c["dtype"]])
    idx.upsert(st["rows"])
    idx.upsert_pooled(st["hidden"], st["lengths"])
    st["idx"] = idx  # the new index takes the place of the last one
    return idx.slab


# ---------------------------------------------------------------------------------------
# what a pass cannot do without, and how far correct implementations may lie apart
# ---------------------------------------------------------------------------------------
def work(case):
    es, d = ELEM[case["dtype"]], case["dim"]
    if case["op"] == "ingest":
        tokens = case["chunks"] * (max(1, case["tokens"] // 16) + case["tokens"]) / 2
        nbytes = case["rows"] * d * (4 + es) + tokens * d * 2 + case["chunks"] * d * es
        return {"bytes": int(nbytes), "flops": int(tokens * d)}
    n, b = case["rows"], case["batch"]
    nbytes = n * d * es + b * d * es + b * case["k"] * 12
    flops = 2 * n * d * b
    if case["op"] != "dense":
        p = _pmf()
        df = n * (1 - np.exp(-CHUNK_TOKENS * p))  # expected chunks of each term
        if case["op"] == "dense_first":  # the candidates' own term lists
            posts = b * case["k_dense"] * df.sum() / n
        else:  # the postings of the batch's distinct terms
            posts = ((1 - (1 - p) ** (b * case["terms"])) * df).sum()
        nbytes += 8 * posts
        flops += 2 * b * case["terms"] * (p * df).sum()
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """About four times what the start showed against 64 bits over the listed and 14 drawn cases."""
    if case["op"] == "ingest":
        # ready vectors are rounded once and the same everywhere; a pooled sum in another order
        # moves a few values by one step of the storage type (bf16: 2^-8 of the value at most)
        return {"rel": 1e-4, "max": 0.01}
    if case["op"] in ("hybrid", "dense_first"):
        # fused values are functions of ranks: where two neighbours of a list are within the sums'
        # rounding of each other and swap, a value moves by 1/61 - 1/62 of 1/61 = 1.6 % at most
        # (seen: no swap, 6e-8; one swap in 256 x 5 values is 5e-4 in the 2-norm)
        return {"rel": 1e-3, "max": 0.02, "differ": 2e-3}
    # seen: 1e-7 to 1.9e-7 (f16, bf16), 2.7e-7 to 3.4e-7 (f32), 9e-7 at most on one value, and
    # 1.6e-4 of the ids (swaps of neighbours at k = 100)
    return {"rel": 1.5e-6 if case["dtype"] == "f32" else 1e-6, "max": 4e-6, "differ": 2e-3}


def _topk(scores, k):
    """Top k of each row by (score descending, id ascending)."""
    kk = min(k, scores.shape[1])
    s, i = torch.sort(scores, dim=1, descending=True, stable=True)
    return s[:, :kk], i[:, :kk]


def _dense64(case, seed):
    """fp64 inner products of every query and row, in pieces of rows: yields (first row, scores)."""
    rows = _rows(case, seed, DTYPE[case["dtype"]])
    q = _queries(case, seed, rows).double()
    step = max(4096, (1 << 28) // max(1, case["batch"]))
    for lo in range(0, case["rows"], step):
        yield lo, q @ rows[lo:lo + step].double().T


def _dense_top64(case, seed, k):
    top = ids = None
    for lo, s in _dense64(case, seed):
        v, i = torch.topk(s, min(k, s.shape[1]), dim=1)
        i = i + lo
        if top is not None:
            v, i = torch.cat([top, v], 1), torch.cat([ids, i], 1)
        order = torch.argsort(i, dim=1)
        v, i = v.gather(1, order), i.gather(1, order)
        v, at = _topk(v, k)
        top, ids = v, i.gather(1, at)
    return top, ids


def _bm25_64(case, seed):
    """fp64 BM25 of every query and chunk."""
    indptr, chunk, tf, length = _corpus(case, seed)
    _, terms = _query_terms(case, seed)
    n, b = case["rows"], case["batch"]
    f, dl = tf.double(), length.double()
    w = f * (K1 + 1) / (f + K1 * (1 - B + B * dl[chunk.long()] / dl.mean()))
    df = (indptr[1:] - indptr[:-1]).double()
    idf = torch.log1p((n - df + 0.5) / (df + 0.5))
    out = torch.zeros((b, n), dtype=torch.float64, device="cuda")
    bounds = indptr.tolist()
    for j, t in enumerate(terms.tolist()):
        lo, hi = bounds[t], bounds[t + 1]
        out[j // case["terms"], chunk[lo:hi].long()] += idf[t] * w[lo:hi]
    return out


def _minmax(x):
    lo, hi = x.amin(1, keepdim=True), x.amax(1, keepdim=True)
    return torch.where(hi > lo, (x - lo) / (hi - lo), torch.zeros_like(x))


def _fuse(case, lists):
    """Reciprocal rank fusion of id lists (-1 past a list's end) per query."""
    b, n, k = case["batch"], case["rows"], case["k"]
    fused = torch.zeros((b, n + 1), dtype=torch.float64, device="cuda")
    for ids in lists:
        rank = 1.0 / (RRF_K + 1 + torch.arange(ids.shape[1], device="cuda", dtype=torch.float64))
        fused.scatter_add_(1, torch.where(ids < 0, n, ids), rank.expand(b, -1))
    top, ids = _topk(fused[:, :n], k)
    return torch.where(top > 0, top, -math.inf), torch.where(top > 0, ids, -1)


def exact(case, seed):
    op = case["op"]
    if op == "ingest":
        hidden, lengths = _hidden(case, seed)
        keep = torch.arange(case["tokens"], device="cuda")[None, :] < lengths[:, None]
        pooled = torch.stack([(h.double() * m[:, None]).sum(0) for h, m in zip(hidden, keep)])
        pooled /= pooled.norm(dim=1, keepdim=True)
        return torch.cat([_rows(case, seed, torch.float32).double(), pooled])
    if op == "dense":
        return list(_dense_top64(case, seed, case["k"]))
    lex = _bm25_64(case, seed)
    if op == "weighted":
        dense = torch.cat([s for _, s in _dense64(case, seed)], 1)
        return list(_topk(0.5 * _minmax(dense) + 0.5 * _minmax(lex), case["k"]))
    _, cand = _dense_top64(case, seed, case["k_dense"])
    if op == "hybrid":
        s, i = _topk(lex, case["k_sparse"])
        return list(_fuse(case, [cand, torch.where(s > 0, i, -1)]))
    # dense first: the candidates ranked by (BM25 descending, id ascending), positive scores only
    by_id = torch.sort(cand, dim=1)[0]
    s, at = _topk(lex.gather(1, by_id), cand.shape[1])
    return list(_fuse(case, [cand, torch.where(s > 0, by_id.gather(1, at), -1)]))
