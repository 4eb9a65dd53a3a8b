"""BM25 selection and term parsing at the edges of their ranges, on the GPU against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import accept, bm25
from tests.gpu_helpers import device, log, make_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [16, 17])       # 64 groups for the threshold, 256 beyond
@pytest.mark.parametrize("terms", [1, 63, 64, 65, 130])  # in the lanes of one wave up to 64
def test_bm25_terms_and_threshold_edges(terms, k):
    """Queries of exactly `terms` occurrences with repeats (a term first met in the first and again
    in the last place), unknown terms between them, over 5,000 chunks.  One query holds a single
    frequent term whose equal scores (tied term frequencies and lengths) overfill the k."""
    dev = device()
    vocab, n_docs, nq = 300, 5000, 24
    ind, toks = synth.sparse_corpus(synth.rng(900 + terms, 3), n_docs, vocab, 1.1, 30.0)
    csr = synth.csr_from_tokens(ind, toks, vocab)
    g = np.random.default_rng(terms * 100 + k)
    qs = [list(g.integers(0, vocab, size=terms)) for _ in range(nq)]
    for q in qs[1:]:
        q[-1] = q[0]
        q[terms // 2] = -1 if g.random() < 0.5 else vocab
    qs[0] = [0] * terms
    qi = (np.arange(nq + 1) * terms).astype(np.int32)
    qt = np.array([t for q in qs for t in q], dtype=np.int32)
    idx = make_index(torch.zeros((n_docs, 128), dtype=torch.bfloat16), "bf16")

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(dev)

    idx.attach_sparse(t(csr.term_indptr), t(csr.post_chunk), t(csr.post_tf), t(csr.doc_len), 1.2, 0.75)
    log("bm25 edges", terms, k)
    sc, ids = idx.search_sparse(t(qi), t(qt), k)
    torch.cuda.synchronize()
    qt_oracle = np.where((qt >= 0) & (qt < vocab), qt, 10 ** 6).astype(np.int64)  # unknown terms match nothing
    B = bm25.scores_batch(ind, toks, qi, qt_oracle, 1.2, 0.75)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    for q in range(nq):
        # fp32 sums of up to 130 products of values rounded to fp32: (130 + 2) 2^-24 < 1e-5
        rep = accept.check_ranked(B[q], ids[q], sc[q], k, rtol=1e-5, ranked=B[q] > 0)
        assert rep.ok, (q, rep.problems)


@pytest.mark.parametrize("n", [32767, 32768])
@pytest.mark.parametrize("k", [5, 16, 17, 128])
def test_a_whole_range_of_equal_scores(n, k):
    """Every chunk of a full range (32,768) has the same score, so the count of ties fills its half of
    the packed counts: identical chunks for BM25 and the hybrid, a zero (padding) query without
    matching terms for the weighted search.  The k smallest ids win."""
    dev = device()
    vocab = 4
    csr = synth.csr_from_tokens(np.arange(n + 1, dtype=np.int64) * 2, np.tile(np.array([1, 2], np.int32), n), vocab)
    idx = make_index(torch.zeros((n, 128), dtype=torch.bfloat16), "bf16")

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(dev)

    idx.attach_sparse(t(csr.term_indptr), t(csr.post_chunk), t(csr.post_tf), t(csr.doc_len), 1.2, 0.75)
    q = torch.zeros((3, 128), dtype=torch.bfloat16, device=dev)
    qi = t(np.array([0, 1, 2, 4], np.int32))
    first = np.tile(np.arange(k), (3, 1))
    log("whole range of ties", n, k)
    sc, ids = idx.search_sparse(qi, t(np.array([1, 2, 1, 2], np.int32)), k)
    assert np.array_equal(ids.cpu().numpy(), first)
    assert (sc == sc[:, :1]).all() and (sc > 0).all()
    fused, fids = idx.search_hybrid(q, qi, t(np.array([1, 2, 1, 2], np.int32)), k, k, 60, k)
    assert np.array_equal(fids.cpu().numpy(), first)
    for terms in ([1, 2, 1, 2], [0, 0, 0, 0]):  # constant lexical rows: every fused score is 0
        sc, ids = idx.search_hybrid_weighted(q, qi, t(np.array(terms, np.int32)), 0.5, 0.5, k)
        assert np.array_equal(ids.cpu().numpy(), first)
        assert (sc == 0).all()
    idx.close()
