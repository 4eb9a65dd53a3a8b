"""The tiled scoring kernel and its selections at the edges of tiles, query blocks, group sizes and
levels.  Integer-valued vectors give exact scores with many exact ties, so ids and scores must equal
the oracle's exactly (ties by ascending id); no tolerance is involved."""
import numpy as np
import pytest
import torch

import synth
from oracle import dense as od
from tests.gpu_helpers import DT, device, log, make_index

pytestmark = pytest.mark.gpu


def _ints(seed, n, d, nq, spread=2):
    g = np.random.default_rng(seed)
    X = g.integers(-spread, spread + 1, size=(n, d)).astype(np.float32)
    Q = g.integers(-spread, spread + 1, size=(nq, d)).astype(np.float32)
    return X, Q


def _check(X, Q, k, dtype, samp=None):
    dev = device()
    idx = make_index(synth.to_storage(X, dtype), dtype)
    sc, ids = idx.search_dense(synth.to_storage(Q, dtype).to(dev), k)
    torch.cuda.synchronize()
    samp = np.arange(Q.shape[0]) if samp is None else samp
    S = Q[samp].astype(np.float64) @ X.astype(np.float64).T
    ref_ids, ref_sc = od.topk_from_scores(S, k)
    assert np.array_equal(ids.cpu().numpy()[samp], ref_ids)
    assert np.array_equal(sc.cpu().numpy()[samp].astype(np.float64), ref_sc)
    idx.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 384), ("f32", 100), ("f32", 4)])
@pytest.mark.parametrize("n,nq,k", [(1, 1, 1), (127, 16, 5), (129, 17, 16), (255, 64, 3), (257, 65, 8), (511, 128, 16),
                                    (513, 129, 5), (4097, 256, 10), (1000, 257, 128), (8193, 300, 17)])
def test_tile_and_block_edges(dtype, d, n, nq, k):
    log("edges", dtype, d, n, nq, k)
    _check(*_ints(n + nq + k, n, d, nq), k, dtype)


@pytest.mark.parametrize("dtype,d,n,nq,k", [
    # k <= 16 at 2^20 scores (rows of up to 768 bytes): every score, and group maxima past it
    ("bf16", 384, 1024, 1024, 10), ("bf16", 384, 1025, 1024, 10), ("f16", 128, 32_768, 32, 16),
    ("f16", 128, 32_767, 33, 16), ("f32", 4, 16_131, 65, 5), ("f32", 4, 16_132, 65, 5),
    # longer rows: as many times more scores, 6 * 2^20 at most; more than 32,768 rows: group maxima
    ("bf16", 1024, 32_768, 64, 3), ("bf16", 1024, 21_845, 129, 3), ("f32", 3000, 6_000, 1040, 2),
    ("f32", 3000, 6_050, 1040, 2), ("bf16", 128, 32_769, 1, 5), ("bf16", 128, 32_897, 16, 16)])
def test_every_score_or_group_maxima(dtype, d, n, nq, k):
    log("scores or maxima", dtype, d, n, nq, k)
    _check(*_ints(n + nq + k, n, d, nq), k, dtype, samp=np.unique(np.r_[0:min(nq, 4), nq - 1]))


@pytest.mark.parametrize("dtype,d,n,nq,k", [
    # every score and the lanes' maxima: 64 bytes of a row per query, and one query more (group maxima)
    ("bf16", 128, 32_769, 4, 16), ("bf16", 128, 33_003, 5, 5), ("f32", 100, 41_001, 6, 10), ("f32", 100, 41_001, 7, 10),
    ("bf16", 1024, 32_785, 16, 16), ("f16", 256, 65_535, 4, 1),
    # tiles of a chunk times queries 80 and past it (group maxima), on 256 CUs
    ("bf16", 256, 655_360, 4, 5), ("bf16", 256, 655_361, 4, 5), ("f32", 32, 2_621_440, 1, 16),
    ("f32", 32, 2_621_441, 1, 16), ("bf16", 1024, 65_536, 16, 3), ("bf16", 256, 163_001, 3, 1)])
@pytest.mark.parametrize("spread", [1, 2])
def test_few_queries_over_long_indexes(dtype, d, n, nq, k, spread):
    log("few queries", dtype, d, n, nq, k, spread)
    _check(*_ints(n + nq, n, d, nq, spread=spread), k, dtype)


@pytest.mark.parametrize("n,nq", [(40_000, 1), (200_003, 2)])
@pytest.mark.parametrize("case", ["ties", "nan", "few"])
def test_few_queries_with_ties_and_nan(n, nq, case):
    """More rows at the threshold than are ranked at once; NaN rows; fewer than k rows with a number."""
    log("few queries", case, n, nq)
    X, Q = _ints(n, n, 128, nq, spread=3)
    if case == "ties":
        X[n // 3:] = 0
        Q[0] = 0
    else:
        bad = np.random.default_rng(n).permutation(n)[:n // 2 if case == "nan" else n - 3]
        X[bad, 0] = np.nan
        Q[:, 0] = 1
    dev = device()
    idx = make_index(synth.to_storage(X, "bf16"), "bf16")
    sc, ids = idx.search_dense(synth.to_storage(Q, "bf16").to(dev), 16)
    sc2, ids2 = idx.search_dense_noalloc(synth.to_storage(Q, "bf16").to(dev), 16)
    assert torch.equal(ids, ids2) and torch.equal(sc, sc2)
    sc, ids = sc.cpu().numpy().astype(np.float64), ids.cpu().numpy()
    S = Q.astype(np.float64) @ X.astype(np.float64).T
    for i in range(nq):
        rows = np.flatnonzero(~np.isnan(S[i]))
        best = rows[np.lexsort((rows, -S[i][rows]))][:16]
        assert np.array_equal(ids[i][:len(best)], best) and np.array_equal(sc[i][:len(best)], S[i][best])
        assert np.all(ids[i][len(best):] == -1) and np.all(sc[i][len(best):] == -np.inf)
    idx.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 384), ("f32", 100)])
@pytest.mark.parametrize("n,nq,k", [(33_025, 1, 1), (33_151, 16, 5), (33_001, 17, 16), (16_511, 64, 3), (16_385, 65, 8),
                                    (8_321, 128, 16), (8_193, 129, 5), (4_097, 257, 10), (1_153, 1000, 16)])
def test_group_maxima_at_the_edges(dtype, d, n, nq, k):
    log("maxima edges", dtype, d, n, nq, k)
    _check(*_ints(n + nq, n, d, nq), k, dtype, samp=np.unique(np.r_[0:min(nq, 8), nq // 2, nq - 1]))


@pytest.mark.parametrize("n,nq,k", [(400_001, 65, 1), (400_001, 130, 10), (393_217, 300, 16), (40_007, 66, 17),
                                    (300_003, 90, 128), (200_000, 5, 100)])
def test_threshold_levels(n, nq, k):
    """More than 64 queries with k <= 16 past 393,216 rows, and k > 16 past 32,768: group maxima of
    some rows, then one or more filtered levels."""
    log("levels", n, nq, k)
    X, Q = _ints(n + k, n, 128, nq, spread=3)
    _check(X, Q, k, "bf16", samp=np.unique(np.r_[0:min(nq, 8), nq // 2, nq - 1]))


@pytest.mark.parametrize("case", ["ascending", "ties"])
@pytest.mark.parametrize("nq,k", [(70, 5), (300, 16)])
def test_levels_overflow_and_repair(case, nq, k):
    """"ascending": scores grow with the row id, in steps of 1,600 equal ones; "ties": a quarter of the
    rows share the top score, so the buffers overflow, the repair's as well, and the group maxima of the
    whole index answer."""
    log("overflow", case, nq, k)
    n, d = 400_000, 128
    r = np.arange(n)
    X = np.zeros((n, d), np.float32)
    if case == "ascending":
        X[:, 0], X[:, 1] = r // 1600, r % 3  # integers below 256: exact in bf16
    else:
        X[:, 0] = np.random.default_rng(3).integers(0, 4, size=n)
    Q = np.zeros((nq, d), np.float32)
    Q[:, 0] = 4.0
    Q[:, 1] = np.arange(nq) % 2
    _check(X, Q, k, "bf16", samp=np.r_[0:4, nq - 1])


def _overflowed(idx, nq, k):
    """The first flag of the levels' workspace: 0 unless a candidate buffer overflowed (which costs
    another pass over the index).  It lies behind the buffers and the counts, 256-byte aligned."""
    cap = 3072 if k <= 16 else max(4096, 64 * k)
    at = nq * cap * 8 + (nq * 4 + 255) // 256 * 256
    return int(idx._ws[at:at + 4].view(torch.int32).item())


@pytest.mark.parametrize("nq,k", [(70, 10), (300, 16), (1000, 5), (70, 60)])
@pytest.mark.parametrize("run", [1500, 5000, 40_000])
@pytest.mark.parametrize("n", [400_003, 600_000])
def test_levels_over_rows_in_topics(n, run, nq, k):
    """Rows in the order of their topics (runs of similar rows, as documents are ingested): the levels'
    rows are spread over the index, so the thresholds of a query on any topic are close, no buffer
    overflows, and the index is read once."""
    log("topics", n, run, nq, k)
    d = 128
    g = np.random.default_rng(n + run)
    centres = g.integers(-7, 8, size=((n - 1) // run + 1, d)).astype(np.float32)
    X = centres[np.arange(n) // run]
    X += g.integers(-4, 5, size=X.shape, dtype=np.int8)
    Q = centres[g.integers(0, len(centres), size=nq)]
    dev = device()
    idx = make_index(synth.to_storage(X, "bf16"), "bf16")
    sc, ids = idx.search_dense(synth.to_storage(Q, "bf16").to(dev), k)
    assert _overflowed(idx, nq, k) == 0
    samp = np.r_[0:3, nq - 1]
    ref_ids, ref_sc = od.topk_from_scores(Q[samp].astype(np.float64) @ X.astype(np.float64).T, k)
    assert np.array_equal(ids.cpu().numpy()[samp], ref_ids)
    assert np.array_equal(sc.cpu().numpy()[samp].astype(np.float64), ref_sc)
    idx.close()


@pytest.mark.parametrize("nq,k", [(70, 10), (600, 16), (70, 40)])
def test_levels_overflow_where_no_level_looked(nq, k):
    """The best rows, more than a buffer holds, all in 256-row blocks that only the last level has (its
    predecessors take every fourth or eighth) and none of them the first level's: the buffers overflow, and
    the repair finds the rows."""
    log("hidden", nq, k)
    n, d = 400_003, 128
    g = np.random.default_rng(k)
    X = g.integers(-2, 3, size=(n, d)).astype(np.float32)
    X[:, :4] = 0
    r = np.arange(n)
    best = (r // 256 % 8 == 5) & (r % 256 < 60)  # 11,700 rows, their scores in no order of the rows
    rows = n
    while rows > 32_000:
        rows = -(-rows // (8 if k <= 16 else 4))
    for bm in (128, 256):  # the first level's tiles have one of these lengths
        pitch = n // (rows // bm)
        apart = (pitch // bm - 1) | 1  # odd
        best[(np.arange(rows // bm)[:, None] * pitch + np.arange(bm) * apart).ravel()] = False
    X[best, 0] = 64
    X[best, 1] = g.integers(0, 128, size=int(best.sum()))
    X[best, 2] = g.integers(0, 128, size=int(best.sum()))
    Q = np.zeros((nq, d), np.float32)
    Q[:, 0], Q[:, 1], Q[:, 2] = 64, 16, 1
    Q[:, 4:8] = g.integers(-1, 2, size=(nq, 4))
    dev = device()
    idx = make_index(synth.to_storage(X, "bf16"), "bf16")
    sc, ids = idx.search_dense(synth.to_storage(Q, "bf16").to(dev), k)
    assert _overflowed(idx, nq, k) > 0
    samp = np.r_[0:3, nq - 1]
    ref_ids, ref_sc = od.topk_from_scores(Q[samp].astype(np.float64) @ X.astype(np.float64).T, k)
    assert np.array_equal(ids.cpu().numpy()[samp], ref_ids)
    assert np.array_equal(sc.cpu().numpy()[samp].astype(np.float64), ref_sc)
    idx.close()


@pytest.mark.parametrize("n", [3000, 32768, 140_000, 400_000])
@pytest.mark.parametrize("k", [5, 16, 40])
def test_zero_queries_tie_everywhere(n, k):
    """Padding queries of zeros: every row ties, and the k smallest ids win."""
    log("zero queries", n, k)
    X, Q = _ints(n + k, n, 128, 80)
    Q[::2] = 0.0
    _check(X, Q, k, "bf16", samp=np.r_[0:6, 78, 79])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,nq,k", [(700, 3, 5), (5000, 70, 16), (5000, 70, 40), (140_000, 70, 10), (400_000, 70, 10)])
def test_rows_that_score_nan_or_minus_inf(dtype, n, nq, k):
    """A row with a NaN is never returned; one that scores -inf ranks last; one that scores +inf first."""
    log("nan", dtype, n, nq, k)
    X, Q = _ints(n, n, 128, nq)
    Q[:, 0] = 1.0
    X[n // 2, 5] = np.nan
    X[3, 0] = -np.inf
    X[n - 1, 0] = np.inf
    dev = device()
    idx = make_index(synth.to_storage(X, dtype), dtype)
    sc, ids = idx.search_dense(synth.to_storage(Q, dtype).to(dev), k)
    S = Q.astype(np.float64) @ np.nan_to_num(X.astype(np.float64), nan=0.0, posinf=1e6, neginf=-1e6).T
    S[:, n // 2] = -2e6
    ref_ids, _ = od.topk_from_scores(S, k)
    assert np.array_equal(ids.cpu().numpy(), ref_ids)
    assert np.isposinf(sc.cpu().numpy()[:, 0]).all()
    idx.close()


@pytest.mark.parametrize("k", [1, 5, 16])
def test_workspace_of_the_capacity_serves_every_row_count_and_batch(k):
    """One workspace sized for 300 queries and the capacity serves smaller batches and any row count."""
    from paper_2608_08340_amd import OP_DENSE, Index
    dev = device()
    X, Q = _ints(11 + k, 400_000, 128, 300)
    idx = Index(128, 400_000, DT["bf16"])
    ws = idx.workspace(OP_DENSE, 300, k)
    lo = 0
    for n in (100, 33_000, 66_000, 160_000, 393_216, 393_217, 400_000):
        idx.upsert(synth.to_storage(X[lo:n], "bf16").to(dev))
        lo = n
        for nq in (1, 16, 64, 65, 300):
            log("workspace", k, n, nq)
            sc, ids = idx.search_dense(synth.to_storage(Q[:nq], "bf16").to(dev), k)
            assert idx.workspace(OP_DENSE, nq, k).data_ptr() == ws.data_ptr()  # never regrown
            samp = np.unique(np.r_[0, nq - 1])
            ref_ids, _ = od.topk_from_scores(Q[samp].astype(np.float64) @ X[:n].astype(np.float64).T, k)
            assert np.array_equal(ids.cpu().numpy()[samp], ref_ids)
    idx.close()


@pytest.mark.parametrize("dtype,nq,k", [("bf16", 9000, 5), ("bf16", 9000, 16), ("f32", 5000, 40)])
def test_large_batches_run_in_parts(dtype, nq, k):
    """More than 4,096 queries run in equal parts, with a workspace and with the fixed array alike."""
    log("parts", dtype, nq, k)
    dev = device()
    X, Q = _ints(nq + k, 3000, 128, nq)
    idx = make_index(synth.to_storage(X, dtype), dtype)
    q = synth.to_storage(Q, dtype).to(dev)
    sc, ids = idx.search_dense(q, k)
    sc2, ids2 = idx.search_dense_noalloc(q, k)
    samp = np.r_[0:3, nq // 2 - 1:nq // 2 + 2, nq - 3:nq]
    ref_ids, ref_sc = od.topk_from_scores(Q[samp].astype(np.float64) @ X.astype(np.float64).T, k)
    assert np.array_equal(ids.cpu().numpy()[samp], ref_ids)
    assert np.array_equal(sc.cpu().numpy()[samp].astype(np.float64), ref_sc)
    assert torch.equal(ids, ids2) and torch.equal(sc, sc2)
    idx.close()
