"""Group maxima over long indexes: chunks of more than 32 tiles, groups that span several tiles, and the
search without a workspace.  Integer-valued vectors of few dimensions give exact scores, so ids and
scores must equal the oracle's exactly (ties by ascending id); no tolerance is involved."""
import numpy as np
import pytest
import torch

from oracle import dense as od
from tests.gpu_helpers import DT, device, log

pytestmark = pytest.mark.gpu


def _index(seed, n, d, nq, dtype, spread):
    from paper_2608_08340_amd import Index
    dev = device()
    g = torch.Generator(device=dev).manual_seed(seed)
    X = torch.randint(-spread, spread + 1, (n, d), generator=g, device=dev).to(DT[dtype])
    Q = torch.randint(-spread, spread + 1, (nq, d), generator=g, device=dev).to(DT[dtype])
    idx = Index(d, n, DT[dtype])
    idx.upsert(X)
    return idx, X, Q


def _check(X, Q, k, sc, ids, samp):
    """samp: the queries compared with the oracle."""
    Xd = X.double().cpu().numpy()
    S = Q[samp].double().cpu().numpy() @ Xd.T
    ref_ids, ref_sc = od.topk_from_scores(S, k)
    assert np.array_equal(ids[samp].cpu().numpy(), ref_ids)
    assert np.array_equal(sc[samp].double().cpu().numpy(), ref_sc)


# spread 2: hundreds of thousands of rows tie; 100: next to none do
@pytest.mark.parametrize("spread", [2, 100])
@pytest.mark.parametrize("dtype,d,n,nq,k", [
    ("bf16", 128, 1_100_003, 16, 10),   # one tile a group, chunks of 34 tiles
    ("f32", 8, 1_500_001, 3, 5),        # the same with 46 tiles
    ("f32", 4, 1_999_999, 13, 16),      # groups of two tiles
    ("f32", 4, 3_000_001, 13, 16),      # the same, more than 32 of them a chunk
    ("f32", 4, 9_000_129, 16, 10),      # of eight
    ("f32", 4, 2_000_000, 63, 10),      # 64-query tiles, groups of two tiles
    ("f32", 4, 9_000_129, 64, 10),      # of sixteen
])
def test_groups_over_long_indexes(dtype, d, n, nq, k, spread):
    log("long", dtype, d, n, nq, k, spread)
    if dtype == "bf16":
        spread = min(spread, 7)  # exact products and sums
    idx, X, Q = _index(n + nq, n, d, nq, dtype, spread)
    sc, ids = idx.search_dense(Q, k)
    sc2, ids2 = idx.search_dense_noalloc(Q, k)
    assert torch.equal(ids, ids2) and torch.equal(sc, sc2)
    _check(X, Q, k, sc, ids, [0, nq - 1])
    idx.close()


@pytest.mark.parametrize("nq", [1, 64, 65])
def test_without_a_workspace_past_33_million_rows(nq):
    """One 4-row group's maximum per query and four bytes of it would take more than the fixed array."""
    n, k = 40_000_000, 10
    log("noalloc long", nq)
    idx, X, Q = _index(nq, n, 4, nq, "f32", 1000)
    sc, ids = idx.search_dense_noalloc(Q, k)
    sc2, ids2 = idx.search_dense(Q, k)
    assert torch.equal(ids, ids2) and torch.equal(sc, sc2)
    _check(X, Q, k, sc, ids, [nq - 1])
    idx.close()


def test_without_a_workspace_more_than_2_to_20_queries():
    """Calls of any batch up to 2^20 queries' worth of 8 bytes per result stay accepted, and past it those
    that were: k = 4 and 2^20 + 5 queries.  One more result each is refused, with nothing enqueued."""
    nq, k = (1 << 20) + 5, 4
    log("noalloc large batch")
    idx, X, Q = _index(5, 300, 4, nq, "f32", 100)
    sc, ids = idx.search_dense_noalloc(Q, k)
    _check(X, Q, k, sc, ids, [0, 4095, 4096, nq // 2, nq - 1])
    from paper_2608_08340_amd import OpragError
    with pytest.raises(OpragError, match="one call"):
        idx.search_dense_noalloc(Q, k + 1)
    idx.close()


@pytest.mark.parametrize("n,nq,k", [(33_000, 70, 17), (150_001, 70, 40), (150_001, 3, 100)])
def test_fp32_levels(n, nq, k):
    """fp32 with k > 16 past 32,768 rows: threshold levels."""
    log("fp32 levels", n, nq, k)
    idx, X, Q = _index(n + k, n, 8, nq, "f32", 50)
    sc, ids = idx.search_dense(Q, k)
    _check(X, Q, k, sc, ids, [0, nq // 2, nq - 1])
    idx.close()


@pytest.mark.parametrize("dtype,d,n,nq,k", [("bf16", 128, 5_000, 4, 5),       # every score
                                            ("bf16", 128, 50_003, 2, 10),     # every score and the lanes' maxima
                                            ("f32", 8, 300_000, 33, 10),      # group maxima
                                            ("bf16", 128, 400_100, 70, 10),   # levels
                                            ("f16", 128, 40_001, 3, 40)])
def test_captured_search_replays_on_new_queries(dtype, d, n, nq, k):
    """One capture, several replays on other queries with eager searches between them."""
    log("capture", dtype, d, n, nq, k)
    idx, X, Q = _index(n + k, n, d, nq, dtype, 7)
    q = Q.clone()
    out = (torch.empty((nq, k), device=q.device), torch.empty((nq, k), dtype=torch.int64, device=q.device))
    idx.search_dense(q, k, out=out)  # the workspace exists before the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        idx.search_dense(q, k, out=out)
    for r in range(4):
        q.copy_(Q.roll(r, 0) * (1 if r % 2 else -1))
        out[0].fill_(7.0)
        out[1].fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        sc, ids = out[0].clone(), out[1].clone()
        esc, eids = idx.search_dense(q, k)
        assert torch.equal(ids, eids) and torch.equal(sc, esc)
        _check(X, q, k, sc, ids, [0, nq - 1])
    idx.close()
