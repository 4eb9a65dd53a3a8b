"""Pooled upserts at the edges of a load set, on the GPU against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import embed_tail
from tests.gpu_helpers import decode, device, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden_dtype,d", [("bf16", 128), ("f32", 1152)])
def test_pooled_upsert_lengths_around_a_load_set(hidden_dtype, d):
    """Token counts around the tokens that eight residues load at once (64 in bf16, 32 in fp32).  Bound:
    2 len 2^-24 sum|h| / ||sum|| for the fp32 sums, against the fp64 oracle."""
    dev = device()
    g = np.random.default_rng(5)
    lengths = np.array([1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 71, 72, 127, 128, 129, 150], dtype=np.int32)
    m, T = len(lengths), 150
    H = torch.from_numpy(g.standard_normal((m, T, d)).astype(np.float32) + 0.3)
    if hidden_dtype == "bf16":
        H = H.to(torch.bfloat16)
    H64 = H.float().numpy().astype(np.float64)
    from paper_2608_08340_amd import Index
    idx = Index(d, m, torch.float32)
    log("pooled lengths", hidden_dtype, d)
    idx.upsert_pooled(H.to(dev), torch.from_numpy(lengths).to(dev))
    torch.cuda.synchronize()
    got = decode(synth.storage_bits(idx.slab[:m].cpu()), "f32")
    ref = embed_tail.pool(H64, lengths)
    for i in range(m):
        n = lengths[i]
        tot = H64[i, :n].sum(axis=0)
        bound = 2 * n * 2.0 ** -24 * np.abs(H64[i, :n]).sum(axis=0) / np.linalg.norm(tot) + 2.0 ** -23
        assert np.all(np.abs(got[i] - ref[i]) <= bound), int(n)
