"""Attention probabilities of index rows whose entries end early, at the edges of the kernel's groups of 16 and 64 slots."""
import math

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 15, 16, 17, 63, 64, 65, 128, 511, 512, 513]


@pytest.mark.parametrize("k", [64, 70, 513, 1000])
def test_rows_that_end_early(oracle, k):
    import paper_2603_12201_amd as ic
    print("[case] probabilities of short rows, k=%d" % k, flush=True)
    counts = sorted({min(n, k) for n in COUNTS} | {k - 1, k})
    g = torch.Generator().manual_seed(k)
    rng = np.random.default_rng(k)
    Tq, Lk = len(counts) + 1, 1200
    Q = torch.randn((1, Tq, 32, 576), generator=g).to(torch.bfloat16)
    KV = torch.randn((1, Lk, 576), generator=g).to(torch.bfloat16)
    idx = np.full((1, Tq, k), -1, dtype=np.int32)
    for t, n in enumerate(counts):
        idx[0, t, :n] = rng.choice(Lk, n, replace=False)
    idx[0, Tq - 1, k - 1] = 7                             # nothing but the last slot
    scale = 1.0 / math.sqrt(576)
    d = torch.from_numpy(idx).cuda()
    _, lse = ic.sparse_attn(Q.cuda(), KV.cuda(), d, 512, 0, scale, want_lse=True)
    torch.full((1, Tq, k), 9.0, device="cuda")            # what the result's memory may hold
    got = ic.attn_probs(Q.cuda(), KV.cuda(), d, scale, lse).cpu().numpy()
    want = oracle.attn_distribution_selected(synth.bits(Q), synth.bits(KV), idx, scale)
    assert np.abs(got - want).max() <= 2e-3 * want.max() + 1e-6
    assert np.all(got[idx < 0] == 0)
