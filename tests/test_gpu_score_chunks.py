"""Indexer scores of problems too small for a workgroup per 512 keys (their keys are dealt out in chunks of 64 up to 512), against
64-bit scores: around the sizes where the chunk changes, ragged ends, both dtypes, rows whose first positions see nothing."""
import pytest
import torch

import paper_2603_12201_amd as ic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,L,H,d,k,fp8", [
    (1, 5, 70, 4, 64, 8, False), (1, 64, 64, 4, 64, 16, False), (1, 200, 200, 4, 64, 64, False), (2, 513, 513, 32, 64, 64, False),
    (1, 1025, 1025, 4, 64, 64, False), (1, 33, 3001, 32, 128, 300, False), (1, 65, 5000, 32, 128, 256, False),
    (2, 31, 1500, 20, 128, 100, False), (1, 40, 2000, 64, 128, 128, True), (1, 300, 700, 32, 128, 96, True), (1, 17, 900, 40, 128, 64, False),
])
def test_chunks(B, T, L, H, d, k, fp8):
    g = torch.Generator().manual_seed(T + L)
    q, kk, w = torch.randn((B, T, H, d), generator=g) / d ** 0.5, torch.randn((B, L, d), generator=g), torch.rand((B, T, H), generator=g)
    qs, ks = torch.ones((B, T)), torch.ones((B, L))
    if fp8:
        qs, ks = torch.rand((B, T), generator=g) + 0.5, torch.rand((B, L), generator=g) + 0.5
        q, kk = (q * 8).to(torch.float8_e4m3fn), kk.to(torch.float8_e4m3fn)
    else:
        q, kk = q.to(torch.bfloat16), kk.to(torch.bfloat16)
    args = (qs.cuda(), ks.cuda()) if fp8 else (None, None)
    idx, sel = ic.indexer_topk(q.cuda(), kk.cuda(), w.cuda(), k, L - T, *args, want_scores=True)
    idx, sel = idx.cpu().long(), sel.cpu().double()
    for b in range(B):
        s = torch.zeros((T, L), dtype=torch.float64)
        for h in range(H):
            s += w[b, :, h, None].double() * torch.relu(q[b, :, h].double() @ kk[b].double().T)
        s *= qs[b].double()[:, None] * ks[b].double()[None, :]
        s = s.masked_fill(torch.arange(L)[None, :] > torch.arange(T)[:, None] + L - T, -float("inf"))
        # d products and H terms summed in fp32: 2^-24 * sqrt(d + H) of the largest scores, ten times that
        tol = 1e-5 * s[torch.isfinite(s)].abs().max().item()
        valid = idx[b] >= 0
        assert torch.equal(valid.sum(-1), (torch.arange(T) + L - T + 1).clamp_max(k))
        at = s.gather(1, idx[b].clamp_min(0))
        assert (at - sel[b])[valid].abs().max().item() < tol
        kth = s.topk(min(k, L), dim=1).values[:, -1]
        low = at.masked_fill(~valid, float("inf")).min(dim=1).values
        assert bool((low >= kth - tol).all())
