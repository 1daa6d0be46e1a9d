"""Indexer scores of problems too small for a workgroup per 512 keys (their keys are dealt out in chunks of 64 up to 512), against
64-bit scores: around the sizes where the chunk changes, ragged ends, both dtypes, rows whose first positions see nothing."""
import ctypes

import pytest
import torch

import paper_2603_12201_amd as ic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,L,H,d,k,fp8", [
    (1, 5, 70, 4, 64, 8, False), (1, 64, 64, 4, 64, 16, False), (1, 200, 200, 4, 64, 64, False), (2, 513, 513, 32, 64, 64, False),
    (1, 1025, 1025, 4, 64, 64, False), (1, 33, 3001, 32, 128, 300, False), (1, 65, 5000, 32, 128, 256, False),
    (2, 31, 1500, 20, 128, 100, False), (1, 40, 2000, 64, 128, 128, True), (1, 300, 700, 32, 128, 96, True), (1, 17, 900, 40, 128, 64, False),
    (1, 600, 600, 64, 128, 64, False), (2, 700, 700, 64, 128, 64, False), (1, 1100, 1100, 64, 128, 64, False), (1, 9, 3000, 64, 128, 64, False),
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


@pytest.mark.parametrize("B,T,L,H,page,low", [
    (1, 1, 40, 32, 0, 40), (2, 1, 6000, 32, 64, 0), (3, 2, 2100, 20, 64, 1), (5, 4, 900, 64, 0, 0), (17, 1, 3000, 32, 128, 1), (40, 1, 4096, 32, 64, 30),
    (65, 1, 257, 32, 0, 0), (70, 2, 128, 40, 64, 0), (130, 1, 320, 32, 64, 0), (33, 1, 2050, 32, 0, 2050),
    # lengths that allow windows of whole sequences (one, two to eight a window, the last ones fewer) and lengths that do not; more
    # places than lanes and than two waves' worth of them
    (2, 1, 20000, 64, 0, 19000), (2, 1, 20000, 32, 64, 0), (15, 1, 3000, 40, 0, 2900), (16, 1, 9000, 32, 64, 8900), (12, 1, 9000, 64, 0, 0),
    (40, 1, 1500, 64, 64, 1450), (30, 3, 700, 32, 0, 690), (64, 2, 600, 64, 64, 590), (100, 1, 900, 32, 0, 880), (43, 3, 300, 32, 64, 290),
    (300, 2, 96, 32, 0, 0),
])
def test_ragged_shares(B, T, L, H, page, low):
    # decode rows whose slots of 32 keys are shared out to windows and waves across sequences: empty and one-key sequences, more
    # tokens than a wave has lanes, fewer slots than waves, several tokens in one wave; every score that a token sees is checked
    g = torch.Generator().manual_seed(B + L)
    d, k = 128, min(L, 2048)
    q = (torch.randn((B, T, H, d), generator=g) / d ** 0.5).to(torch.bfloat16)
    kk, w = torch.randn((B, L, d), generator=g).to(torch.bfloat16), torch.rand((B, T, H), generator=g)
    lens = torch.randint(low, L + 1, (B,), generator=g)
    lens[B // 2] = L
    cache, table = kk, None
    if page:
        per = -(-L // page)
        order = torch.randperm(B * per, generator=g)
        table = order.view(B, per).to(torch.int32)
        cache = torch.full((B * per, page, d), 3e4, dtype=torch.bfloat16)
        padded = torch.cat([kk, torch.zeros((B, per * page - L, d), dtype=torch.bfloat16)], 1).view(B * per, page, d)
        cache[order] = padded
        cache = cache.view(B * per * page, d)
    pc = ic.paged_cache(lens.to(torch.int32).cuda(), table.cuda() if page else None, page)
    idx, sel = ic.indexer_topk_paged(q.cuda(), cache.cuda(), w.cuda(), k, L, pc, want_scores=True)
    idx, sel = idx.cpu().long(), sel.cpu().double()
    s = torch.matmul(q.double().view(B, T * H, d), kk.double().transpose(1, 2).contiguous()).view(B, T, H, L)
    s = (torch.relu(s) * w.double()[..., None]).sum(2)
    seen = torch.arange(L)[None, None, :] < (lens[:, None, None] - T + torch.arange(T)[None, :, None] + 1)
    s = s.masked_fill(~seen, -float("inf"))
    valid, n_seen = idx >= 0, seen.sum(-1)
    assert torch.equal(valid.sum(-1), n_seen.clamp_max(k))
    assert bool(seen.gather(2, idx.clamp_min(0))[valid].all())
    # 128 products and 64 terms at most summed in fp32: 2^-24 * sqrt(192) of the largest score, ten times that
    tol = 1e-5 * s.max().item()
    at = s.gather(2, idx.clamp_min(0))
    assert not bool(valid.any()) or (at - sel)[valid].abs().max().item() < tol
    low = at.masked_fill(~valid, float("inf")).min(dim=-1).values
    assert bool((low >= s.topk(k, dim=-1).values[..., -1] - tol).all())
    full = (n_seen <= k)[..., None] & (torch.arange(k) < n_seen[..., None])       # whatever a token sees: all of it, in order
    assert torch.equal(idx[full], torch.arange(k).expand_as(idx)[full])


@pytest.mark.parametrize("B,T,L,H,k", [
    (1, 1, 100, 64, 20), (3, 2, 3001, 64, 200), (2, 3, 1090, 32, 100), (5, 4, 640, 40, 64), (2, 2, 65, 32, 30), (1, 1, 9000, 20, 512),
    (40, 3, 700, 64, 128), (1, 2, 40000, 64, 1024), (7, 4, 2500, 20, 300),
])
def test_fp8_decode_rows(B, T, L, H, k):
    # few rows per sequence, in pairs where there are several: odd counts, both head counts, one chunk to many, ragged tiles.  Whole
    # numbers, and powers of two as weights and scales: every sum is below 2^24 and exact, so the scores are those of 64 bits
    g = torch.Generator().manual_seed(B * T + L)
    d = 128
    q, kk = torch.randint(-3, 4, (B, T, H, d), generator=g).float(), torch.randint(-3, 4, (B, L, d), generator=g).float()
    two = lambda *shape: 2.0 ** torch.randint(-1, 2, shape, generator=g)
    w, qs, ks = two(B, T, H), two(B, T), two(B, L)
    f8 = torch.float8_e4m3fn
    idx, sel = ic.indexer_topk(q.to(f8).cuda(), kk.to(f8).cuda(), w.cuda(), k, L - T, qs.cuda(), ks.cuda(), want_scores=True)
    idx, sel = idx.cpu().long(), sel.cpu().double()
    s = torch.matmul(q.double().view(B, T * H, d), kk.double().transpose(1, 2).contiguous()).view(B, T, H, L)
    s = (torch.relu(s) * w.double()[..., None]).sum(2) * qs.double()[..., None] * ks.double()[:, None, :]
    s = s.masked_fill(torch.arange(L)[None, :] > torch.arange(T)[:, None] + L - T, -float("inf"))
    valid = idx >= 0
    assert torch.equal(valid.sum(-1), (torch.arange(T) + L - T + 1).clamp_max(k).expand(B, T))
    at = s.gather(2, idx.clamp_min(0))
    assert torch.equal(at[valid], sel[valid])
    assert torch.equal(at.masked_fill(~valid, float("inf")).min(dim=-1).values, s.topk(k, dim=-1).values.masked_fill(~valid, float("inf")).min(dim=-1).values)


@pytest.mark.parametrize("B,T,L,H,k", [
    (1, 1, 9000, 64, 500), (1, 3, 9000, 64, 500), (2, 4, 6000, 32, 300), (13, 1, 3000, 32, 200), (15, 3, 2000, 64, 150), (16, 2, 2000, 20, 150),
    (17, 1, 2500, 64, 200), (33, 4, 500, 32, 64), (85, 3, 200, 40, 32), (200, 4, 150, 32, 20),
])
def test_windows_of_whole_tokens(B, T, L, H, k):
    # decode rows of one length: as many whole tokens for every window (fewer than 16, 16 and several times that) or shares of them
    # all.  Whole numbers and powers of two as above: the scores are those of 64 bits
    g = torch.Generator().manual_seed(B * T + L)
    d = 128
    q, kk = torch.randint(-3, 4, (B, T, H, d), generator=g).float(), torch.randint(-3, 4, (B, L, d), generator=g).float()
    w = 2.0 ** torch.randint(-1, 2, (B, T, H), generator=g)
    idx, sel = ic.indexer_topk(q.to(torch.bfloat16).cuda(), kk.to(torch.bfloat16).cuda(), w.cuda(), k, L - T, want_scores=True)
    idx, sel = idx.cpu().long(), sel.cpu().double()
    s = torch.matmul(q.double().view(B, T * H, d), kk.double().transpose(1, 2).contiguous()).view(B, T, H, L)
    s = (torch.relu(s) * w.double()[..., None]).sum(2)
    s = s.masked_fill(torch.arange(L)[None, :] > torch.arange(T)[:, None] + L - T, -float("inf"))
    assert bool((idx >= 0).all())
    at = s.gather(2, idx)
    assert torch.equal(at, sel)
    assert torch.equal(at.min(dim=-1).values, s.topk(k, dim=-1).values[..., -1])


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("H", [32, 64])
def test_fp8_ragged_rows(T, H):
    # fp8 rows of ragged sequences (no page table): empty ones, fewer keys than rows, ends off a tile, the full length.  Exact as above
    lens = torch.tensor([0, 1, max(T - 1, 0), T, 63, 64, 65, 130, 700, 1001, 2048], dtype=torch.int32)
    B, L, d, k = len(lens), 2048, 128, 100
    g = torch.Generator().manual_seed(T * H)
    q, kk = torch.randint(-3, 4, (B, T, H, d), generator=g).float(), torch.randint(-3, 4, (B, L, d), generator=g).float()
    two = lambda *shape: 2.0 ** torch.randint(-1, 2, shape, generator=g)
    w, qs, ks = two(B, T, H), two(B, T), two(B, L)
    f8 = torch.float8_e4m3fn
    qd, kd, wd, qsd, ksd, ld = q.to(f8).cuda(), kk.to(f8).cuda(), w.cuda(), qs.cuda(), ks.cuda(), lens.cuda()
    desc = ic.IndexerDesc(B, T, L, H, d, k, 0, 1, 0, qsd.data_ptr(), ksd.data_ptr())
    pc = ic.paged_cache(ld)
    ws = torch.empty(ic.indexer_topk_workspace(desc), dtype=torch.uint8, device="cuda")
    idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    sel = torch.empty((B, T, k), dtype=torch.float32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert ic.lib().ic_indexer_topk_paged(ctypes.byref(desc), ctypes.byref(pc), p(qd), p(kd), p(wd), p(idx), p(sel), p(ws), ws.numel(),
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    idx, sel = idx.cpu().long(), sel.cpu().double()
    s = torch.matmul(q.double().view(B, T * H, d), kk.double().transpose(1, 2).contiguous()).view(B, T, H, L)
    s = (torch.relu(s) * w.double()[..., None]).sum(2) * qs.double()[..., None] * ks.double()[:, None, :]
    n_seen = (lens[:, None].long() - T + 1 + torch.arange(T)[None, :]).clamp_min(0)
    s = s.masked_fill(torch.arange(L) >= n_seen[..., None], -float("inf"))
    valid = idx >= 0
    assert torch.equal(valid.sum(-1), n_seen.clamp_max(k))
    at = s.gather(2, idx.clamp_min(0))
    assert torch.equal(at[valid], sel[valid])
    low = at.masked_fill(~valid, float("inf")).min(dim=-1).values
    assert torch.equal(low, s.topk(k, dim=-1).values.masked_fill(~valid, float("inf")).min(dim=-1).values)


@pytest.mark.parametrize("B,T,L,H,d,fp8,low,q0", [
    # one workgroup a CU: rows that see about the same keys (448 and 512 keys a workgroup), the last chunk hidden from half of the blocks
    (8, 64, 2000, 32, 128, 0, None, None), (4, 200, 1000, 64, 128, 1, None, None), (4, 200, 1000, 64, 64, 0, None, None), (1, 300, 2000, 64, 128, 1, None, None),
    # two a CU: triangles, and more than one a CU at 512 keys (16 x 17 rows)
    (1, 1024, 1024, 64, 128, 1, None, None), (3, 600, 600, 32, 128, 0, None, None), (16, 17, 3000, 64, 64, 0, None, None), (1, 701, 701, 64, 128, 1, None, None),
    (4, 201, 1001, 32, 128, 1, None, None), (2, 701, 701, 4, 64, 0, None, None), (1, 5, 40000, 4, 64, 0, None, None),
    # neither
    (5, 700, 700, 64, 128, 1, None, None),
    # more rows than keys: the first see nothing; keys behind the last row
    (2, 300, 170, 32, 128, 1, None, None), (2, 90, 900, 32, 128, 0, None, 64),
    # ragged lengths, whose visible keys the host does not know
    (8, 64, 2000, 32, 128, 0, 500, None), (16, 60, 1000, 32, 128, 0, 0, None), (8, 64, 2000, 64, 128, 0, 0, None), (3, 130, 700, 64, 128, 1, 0, None),
])
def test_workgroups_per_cu(B, T, L, H, d, fp8, low, q0):
    # whole numbers and powers of two: every sum is exact, so every score is
    g = torch.Generator().manual_seed(B * T + L)
    q, kk = torch.randint(-2, 3, (B, T, H, d), generator=g).float(), torch.randint(-2, 3, (B, L, d), generator=g).float()
    w = 2.0 ** torch.randint(-1, 2, (B, T, H), generator=g)
    k, dtype = min(L, 40), torch.float8_e4m3fn if fp8 else torch.bfloat16
    qd, kd, wd = q.to(dtype).cuda(), kk.to(dtype).cuda(), w.cuda()
    one = (torch.ones((B, T)).cuda(), torch.ones((B, L)).cuda()) if fp8 else (None, None)
    if low is None:
        q0 = L - T if q0 is None else q0
        idx, sel = ic.indexer_topk(qd, kd, wd, k, q0, *one, want_scores=True)
        n_seen = (torch.arange(T) + q0 + 1).clamp(0, L).expand(B, T)
    else:
        lens = torch.randint(low, L + 1, (B,), generator=g)
        lens[0], lens[B // 2] = low, L
        pc = ic.paged_cache(lens.to(torch.int32).cuda())
        desc = ic.IndexerDesc(B, T, L, H, d, k, 0, 1 if fp8 else 0, 0, one[0].data_ptr() if fp8 else None, one[1].data_ptr() if fp8 else None)
        ws = torch.empty(ic.indexer_topk_workspace(desc), dtype=torch.uint8, device="cuda")
        idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
        sel = torch.empty((B, T, k), dtype=torch.float32, device="cuda")
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        assert ic.lib().ic_indexer_topk_paged(ctypes.byref(desc), ctypes.byref(pc), p(qd), p(kd), p(wd), p(idx), p(sel), p(ws), ws.numel(),
                                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        n_seen = (lens[:, None] - T + 1 + torch.arange(T)[None, :]).clamp_min(0)
    idx, sel = idx.cpu().long(), sel.cpu()
    for b in range(B):
        s = torch.zeros((T, L))
        for h in range(H):
            s += w[b, :, h, None] * torch.relu(q[b, :, h] @ kk[b].T)
        s = s.masked_fill(torch.arange(L) >= n_seen[b][:, None], -float("inf"))
        valid = idx[b] >= 0
        assert torch.equal(valid.sum(-1), n_seen[b].clamp_max(k))
        at = s.gather(1, idx[b].clamp_min(0))
        assert torch.equal(at[valid], sel[b][valid])
        top = s.topk(k, dim=-1).values
        assert torch.equal(at.masked_fill(~valid, float("inf")).min(-1).values, top.masked_fill(~valid, float("inf")).min(-1).values)
        once = idx[b].masked_fill(~valid, 0).sort(-1).values                     # no key twice
        assert bool(((once[:, 1:] > once[:, :-1]) | (once[:, 1:] == 0)).all())
