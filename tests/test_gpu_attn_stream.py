"""Unsplit sparse attention of 576 / 512 rows against a 64-bit reference at the sizes where its streams of rows can go
wrong: selections of one entry to a few granules and their remainders, query counts around the number of workgroups (chains of
one, two and unequal lengths), few heads, empty slots and rows, ragged and paged caches, outputs at any address, several layers."""
import pytest
import torch

import paper_2603_12201_amd as ic

pytestmark = pytest.mark.gpu
D_QK, D_V, SCALE = 576, 512, 1.0 / 24.0


def _case(B, T, L, H, k, seed, holes):
    g = torch.Generator().manual_seed(seed)
    Q = torch.randn((B, T, H, D_QK), generator=g).to(torch.bfloat16)
    KV = torch.randn((B, L, D_QK), generator=g).to(torch.bfloat16)
    idx = torch.rand((B, T, L), generator=g).topk(k, dim=-1).indices.sort(dim=-1).values.to(torch.int32)
    if holes:                                # empty slots anywhere, and some rows without any entry
        idx[torch.rand((B, T, k), generator=g) < 0.3] = -1
        idx[:, ::7] = -1
    return Q, KV, idx


def _reference(Q, KV, idx):
    rows, valid = idx.clamp_min(0).long(), idx >= 0
    O, lse = [], []
    for b in range(Q.shape[0]):
        kv = KV[b].double()[rows[b]]                                             # [T, k, 576]
        s = torch.matmul(Q[b].double(), kv.transpose(1, 2).contiguous()) * SCALE   # [T, H, k]
        s = s.masked_fill(~valid[b][:, None, :], -float("inf"))
        l = torch.logsumexp(s, dim=-1)
        p = torch.exp(s - l.clamp_min(-1e300)[..., None]).nan_to_num(0.0)
        O.append(torch.matmul(p, kv[..., :D_V].contiguous()))
        lse.append(l)
    return torch.stack(O), torch.stack(lse)


def _check(O, lse, ref_O, ref_lse):
    # the probabilities and the output are rounded to bf16 once each: 2^-9 of a value at the worst, 2^-9 / sqrt(3) on average for
    # either, 0.0016 together; 0.004 leaves room for the few entries of the short selections
    assert ((O.double().cpu() - ref_O).norm() / ref_O.norm()).item() < 4e-3
    if lse is not None:
        full = torch.isfinite(ref_lse)
        assert torch.equal(torch.isfinite(lse.cpu()), full)
        # 576 products of unit values scaled by 1 / 24, summed in fp32: 2^-24 * sqrt(576) of a score's size of 1 each, ten times that
        assert (lse.double().cpu()[full] - ref_lse[full]).abs().max().item() < 2e-5


@pytest.mark.parametrize("k", [1, 31, 32, 33, 63, 64, 65, 96, 129])
@pytest.mark.parametrize("T,H,holes", [(257, 32, False), (300, 5, True), (515, 32, True), (1024, 17, False)])
def test_sizes(k, T, H, holes):
    Q, KV, idx = _case(1, T, 200, H, k, seed=k + T, holes=holes)
    O, lse = ic.sparse_attn(Q.cuda(), KV.cuda(), idx.cuda(), D_V, 0, SCALE, want_lse=True)
    _check(O, lse, *_reference(Q, KV, idx))


@pytest.mark.parametrize("shift", [1, 4])
def test_output_address(shift):
    B, T, H, k = 2, 260, 3, 70
    Q, KV, idx = _case(B, T, 150, H, k, seed=5, holes=True)
    buf = torch.full((B * T * H * D_V + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    O = buf[shift:shift + B * T * H * D_V].view(B, T, H, D_V)
    ic.sparse_attn(Q.cuda(), KV.cuda(), idx.cuda(), D_V, 0, SCALE, out=O)
    _check(O, None, *_reference(Q, KV, idx))
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + B * T * H * D_V:] == 7).all())


@pytest.mark.parametrize("k", [40, 300])
def test_large_scores_and_moving_reference(k):
    # scores that grow along the selection: the reference moves in most granules, the last of which decide the row
    Q, KV, idx = _case(1, 270, 400, 32, k, seed=11, holes=False)
    KV *= torch.linspace(0.05, 4.0, 400)[None, :, None].to(torch.bfloat16)
    Q *= 6
    O, _ = ic.sparse_attn(Q.cuda(), KV.cuda(), idx.cuda(), D_V, 0, SCALE, want_lse=True)
    ref, _ = _reference(Q, KV, idx)
    # two roundings of relative size 2^-9 each, and one of them again where a reference moves: of the largest term, at most
    assert ((O.double().cpu() - ref).norm() / ref.norm()).item() < 8e-3


@pytest.mark.parametrize("page", [0, 64])
def test_ragged_paged(page):
    B, T, H, k, L = 70, 4, 8, 100, 256
    Q, KV, idx = _case(B, T, L, H, k, seed=3, holes=False)
    g = torch.Generator().manual_seed(1)
    lens = torch.randint(0, L + 1, (B,), generator=g)
    lens[0], lens[1] = 0, L
    seen = idx.clone()
    seen[idx >= lens[:, None, None]] = -1
    if page:
        per = L // page
        order = torch.randperm(B * per, generator=g)
        pool = torch.full((B * per * page, D_QK), 3e4, dtype=torch.bfloat16)
        table = order.view(B, per).to(torch.int32)
        for b in range(B):
            for j in range(-(-int(lens[b]) // page)):
                n = min(page, int(lens[b]) - j * page)
                pool[int(table[b, j]) * page:int(table[b, j]) * page + n] = KV[b, j * page:j * page + n]
        pool[:1] = KV[1, :1]                 # (an empty slot reads row 0, whose values have to be finite)
        if int(order[0]) >= 0:
            owner = int((order == 0).nonzero()[0])
            if int(lens[owner // per]) > (owner % per) * page:
                pool[:1] = KV[owner // per, (owner % per) * page:(owner % per) * page + 1]
        pc = ic.paged_cache(lens.to(torch.int32).cuda(), table.cuda(), page)
        O = ic.sparse_attn_paged(Q.cuda(), pool.cuda(), idx.cuda(), L, D_V, 0, SCALE, pc)
    else:
        pc = ic.paged_cache(lens.to(torch.int32).cuda(), None, 0)
        O = ic.sparse_attn_paged(Q.cuda(), KV.cuda(), idx.cuda(), L, D_V, 0, SCALE, pc)
    O = O[0] if isinstance(O, tuple) else O
    ref, _ = _reference(Q, KV, seen)
    _check(O, None, ref, None)


def test_layers_and_short_causal_rows():
    # three layers behind one index tensor; the first rows of a sequence hold fewer entries than k
    B, T, H, k, n = 2, 150, 32, 96, 3
    g = torch.Generator().manual_seed(9)
    layers = []
    for i in range(n):
        t = {"Q": torch.randn((B, T, H, D_QK), generator=g).to(torch.bfloat16).cuda(),
             "KV": torch.randn((B, T, D_QK), generator=g).to(torch.bfloat16).cuda()}
        if i == 0:
            t["q"] = (torch.randn((B, T, 32, 128), generator=g) / 11).to(torch.bfloat16).cuda()
            t["k"] = torch.randn((B, T, 128), generator=g).to(torch.bfloat16).cuda()
            t["w"] = torch.rand((B, T, 32), generator=g).cuda()
        layers.append(t)
    flat = torch.zeros((n, B * T * H * D_V + 8), dtype=torch.bfloat16, device="cuda")
    # (outputs two bytes off 16 keep the dense form out of it)
    outs = [flat[i, 1:1 + B * T * H * D_V].view(B, T, H, D_V) for i in range(n)]
    arr = ic.make_layers(layers, k, 0, D_V, 0, SCALE, outs)
    idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
    ic.forward_stack(arr, [True, False, False], idx, ws)
    for t, out in zip(layers, outs):
        ref, _ = _reference(t["Q"].cpu(), t["KV"].cpu(), idx.cpu())
        _check(out, None, ref, None)


@pytest.mark.parametrize("k", [1, 31, 32, 33, 64, 100, 1030])
@pytest.mark.parametrize("B,T,H", [(1, 1, 32), (3, 3, 5), (1, 257, 32), (2, 300, 17)])
def test_probs(k, B, T, H):
    # chains of one to three queries, the second in reverse; rows without entries, with entries in front only and anywhere
    Q, KV, idx = _case(B, T, max(200, k), H, k, seed=k + T, holes=k != 64)
    idx[:, 1::3, (k + 1) // 2:] = -1
    ref_O, ref_lse = _reference(Q, KV, idx)
    lse = ref_lse.float().cuda()
    got = ic.attn_probs(Q.cuda(), KV.cuda(), idx.cuda(), SCALE, lse).double().cpu()
    rows, valid = idx.clamp_min(0).long(), idx >= 0
    for b in range(B):
        s = torch.matmul(Q[b].double(), KV[b].double()[rows[b]].transpose(1, 2).contiguous()) * SCALE
        p = torch.exp(s - ref_lse[b].clamp_min(-1e300)[..., None]).masked_fill(~valid[b][:, None, :], 0.0).mean(dim=1)
        # scores to 2^-24 * sqrt(576) as above and lse rounded to 2^-24 of about 8: 2e-6 of a probability of at most 1, five times that
        assert (got[b] - p).abs().max().item() < 1e-5
        assert bool((got[b][~valid[b]] == 0).all())


@pytest.mark.parametrize("B,T,H,broken", [(1, 1100, 32, ()), (2, 900, 20, (300,)), (3, 700, 32, (650, 1)), (5, 520, 17, (0, 519, 64, 65))])
def test_prefix_rows_in_chains(B, T, H, broken):
    # whole prefixes: more blocks of 64 (query, head) rows than workgroups, so that a workgroup walks several; from a sequence's
    # broken row on (two entries swapped) its rows are not counted and their blocks leave gaps in the chains
    g = torch.Generator().manual_seed(T)
    Q = torch.randn((B, T, H, D_QK), generator=g).to(torch.bfloat16)
    KV = torch.randn((B, T, D_QK), generator=g).to(torch.bfloat16)
    pos = torch.arange(T, dtype=torch.int32)
    idx = torch.where(pos[None, :] <= pos[:, None], pos[None, :], torch.tensor(-1, dtype=torch.int32)).repeat(B, 1, 1)
    for b, t in enumerate(broken):
        if t > 0:
            idx[b, t, :2] = torch.tensor([1, 0], dtype=torch.int32)
        else:
            idx[b, 0, :2] = torch.tensor([-1, 0], dtype=torch.int32)
    O, lse = ic.sparse_attn(Q.cuda(), KV.cuda(), idx.cuda(), D_V, 0, SCALE, want_lse=True)
    ref_O, ref_lse = [], []
    mask = pos[None, :] <= pos[:, None]
    for b in range(B):
        kv = KV[b].double()
        s = torch.einsum("thd,sd->ths", Q[b].double(), kv) * SCALE
        s = s.masked_fill(~mask[:, None, :], -float("inf"))
        ref_lse.append(torch.logsumexp(s, dim=-1))
        ref_O.append(torch.einsum("ths,sd->thd", torch.softmax(s, dim=-1), kv[:, :D_V]))
    _check(O, lse, torch.stack(ref_O), torch.stack(ref_lse))


@pytest.mark.parametrize("page", [0, 64])
def test_negative_length_holds_nothing(page):
    # a length below zero is that of an empty sequence: no id of it counts, and nothing is read behind it
    B, H, k, L = 300, 8, 40, 128
    Q, KV, idx = _case(B, 1, L, H, k, seed=13, holes=False)
    lens = torch.full((B,), L, dtype=torch.int32)
    lens[::3] = -5
    lens[1::3] = 60
    lens[6] = -2 ** 31
    seen = idx.clone()
    seen[idx >= lens[:, None, None]] = -1
    table = torch.arange(B * (L // 64), dtype=torch.int32).view(B, L // 64).cuda() if page else None
    pc = ic.paged_cache(lens.cuda(), table, page)
    O, lse = ic.sparse_attn_paged(Q.cuda(), (KV.view(B * L, D_QK) if page else KV).cuda(), idx.cuda(), L, D_V, 0, SCALE, pc, want_lse=True)
    _check(O, lse, *_reference(Q, KV, seen))
    assert bool((O[::3] == 0).all())


@pytest.mark.parametrize("H", [5, 16, 32])
def test_probs_of_infinite_lse(H):
    # exp(s - inf) is 0 for a finite score and NaN for an infinite one, for every head there is
    Q, KV, idx = _case(1, 6, 100, H, 50, seed=H, holes=False)
    Q[..., 0] = 1.0
    KV[0, 7, 0] = float("inf")
    KV[0, 8, 0] = -float("inf")
    lse = torch.zeros((1, 6, H), dtype=torch.float32)
    lse[:, 1] = float("inf")
    lse[:, 2, H - 1] = float("inf")
    lse[:, 3, 0] = -float("inf")
    lse[:, 4, 0] = float("nan")
    lse[:, 5] = 10.0
    got = ic.attn_probs(Q.cuda(), KV.cuda(), idx.cuda(), SCALE, lse.cuda()).double().cpu()
    s = torch.matmul(Q[0].double(), KV[0].double()[idx[0].long()].transpose(1, 2).contiguous()) * SCALE
    p = torch.exp(s - lse[0].double()[..., None]).mean(dim=1)
    assert torch.equal(torch.isnan(got[0]), torch.isnan(p)) and torch.equal(torch.isinf(got[0]), torch.isinf(p))
    fin = torch.isfinite(p)
    # scores to 1e-6 (see above), so probabilities to 1e-6 of themselves, ten times that
    assert ((got[0] - p)[fin].abs() <= 1e-5 * p[fin].abs() + 1e-30).all()


@pytest.mark.parametrize("k", [1, 16, 63, 64, 65, 128, 129, 192])
@pytest.mark.parametrize("B,T,H,page", [(1, 1, 32, 0), (3, 21, 5, 0), (256, 1, 32, 0), (2, 129, 17, 0), (64, 1, 32, 64), (65, 1, 8, 64), (16, 16, 20, -1)])
def test_short_selections_of_resident_queries(k, B, T, H, page):
    # up to a query per CU and up to three tiles of 64: row-slab form or stream (one query more; a tile more).  page -1: ragged only
    L = 256
    Q, KV, idx = _case(B, T, L, H, k, seed=B + k, holes=k % 2 == 1 and T > 1)   # (holes: row 0 is empty)
    Qd, KVd, idxd, seen = Q.cuda(), KV.cuda(), idx.cuda(), idx
    if page == 0:
        O, lse = ic.sparse_attn(Qd, KVd, idxd, D_V, 0, SCALE, want_lse=True)
    else:
        lens = torch.randint(-1, L + 1, (B,), generator=torch.Generator().manual_seed(k)).to(torch.int32)
        table = torch.arange(B * (L // 64), dtype=torch.int32).view(B, L // 64).cuda() if page > 0 else None
        pc = ic.paged_cache(lens.cuda(), table, max(page, 0))
        O, lse = ic.sparse_attn_paged(Qd, KVd.view(B * L, D_QK) if page > 0 else KVd, idxd, L, D_V, 0, SCALE, pc, want_lse=True)
        seen = torch.where(idx >= lens[:, None, None], torch.tensor(-1, dtype=torch.int32), idx)
    _check(O, lse, *_reference(Q, KV, seen))


def test_short_selections_of_several_layers_at_any_address():
    # decode of three layers behind one index tensor in one launch, outputs two bytes off 16
    B, H, k, n, L = 40, 32, 64, 3, 300
    g = torch.Generator().manual_seed(21)
    layers = []
    for i in range(n):
        t = {"Q": torch.randn((B, 1, H, D_QK), generator=g).to(torch.bfloat16).cuda(), "KV": torch.randn((B, L, D_QK), generator=g).to(torch.bfloat16).cuda()}
        if i == 0:
            t["q"] = (torch.randn((B, 1, 32, 128), generator=g) / 11).to(torch.bfloat16).cuda()
            t["k"] = torch.randn((B, L, 128), generator=g).to(torch.bfloat16).cuda()
            t["w"] = torch.rand((B, 1, 32), generator=g).cuda()
        layers.append(t)
    flat = torch.full((n, B * H * D_V + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    outs = [flat[i, 1:1 + B * H * D_V].view(B, 1, H, D_V) for i in range(n)]
    arr = ic.make_layers(layers, k, L - 1, D_V, 0, SCALE, outs)
    idx = torch.empty((B, 1, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
    ic.forward_stack(arr, [True, False, False], idx, ws)
    for t, out in zip(layers, outs):
        _check(out, None, _reference(t["Q"].cpu(), t["KV"].cpu(), idx.cpu())[0], None)
    assert bool((flat[:, :1] == 7).all()) and bool((flat[:, 1 + B * H * D_V:] == 7).all())


@pytest.mark.parametrize("k", [40, 130])
@pytest.mark.parametrize("T,H", [(300, 32), (530, 7)])
def test_infinities_and_nan_stay_where_they_belong(T, H, k):
    # a NaN or +inf score makes its row NaN, a score of -inf leaves NaN in the columns in which the key is not finite; other heads, other
    # queries and what follows in the same workgroup see nothing of it
    L = 400
    Q, KV, idx = _case(1, T, L, H, k, seed=T + k, holes=True)
    Q[..., 570] = 1.0
    Q[:, 3::50, :, 570] = -1.0
    KV[0, 11, 570] = float("inf")                        # (a feature that is no value)
    KV[0, 12, 570] = -float("inf")
    KV[0, 13, 5] = float("nan")
    KV[0, 14, 7], KV[0, 14, 570] = float("inf"), -float("inf")
    Q[0, 20, H - 1, 3] = float("nan")
    Q[0, 21, 0, 3] = float("inf")
    Q[..., 7] = Q[..., 7].abs().clamp_min(0.1)           # (KV[14] scores -inf + inf = NaN for Q[570] = 1, +inf for -1)
    O, _ = ic.sparse_attn(Q.cuda(), KV.cuda(), idx.cuda(), D_V, 0, SCALE, want_lse=True)
    O = O.double().cpu()[0]
    rows, valid = idx[0].clamp_min(0).long(), idx[0] >= 0
    kv = KV[0].double()[rows]
    s = torch.einsum("thd,tkd->thk", Q[0].double(), kv) * SCALE
    s = s.masked_fill(~valid[:, None, :], -float("inf"))
    m = s.amax(-1, keepdim=True)
    p = torch.exp(s - torch.where(m == -float("inf"), torch.zeros_like(m), m)).masked_fill(~valid[:, None, :], 0.0)
    ref = torch.einsum("thk,tkd->thd", p, torch.where(valid[..., None], kv[..., :D_V], torch.zeros((), dtype=torch.float64)))
    l = p.sum(-1, keepdim=True)
    ref = torch.where(l > 0, ref / l, ref)
    assert torch.equal(torch.isnan(O), torch.isnan(ref)) and not bool(torch.isinf(O).any())
    fin = torch.isfinite(ref)
    assert 0 < int((~fin).sum()) < fin.numel() // 2
    assert ((O - ref)[fin].norm() / ref[fin].norm()).item() < 4e-3       # (as in _check)
