"""Query rows that see at most k keys inside forward_stack (the dense attention form), alone and followed by rows with a
real selection: edges of the 64-row blocks and 64-key tiles, head counts, offsets, a page table, logits that move the
softmax reference."""
import pytest
import torch

from tests import parity
import synth

pytestmark = pytest.mark.gpu

CASES = [
    # B, Tq, pos0, H_q, k, row_elems, page, scale
    (1, 16, 0, 32, 64, 576, 0, 1 / 24.0),
    (2, 65, 0, 32, 256, 576, 0, 1 / 24.0),
    (1, 129, 0, 20, 2048, 640, 0, 1 / 24.0),
    (3, 100, 40, 7, 512, 576, 0, 1 / 24.0),
    (1, 200, 0, 1, 300, 576, 0, 1 / 24.0),
    (1, 320, 0, 32, 256, 576, 0, 1 / 24.0),       # 256 dense rows, 64 with a selection
    (2, 300, 0, 16, 130, 576, 0, 1 / 24.0),       # the same for two sequences
    (1, 257, 0, 32, 256, 576, 0, 1 / 24.0),       # one row with a selection
    (5, 70, 200, 32, 256, 576, 0, 1 / 24.0),      # few rows with a selection in each of five sequences: one launch, split
    (9, 90, 200, 32, 256, 576, 0, 1 / 24.0),      # more of them than workgroups: chains over sequences
    (9, 90, 200, 32, 256, 576, 64, 1 / 24.0),     # paged
    (64, 8, 252, 32, 256, 576, 0, 1 / 24.0),      # four and four rows of many sequences
    (2, 190, 0, 32, 256, 576, 64, 1 / 24.0),      # paged
    (2, 150, 0, 32, 128, 576, 64, 1 / 24.0),      # paged, with a selection
    (1, 300, 700, 32, 1100, 576, 0, 1 / 24.0),    # behind a prefix
    (1, 20, 400, 32, 500, 576, 0, 1 / 24.0),      # too few blocks for it
    (1, 150, 0, 32, 256, 576, 0, 2.0),            # scores hundreds apart: the reference moves
]


@pytest.mark.parametrize("case", CASES)
def test_dense_rows(oracle, case):
    import paper_2603_12201_amd as ic
    B, Tq, pos0, H_q, ks, row, page, scale = case
    print("[case] dense B=%d Tq=%d pos0=%d H_q=%d k=%d row=%d page=%d scale=%g" % case, flush=True)
    Lk = pos0 + Tq
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Lk, q_pos0=pos0, H_q=H_q, k_sel=ks, row_elems=row, H_I=4, seed=Tq + H_q)
    t = synth.indexer_layer(cfg, 0)
    t.update(synth.attn_layer(cfg, 0))
    g = {n: v.cuda() for n, v in t.items()}
    out = torch.full((B, Tq, H_q, 512), 7.0, dtype=torch.bfloat16, device="cuda")
    idx = torch.empty((B, Tq, ks), dtype=torch.int32, device="cuda")
    if page:
        n = -(-Lk // page)
        order = torch.randperm(B * n, generator=torch.Generator().manual_seed(1))
        table = order.view(B, n).to(torch.int32)
        for name in ("k", "KV"):
            pool = torch.full((B * n * page, g[name].shape[-1]), 300.0, dtype=torch.bfloat16, device="cuda")
            for b in range(B):
                for p in range(n):
                    src = g[name][b, p * page:(p + 1) * page]
                    pool[int(table[b, p]) * page:int(table[b, p]) * page + src.shape[0]] = src
            g[name] = pool
        pc = ic.paged_cache(page_table=table.cuda(), page_size=page)
    arr = ic.make_layers([g], ks, pos0, 512, 0, scale, [out], Lk=Lk if page else None)
    if page:
        arr[0].ix.q_pos0 = pos0
    ws = torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda")
    if page:
        ic.forward_stack_paged(arr, [True], pc, idx, ws)
    else:
        ic.forward_stack(arr, [True], idx, ws)
    torch.cuda.synchronize()
    lb = synth.bits_layer(t)
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], idx.cpu().numpy(), 512, 0, scale)
    err = parity.check_attn(out.float().cpu().numpy(), want)
    print("max abs err %.3g" % err)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("B, Tq, H_q, row", [(1, 300, 32, 199), (1, 300, 32, 224), (1, 300, 32, 1), (2, 200, 32, 199), (1, 500, 20, 333)])
def test_later_keys_do_not_reach_earlier_rows(bad, B, Tq, H_q, row):
    """One KV row of infinities or NaN: the query rows that do not see it are what they are without it, bit for bit."""
    import paper_2603_12201_amd as ic
    print("[case] dense, row %d of %d is %g, B=%d H_q=%d" % (row, Tq, bad, B, H_q), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Tq, q_pos0=0, H_q=H_q, k_sel=512, row_elems=576, H_I=4, seed=row)
    t = synth.indexer_layer(cfg, 0)
    t.update(synth.attn_layer(cfg, 0))
    g = {n: v.cuda() for n, v in t.items()}
    outs = []
    for spoil in (False, True):
        kv = g["KV"].clone()
        if spoil:
            kv[:, row, 0::2] = bad
        out = torch.empty((B, Tq, H_q, 512), dtype=torch.bfloat16, device="cuda")
        arr = ic.make_layers([dict(g, KV=kv)], 512, 0, 512, 0, 1 / 24.0, [out])
        idx = torch.empty((B, Tq, 512), dtype=torch.int32, device="cuda")
        ic.forward_stack(arr, [True], idx, torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda"))
        outs.append(out.cpu())
    assert torch.equal(outs[0][:, :row].view(torch.int16), outs[1][:, :row].view(torch.int16))
    if bad != bad:
        assert torch.isnan(outs[1][:, row:].float()).all()


@pytest.mark.parametrize("B, Tq, pos0, lk_full, lk_shared, k, page", [
    (1, 120, 0, 100, 120, 2048, 0),               # rows 100 .. 119 select 0 .. 99 only
    (2, 300, 10, 200, 400, 256, 0),               # fewer keys than k, then none of the later rows dense
    (1, 70, 40, 100, 128, 2048, 64),              # paged
])
def test_shared_cache_longer_than_the_full_layers(oracle, B, Tq, pos0, lk_full, lk_shared, k, page):
    """A Shared layer attends to what its Full layer selected, among the Full layer's keys, however long its own cache is."""
    import paper_2603_12201_amd as ic
    print("[case] dense B=%d Tq=%d pos0=%d Lk full %d shared %d k=%d page=%d" % (B, Tq, pos0, lk_full, lk_shared, k, page), flush=True)
    mk = lambda lk, l: synth.config("c2", B=B, Tq=Tq, Lk=lk, q_pos0=pos0, H_q=32, k_sel=k, row_elems=576, H_I=4, seed=3 + l)
    full = synth.indexer_layer(mk(lk_full, 0), 0)
    full.update(synth.attn_layer(mk(lk_full, 0), 0))
    shared = synth.attn_layer(mk(lk_shared, 1), 1)
    want_kv = shared["KV"].clone()
    shared["KV"][:, lk_full:] = 50.0              # nobody selects these
    g = [{n: v.cuda() for n, v in t.items()} for t in (full, shared)]
    outs = [torch.empty((B, Tq, 32, 512), dtype=torch.bfloat16, device="cuda") for _ in g]
    idx = torch.empty((B, Tq, k), dtype=torch.int32, device="cuda")
    pc = None
    if page:
        n = -(-max(lk_full, lk_shared) // page)
        table = torch.arange(B * n, dtype=torch.int32).flip(0).view(B, n)
        for t in g:
            for name in ("k", "KV"):
                if name not in t:
                    continue
                pool = torch.full((B * n * page, t[name].shape[-1]), 50.0, dtype=torch.bfloat16, device="cuda")
                for b in range(B):
                    for p in range(n):
                        src = t[name][b, p * page:(p + 1) * page]
                        pool[int(table[b, p]) * page:int(table[b, p]) * page + src.shape[0]] = src
                t[name] = pool
        pc = ic.paged_cache(page_table=table.cuda(), page_size=page)
    arr = ic.make_layers(g, k, pos0, 512, 0, 1 / 24.0, outs, Lk=lk_full if page else None)
    arr[1].at.Lk = lk_shared
    for a in arr:
        a.ix.q_pos0 = pos0
    ws = torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda")
    if page:
        ic.forward_stack_paged(arr, [True, False], pc, idx, ws)
    else:
        ic.forward_stack(arr, [True, False], idx, ws)
    torch.cuda.synchronize()
    sel = idx.cpu().numpy()
    assert sel.max() == lk_full - 1
    lb = synth.bits_layer(dict(shared, KV=want_kv))
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], sel, 512, 0, 1 / 24.0)
    parity.check_attn(outs[1].float().cpu().numpy(), want)
    lb = synth.bits_layer(full)
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], sel, 512, 0, 1 / 24.0)
    parity.check_attn(outs[0].float().cpu().numpy(), want)


@pytest.mark.parametrize("col", [0, 300, 511, 540])
@pytest.mark.parametrize("B, Tq, H_q, row, page", [(1, 300, 32, 199, 0), (1, 300, 32, 224, 0), (1, 300, 32, 3, 0), (2, 200, 32, 198, 64),
                                                   (1, 500, 20, 333, 0), (1, 100, 1, 70, 0)])
def test_minus_infinity_in_a_key_that_a_row_sees(oracle, B, Tq, H_q, row, page, col):
    """A key whose score is -inf has weight 0 like everywhere else: 0 times its infinite element is NaN in that column of the
    rows that see it (none for an element behind the values), and the other columns are those without the key."""
    import paper_2603_12201_amd as ic
    print("[case] dense, -inf in column %d of row %d, B=%d Tq=%d H_q=%d page=%d" % (col, row, B, Tq, H_q, page), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Tq, q_pos0=0, H_q=H_q, k_sel=512, row_elems=576, H_I=4, seed=row + col)
    t = synth.indexer_layer(cfg, 0)
    t.update(synth.attn_layer(cfg, 0))
    t["Q"][..., col] = 1.0
    want_kv = t["KV"].clone()
    want_kv[:, row] = 0
    t["KV"][:, row, col] = float("-inf")
    g = {n: v.cuda() for n, v in t.items()}
    pc = None
    if page:
        n = -(-Tq // page)
        table = torch.arange(B * n, dtype=torch.int32).flip(0).view(B, n)
        for name in ("k", "KV"):
            pool = torch.full((B * n * page, t[name].shape[-1]), 50.0, dtype=torch.bfloat16, device="cuda")
            for b in range(B):
                for p in range(n):
                    src = g[name][b, p * page:(p + 1) * page]
                    pool[int(table[b, p]) * page:int(table[b, p]) * page + src.shape[0]] = src
            g[name] = pool
        pc = ic.paged_cache(page_table=table.cuda(), page_size=page)
    out = torch.empty((B, Tq, H_q, 512), dtype=torch.bfloat16, device="cuda")
    arr = ic.make_layers([g], 512, 0, 512, 0, 1 / 24.0, [out], Lk=Tq if page else None)
    idx = torch.empty((B, Tq, 512), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda")
    if page:
        ic.forward_stack_paged(arr, [True], pc, idx, ws)
    else:
        ic.forward_stack(arr, [True], idx, ws)
    got = out.float().cpu()
    nan = torch.isnan(got)
    expect = torch.zeros_like(nan)
    if col < 512:
        expect[:, row:, :, col] = True
    assert torch.equal(nan, expect)
    sel = idx.cpu().numpy().copy()
    sel[sel == row] = -1
    lb = synth.bits_layer(dict(t, KV=want_kv))
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], sel, 512, 0, 1 / 24.0)
    want[expect.numpy().reshape(want.shape)] = 0
    got[expect] = 0
    parity.check_attn(got.numpy(), want)


@pytest.mark.parametrize("power", [0, 60, 100])
@pytest.mark.parametrize("jump", [6.0, 40.0, 59.0, 90.0])
def test_large_values_behind_a_rising_score(oracle, jump, power):
    """Scores that rise by 2^jump behind the first tile with values of 2^power: no partial sum leaves the range of fp32."""
    import paper_2603_12201_amd as ic
    B, Tq, H_q, scale = 1, 200, 32, 1.0
    print("[case] dense, scores rise by 2^%g, values of 2^%d" % (jump, power), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Tq, q_pos0=0, H_q=H_q, k_sel=512, row_elems=576, H_I=4, seed=int(jump))
    t = synth.indexer_layer(cfg, 0)
    t.update(synth.attn_layer(cfg, 0))
    t["Q"].zero_()
    t["Q"][..., 575] = 1.0
    t["KV"][..., 575] = torch.linspace(0, 0.5, Tq).to(torch.bfloat16)
    t["KV"][:, 40:, 575] = jump * 0.6931472
    g = {n: v.cuda() for n, v in t.items()}
    g["KV"][..., :512] *= 2.0 ** power
    out = torch.empty((B, Tq, H_q, 512), dtype=torch.bfloat16, device="cuda")
    arr = ic.make_layers([g], 512, 0, 512, 0, scale, [out])
    idx = torch.empty((B, Tq, 512), dtype=torch.int32, device="cuda")
    ic.forward_stack(arr, [True], idx, torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda"))
    got = out.double().cpu() * 2.0 ** -power
    lb = synth.bits_layer(t)
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], idx.cpu().numpy(), 512, 0, scale)
    parity.check_attn(got.float().numpy(), want)


@pytest.mark.parametrize("B, Tq, pos0, k", [(1, 300, 0, 512), (2, 40, 900, 512), (1, 3, 5000, 2048)])
def test_any_output_address(B, Tq, pos0, k):
    """Outputs two bytes past a 16-byte boundary (dense form, splits merged by a wave and by a workgroup): the same, to the order
    of sums, as aligned ones, and nothing beside them is touched."""
    import paper_2603_12201_amd as ic
    print("[case] output address B=%d Tq=%d pos0=%d k=%d" % (B, Tq, pos0, k), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=pos0 + Tq, q_pos0=pos0, H_q=32, k_sel=k, row_elems=576, H_I=4, seed=Tq)
    t = synth.indexer_layer(cfg, 0)
    t.update(synth.attn_layer(cfg, 0))
    g = {n: v.cuda() for n, v in t.items()}
    n = B * Tq * 32 * 512
    outs = []
    for off in (0, 1):
        buf = torch.full((n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
        out = buf[off:off + n].view(B, Tq, 32, 512)
        arr = ic.make_layers([g, g], k, pos0, 512, 0, 1 / 24.0, [out, torch.empty_like(out)])
        idx = torch.empty((B, Tq, k), dtype=torch.int32, device="cuda")
        ws = torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda")
        ic.forward_stack(arr, [True, False], idx, ws)
        torch.cuda.synchronize()
        assert (buf[:off] == 7.0).all() and (buf[off + n:] == 7.0).all()
        outs.append(out.float())
    assert ((outs[0] - outs[1]).norm() / outs[0].norm()).item() < 4e-3


@pytest.mark.parametrize("B, Tq, pos0, k, n, page", [
    (1, 300, 0, 2048, 4, 0), (3, 130, 0, 512, 3, 0), (1, 257, 40, 512, 8, 0), (2, 200, 0, 512, 2, 64),      # every row a whole prefix
    (1, 600, 0, 512, 4, 0), (2, 400, 100, 450, 3, 0), (2, 400, 100, 450, 3, 64),                            # and rows behind them
    (1, 1021, 0, 2048, 3, 0), (1, 1100, 0, 2048, 2, 0), (1, 1600, 0, 2048, 3, 0), (1, 1600, 0, 2048, 3, 64),  # rounds that a layer fills: one, two, three
])
def test_dense_rows_of_several_layers(B, Tq, pos0, k, n, page):
    """Layers that share their dense launch give what each gives alone: a block does not know its neighbours, and the rows behind
    (in other splits, maybe) are bf16 roundings of the same sums."""
    import paper_2603_12201_amd as ic
    print("[case] dense layers B=%d Tq=%d pos0=%d k=%d n=%d page=%d" % (B, Tq, pos0, k, n, page), flush=True)
    H, Lk = 32, pos0 + Tq
    g = torch.Generator(device="cuda").manual_seed(Tq + k)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    pages = -(-Lk // 64)
    cache = (B * pages * 64,) if page else (B, Lk)
    layers = [{"Q": rnd(B, Tq, H, 576), "KV": rnd(*cache, 576)} for _ in range(n)]
    ixr = {"q": rnd(B, Tq, 4, 64), "k": rnd(*cache, 64), "w": torch.rand((B, Tq, 4), generator=g, device="cuda")}
    for t in layers:
        t.update(ixr)
    if page:
        table = torch.randperm(B * pages, generator=torch.Generator().manual_seed(1)).view(B, pages).to(torch.int32).cuda()
        pc = ic.paged_cache(page_table=table, page_size=page)

    def run(some):
        outs = [torch.full((B, Tq, H, 512), 7.0, dtype=torch.bfloat16, device="cuda") for _ in some]
        arr = ic.make_layers(some, k, pos0, 512, 0, 1 / 24.0, outs, Lk=Lk if page else None)
        for l in arr:
            l.ix.q_pos0 = pos0
        ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
        idx = torch.empty((B, Tq, k), dtype=torch.int32, device="cuda")
        mask = [True] + [False] * (len(some) - 1)
        if page:
            ic.forward_stack_paged(arr, mask, pc, idx, ws)
        else:
            ic.forward_stack(arr, mask, idx, ws)
        return outs
    together = run(layers)
    for t, out in zip(layers, together):
        alone = run([t])[0]
        assert torch.isfinite(out.float()).all()
        # two roundings of the same value to bf16 (of outputs below 4: at most 2^-7 apart, twice)
        assert (out.float() - alone.float()).abs().max() <= 2 ** -6


def test_layers_in_front_of_one_whose_output_is_at_an_odd_address():
    """The dense form stores 16 bytes at a time: a layer whose output it cannot store takes the row form, those in front of it do not."""
    import paper_2603_12201_amd as ic
    print("[case] dense layers, the third output at an odd address", flush=True)
    B, Tq, H, k, n = 1, 700, 32, 2048, 4
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    layers = [{"Q": rnd(B, Tq, H, 576), "KV": rnd(B, Tq, 576)} for _ in range(n)]
    ixr = {"q": rnd(B, Tq, 4, 64), "k": rnd(B, Tq, 64), "w": torch.rand((B, Tq, 4), generator=g, device="cuda")}
    for t in layers:
        t.update(ixr)
    size = B * Tq * H * 512

    def run(odd):
        bufs = [torch.full((size + 8,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(n)]
        outs = [b[1 if l == odd else 0:][:size].view(B, Tq, H, 512) for l, b in enumerate(bufs)]
        arr = ic.make_layers(layers, k, 0, 512, 0, 1 / 24.0, outs)
        ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
        ic.forward_stack(arr, [True] + [False] * (n - 1), torch.empty((B, Tq, k), dtype=torch.int32, device="cuda"), ws)
        return outs
    even, odd = run(None), run(2)
    for l in range(2):                            # the same form: bit for bit the same
        assert torch.equal(even[l].view(torch.int16), odd[l].view(torch.int16)), l
    for l in range(2, n):                         # the row form, for the layer behind it as well: two roundings to bf16
        assert ((even[l].float() - odd[l].float()).norm() / even[l].float().norm()).item() < 4e-3
