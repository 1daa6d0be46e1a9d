"""Top-k of rows of up to 32768 keys: lengths around the limits of every instance, with few and with many rows, and scores
that drive a row through every way out (a full boundary bin, bins of a bin, ties cut at any place, infinite scores)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ic():
    import paper_2603_12201_amd as m
    m.lib()
    return m


def check(ic, oracle, q, k, w, ks, p0):
    """The kernel's choice against the oracle's on the kernel's own scores: equal, position for position."""
    idx, sel = ic.indexer_topk(q, k, w, ks, p0, want_scores=True)
    sc = ic.debug_indexer_scores(q, k, w, p0, 0, q.shape[1]).cpu().numpy()
    idx, sel = idx.cpu().numpy(), sel.cpu().numpy()
    for b in range(q.shape[0]):
        for i in range(q.shape[1]):
            n = max(0, min(p0 + i + 1, k.shape[1]))
            if n == 0:
                assert np.all(idx[b, i] == -1)
                continue
            want = oracle.topk_row(sc[b, i], n, ks)["idx"]
            want = np.sort(want[want >= 0])
            assert np.array_equal(idx[b, i][:len(want)], want), (b, i, n)
            assert np.all(idx[b, i][len(want):] == -1)
            assert np.array_equal(sel[b, i][:len(want)], sc[b, i][want])


@pytest.mark.parametrize("L", [1, 5, 511, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 32767, 32768])
@pytest.mark.parametrize("ks", [1, 64, 2048])
def test_lengths(ic, oracle, L, ks):
    print("[case] bins L=%d k=%d" % (L, ks), flush=True)
    T = min(L, 3)
    g = torch.Generator().manual_seed(L + ks)
    q = (torch.randn((1, T, 4, 64), generator=g) / 8).to(torch.bfloat16).cuda()
    k = torch.randn((1, L, 64), generator=g).to(torch.bfloat16).cuda()
    w = torch.randn((1, T, 4), generator=g).cuda()
    check(ic, oracle, q, k, w, ks, L - T)


def test_many_rows(ic, oracle):
    """More rows than the few-row rule of 16384 keys, from a row with one key on."""
    print("[case] bins, 1100 rows of 15000", flush=True)
    g = torch.Generator().manual_seed(8)
    q = (torch.randn((1, 1100, 4, 64), generator=g) / 8).to(torch.bfloat16).cuda()
    k = torch.randn((1, 15000, 64), generator=g).to(torch.bfloat16).cuda()
    w = torch.rand((1, 1100, 4), generator=g).cuda()
    idx = ic.indexer_topk(q, k, w, 300, 13900).cpu().numpy()
    for i in range(0, 1100, 90):
        sc = ic.debug_indexer_scores(q, k, w, 13900, i, 1).cpu().numpy()
        assert np.array_equal(idx[0, i], np.sort(oracle.topk_row(sc[0, 0], 13901 + i, 300)["idx"])), i


@pytest.mark.parametrize("L", [700, 1500, 4000, 7000, 12000, 30000])
@pytest.mark.parametrize("kind", ["rising", "falling", "constant", "two_values", "levels", "outlier", "wide", "signed", "infinite", "lowest"])
def test_score_shapes(ic, oracle, L, kind):
    # one head, one-hot q: the score of a key is w times the key's own feature where that is positive
    print("[case] bins, %s scores, L=%d" % (kind, L), flush=True)
    x = torch.arange(L, dtype=torch.float32)
    g = torch.Generator().manual_seed(L)
    r = torch.rand(L, generator=g)
    inf = float("inf")
    v = {"rising": 1 + x / 64, "falling": 1 + (L - x) / 64, "constant": torch.ones(L), "two_values": 1.0 + (x % 41 == 0).float(),
         "levels": 1.0 + (x % 3), "outlier": 1 + r + (x == L // 2).float() * 1e30, "wide": torch.exp2(200 * r - 100),
         "signed": 1 + r, "infinite": torch.where(x % 50 == 7, torch.tensor(inf), 1 + r), "lowest": torch.where(x % 5 != 0, torch.tensor(inf), 1 + r)}[kind]
    q = torch.zeros((1, 2, 1, 64)); q[..., 5] = 1.0
    k = torch.zeros((1, L, 64)); k[0, :, 5] = v
    w = torch.ones((1, 2, 1))
    if kind in ("signed", "lowest"):           # every score negative, or -inf
        w = -w
    q, k, w = q.to(torch.bfloat16).cuda(), k.to(torch.bfloat16).cuda(), w.cuda()
    for ks in (7, 600):
        check(ic, oracle, q, k, w, ks, L - 2)


@pytest.mark.parametrize("L, ks", [(40, 39), (700, 699), (700, 640), (1030, 1000), (2050, 2048), (2100, 2048)])
@pytest.mark.parametrize("kind", ["rising", "zeros", "low", "first"])
def test_last_key_wanted_lies_in_the_lowest_bin(ic, oracle, L, ks, kind):
    """That bin's members are not counted: few of them, many, as many as are ranked, and slots behind the row that lie in it or do not."""
    print("[case] bins, %s, L=%d k=%d" % (kind, L, ks), flush=True)
    x = torch.arange(L, dtype=torch.float32)
    r = torch.rand(L, generator=torch.Generator().manual_seed(L))
    v = {"rising": 1 + x / 64, "zeros": (r - 0.5).clamp(min=0), "low": 1 + r + 1e4 * (x % 7 == 3), "first": 1 + r + 1e4 * (x == 0)}[kind]
    q = torch.zeros((1, 2, 1, 64)); q[..., 5] = q[..., 6] = 1.0
    k = torch.zeros((1, L, 64)); k[0, :, 5] = v.to(torch.bfloat16).float(); k[0, :, 6] = v - k[0, :, 5]
    check(ic, oracle, q.to(torch.bfloat16).cuda(), k.to(torch.bfloat16).cuda(), torch.ones((1, 2, 1)).cuda(), ks, L - 2)


@pytest.mark.parametrize("L, H", [(700, 1), (700, 40), (1500, 1), (4000, 1), (7000, 1), (12000, 1), (30000, 1)])
@pytest.mark.parametrize("kind", ["few", "many", "all"])
def test_scores_that_are_no_numbers(ic, L, H, kind):
    """They are chosen by their bits, as larger than infinity (sign bit clear) or smaller than -infinity (set): the order of the keys."""
    print("[case] bins, NaN, %s, L=%d H=%d" % (kind, L, H), flush=True)
    x = torch.arange(L)
    r = torch.rand(L, generator=torch.Generator().manual_seed(L))
    hit = {"few": x % (L // 5) == 3, "many": x % 3 == 1, "all": x >= 0}[kind]
    v = torch.where(hit, torch.tensor(float("nan")), 1 + r)
    v = torch.where((x % 97 == 5) & ~hit, torch.tensor(float("inf")), v)
    q = torch.zeros((1, 2, H, 64)); q[:, :, 0, 5] = 1.0
    k = torch.zeros((1, L, 64)); k[0, :, 5] = v
    q, k, w = q.to(torch.bfloat16).cuda(), k.to(torch.bfloat16).cuda(), torch.ones((1, 2, H)).cuda()
    for ks in (7, 600):
        idx, sel = ic.indexer_topk(q, k, w, ks, L - 2, want_scores=True)
        sc = ic.debug_indexer_scores(q, k, w, L - 2, 0, 2).cpu().numpy()
        idx, sel = idx.cpu().numpy(), sel.cpu().numpy()
        for i in range(2):
            u = sc[0, i][:L - 1 + i].view(np.uint32).astype(np.int64)
            keys = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
            want = np.sort(np.argsort(-keys, kind="stable")[:ks])
            assert np.array_equal(idx[0, i], want), (i, ks)
            assert np.array_equal(sel[0, i], sc[0, i][want], equal_nan=True)


@pytest.mark.parametrize("L", [5, 511, 1024, 1025])
@pytest.mark.parametrize("ks", [3, 200])
def test_lengths_of_two_head_tiles(ic, oracle, L, ks):
    """40 heads: scores and selection are launches of their own at any length."""
    print("[case] bins, 40 heads, L=%d k=%d" % (L, ks), flush=True)
    g = torch.Generator().manual_seed(L + ks)
    T = min(L, 3)
    q = (torch.randn((2, T, 40, 64), generator=g) / 8).to(torch.bfloat16).cuda()
    k = torch.randn((2, L, 64), generator=g).to(torch.bfloat16).cuda()
    check(ic, oracle, q, k, torch.randn((2, T, 40), generator=g).cuda(), ks, L - T)


@pytest.mark.parametrize("B, T, L, H, d, p0, ks", [
    (1, 512, 512, 4, 64, 0, 64), (3, 37, 200, 1, 64, 163, 20), (2, 31, 31, 17, 64, -3, 4), (1, 1, 1024, 32, 64, 1023, 1023),
    (1, 5, 1024, 32, 64, 1020, 1024), (2, 9, 512, 32, 128, 503, 100), (1, 300, 300, 20, 128, 0, 33), (1, 511, 512, 31, 128, 0, 511),
    (1, 40, 40, 8, 128, 100, 7), (1023, 1, 1024, 2, 64, 1023, 100),
])
def test_scores_and_selection_in_one_launch(ic, oracle, B, T, L, H, d, p0, ks):
    """Against the scores of the kernel that writes them out: bit for bit the same, so the same choice and the same values."""
    print("[case] short B=%d T=%d L=%d H=%d d=%d p0=%d k=%d" % (B, T, L, H, d, p0, ks), flush=True)
    g = torch.Generator().manual_seed(B + T + L)
    q = (torch.randn((B, T, H, d), generator=g) / d ** 0.5).to(torch.bfloat16).cuda()
    k = torch.randn((B, L, d), generator=g).to(torch.bfloat16).cuda()
    w = torch.randn((B, T, H), generator=g).cuda()
    if B > 100:
        idx = ic.indexer_topk(q, k, w, ks, p0).cpu().numpy()
        sc = ic.debug_indexer_scores(q, k, w, p0, 0, T).cpu().numpy()
        for b in range(0, B, 60):
            assert np.array_equal(idx[b, 0], np.sort(oracle.topk_row(sc[b, 0], L, ks)["idx"])), b
    else:
        check(ic, oracle, q, k, w, ks, p0)


@pytest.mark.parametrize("B, T, L, H, d, two", [
    (1, 1, 1024, 4, 64, 1), (1, 1, 513, 4, 64, 1), (1, 1, 512, 4, 64, 0), (64, 1, 1024, 4, 64, 1), (64, 1, 768, 4, 64, 0), (96, 1, 1024, 4, 64, 0),
    (4, 4, 512, 32, 64, 1), (4, 4, 256, 32, 64, 0), (1, 16, 1024, 32, 64, 1), (1, 16, 768, 32, 64, 0),
    (1, 1, 512, 4, 128, 1), (1, 1, 256, 4, 128, 0), (1, 1, 129, 32, 128, 1), (1, 1, 128, 32, 128, 0), (1, 8, 512, 32, 128, 0),
])
def test_few_rows_take_the_launches_that_are_faster(ic, oracle, B, T, L, H, d, two):
    """Scores and selection of few rows in one launch up to the length where a workgroup per row takes as long as two launches."""
    print("[case] few rows B=%d T=%d L=%d H=%d d=%d" % (B, T, L, H, d), flush=True)
    g = torch.Generator().manual_seed(B + T + L)
    q = (torch.randn((B, T, H, d), generator=g) / d ** 0.5).to(torch.bfloat16).cuda()
    k = torch.randn((B, L, d), generator=g).to(torch.bfloat16).cuda()
    w = torch.randn((B, T, H), generator=g).cuda()
    ic.prof_reset()
    ic.prof_enable(True)
    ic.indexer_topk(q, k, w, 64, L - T)
    torch.cuda.synchronize()
    ic.prof_collect()
    launches = ic.prof_get(0)[0], ic.prof_get(1)[0]
    ic.prof_enable(False)
    ic.prof_reset()
    assert launches == (1, two)
    check(ic, oracle, q[:2], k[:2], w[:2], 64, L - T)


@pytest.mark.parametrize("L, ks", [(32900, 2048), (60001, 100), (131072, 2048)])
def test_more_long_rows_than_workgroups(ic, oracle, L, ks):
    """The candidate form with two rows per CU: rows at random, of one value, and with their best scores together."""
    print("[case] many long rows L=%d k=%d" % (L, ks), flush=True)
    T = 300
    g = torch.Generator().manual_seed(L)
    q = (torch.randn((1, T, 2, 64), generator=g) / 8)
    q[0, 5] = 0                                                             # all scores equal
    q[0, 7] = 0
    q[0, 7, 0, 3] = 1.0                                                     # the score is the key's third feature: one stretch stands out
    k = torch.randn((1, L, 64), generator=g)
    k[0, 20000:23000, 3] = 5 + torch.rand(3000, generator=g)
    q, k, w = q.to(torch.bfloat16).cuda(), k.to(torch.bfloat16).cuda(), torch.rand((1, T, 2), generator=g).cuda()
    idx = ic.indexer_topk(q, k, w, ks, L - T).cpu().numpy()
    for i in (0, 5, 7, 100, 256, 299):
        sc = ic.debug_indexer_scores(q, k, w, L - T, i, 1).cpu().numpy()
        assert np.array_equal(idx[0, i], np.sort(oracle.topk_row(sc[0, 0], L - T + i + 1, ks)["idx"])), i
