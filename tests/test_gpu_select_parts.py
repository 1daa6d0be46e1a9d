"""Top-k of few long rows, selected in parts: sizes around the form's limits, ragged rows too short for it, scores that
drive a row through every way out (too few candidates, an overflowing list, ties in the boundary bin)."""
import numpy as np
import pytest
import torch

from tests import parity
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ic():
    import paper_2603_12201_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("case", [
    # B, Tq, Lk, H, d, k
    (1, 1, 65537, 32, 128, 2048),
    (3, 2, 70001, 32, 128, 2048),
    (1, 1, 200003, 32, 128, 2048),
    (1, 2, 150000, 4, 64, 7),
    (64, 1, 66000, 4, 64, 100),
    (66, 1, 131073, 1, 64, 33),
    # parts that are no power of two, whose lists end inside a wave's slots: 36, 17, 42 and 9 of them
    (1, 7, 400000, 2, 64, 2048),
    (3, 5, 450000, 2, 64, 2048),
    (1, 6, 700001, 2, 64, 2048),
    (2, 14, 300000, 2, 64, 2000),
])
def test_rows_in_parts(ic, oracle, case):
    B, Tq, Lk, H, d, ks = case
    print("[case] parts B=%d Tq=%d Lk=%d H=%d k=%d" % (B, Tq, Lk, H, ks), flush=True)
    g = torch.Generator().manual_seed(Lk)
    q = (torch.randn((B, Tq, H, d), generator=g) / d ** 0.5).to(torch.bfloat16)
    k = torch.randn((B, Lk, d), generator=g).to(torch.bfloat16)
    w = torch.rand((B, Tq, H), generator=g)
    idx, sel = ic.indexer_topk(q.cuda(), k.cuda(), w.cuda(), ks, Lk - Tq, want_scores=True)
    got = ic.debug_indexer_scores(q.cuda(), k.cuda(), w.cuda(), Lk - Tq, 0, Tq)
    idx, sel, got = idx.cpu().numpy(), sel.cpu().numpy(), got.cpu().numpy()
    for b in range(0, B, max(1, B // 4)):
        sc = oracle.indexer_scores(synth.bits(q[b:b + 1]), synth.bits(k[b:b + 1]), synth.bits(w[b:b + 1]), Lk - Tq)
        for i in range(Tq):
            parity.check_idx_row(idx[b, i], sc[0, i], Lk - Tq + i + 1, ks, oracle)
            assert np.array_equal(sel[b, i], got[b, i][idx[b, i]])


@pytest.mark.parametrize("kind", ["rising", "falling", "constant", "two_values", "spike"])
def test_score_shapes(ic, oracle, kind):
    # one head, one-hot q: the score of a key is the key's own feature, exact on both sides
    Lk, ks, Tq = 100000, 2048, 2
    print("[case] parts, %s scores" % kind, flush=True)
    x = torch.arange(Lk, dtype=torch.float32)
    v = {"rising": x / 64, "falling": (Lk - x) / 64, "constant": torch.ones(Lk), "two_values": 1.0 + (x % 41 == 0).float(),
         "spike": (x % 97 == 3).float() * (1 + x / Lk) + (x == 12345).float() * 1e30}[kind]
    q = torch.zeros((1, Tq, 1, 64)); q[..., 5] = 1.0
    k = torch.zeros((1, Lk, 64)); k[0, :, 5] = v
    w = torch.ones((1, Tq, 1))
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    idx = ic.indexer_topk(q.cuda(), k.cuda(), w.cuda(), ks, Lk - Tq).cpu().numpy()
    sc = oracle.indexer_scores(synth.bits(q), synth.bits(k), synth.bits(w), Lk - Tq)
    for i in range(Tq):
        parity.check_idx_row(idx[0, i], sc[0, i], Lk - Tq + i + 1, ks, oracle)


def test_ragged_rows(ic, oracle):
    lens, Lk, ks = [80000, 8191, 3000, 50, 0, 66000, 9000, 79999], 80000, 512
    B = len(lens)
    print("[case] parts, ragged", flush=True)
    g = torch.Generator().manual_seed(4)
    q = (torch.randn((B, 1, 8, 128), generator=g) / 11.3).to(torch.bfloat16)
    k = torch.randn((B, Lk, 128), generator=g).to(torch.bfloat16)
    w = torch.rand((B, 1, 8), generator=g)
    pc = ic.paged_cache(seq_lens=torch.tensor(lens, dtype=torch.int32).cuda())
    idx = ic.indexer_topk_paged(q.cuda(), k.cuda(), w.cuda(), ks, Lk, pc).cpu().numpy()
    for b, n in enumerate(lens):
        if n == 0:
            assert np.all(idx[b] == -1)
            continue
        sc = oracle.indexer_scores(synth.bits(q[b:b + 1]), synth.bits(k[b:b + 1, :n].contiguous()), synth.bits(w[b:b + 1]), n - 1)
        parity.check_idx_row(idx[b, 0], sc[0, 0], n, ks, oracle)


@pytest.mark.parametrize("ks, Lk, pos0", [(2048, 1052000, 1051999), (16, 1700000, 1568767), (2048, 1200000, 90000)])
def test_rows_about_as_long_as_the_candidates_allow(ic, oracle, ks, Lk, pos0):
    """Rows beyond what the candidate lists hold, about as long as that, and a short row of a long cache."""
    print("[case] parts, k=%d Lk=%d pos0=%d" % (ks, Lk, pos0), flush=True)
    g = torch.Generator().manual_seed(ks)
    q = (torch.randn((1, 1, 2, 64), generator=g) / 8).to(torch.bfloat16)
    k = torch.randn((1, Lk, 64), generator=g).to(torch.bfloat16)
    w = torch.rand((1, 1, 2), generator=g)
    idx = ic.indexer_topk(q.cuda(), k.cuda(), w.cuda(), ks, pos0).cpu().numpy()
    n = pos0 + 1
    sc = oracle.indexer_scores(synth.bits(q), synth.bits(k[:, :n].contiguous()), synth.bits(w), pos0)
    parity.check_idx_row(idx[0, 0], sc[0, 0], n, ks, oracle)


@pytest.mark.parametrize("Lk, run", [(100000, 2500), (300000, 5000), (1100000, 3000)])
def test_best_keys_that_lie_together(ic, oracle, Lk, run):
    """The best scores in one stretch of the row (what a query that looks at its neighbourhood selects), across a part's and the
    bitmap's limits, with ties inside."""
    print("[case] parts, best keys together, Lk=%d" % Lk, flush=True)
    for at in (0, Lk - run, min(Lk, 1 << 20) - run // 2):
        at = min(at, Lk - run)
        v = torch.rand(Lk, generator=torch.Generator().manual_seed(Lk + at))
        v[at:at + run] += 4
        q = torch.zeros((1, 1, 1, 64)); q[..., 5] = 1.0
        k = torch.zeros((1, Lk, 64)); k[0, :, 5] = v
        q, k, w = q.to(torch.bfloat16), k.to(torch.bfloat16), torch.ones((1, 1, 1))
        idx = ic.indexer_topk(q.cuda(), k.cuda(), w.cuda(), 2000, Lk - 1).cpu().numpy()
        sc = k[0, :, 5].double().numpy()
        assert np.array_equal(idx[0, 0], np.sort(oracle.topk_row(sc, Lk, 2000)["idx"]))
