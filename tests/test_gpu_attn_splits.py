"""Split attention launches (fewer queries than the chip holds workgroups) and their merge, at the edges of the rules
that choose the number of splits: one split, as many as fit one round, more splits than the merge handles side by side or
in one wave."""
import math

import numpy as np
import pytest
import torch

from tests import parity
import synth

pytestmark = pytest.mark.gpu

CASES = [
    # B, Tq, Lk, Hq, d_qk, d_v, v_off, row, k_sel
    (1, 1, 2500, 32, 576, 512, 0, 576, 2200),    # 35 splits of one tile
    (1, 1, 2500, 5, 64, 64, 64, 128, 2200),      # 35 splits, 32 handled side by side
    (40, 1, 700, 32, 576, 512, 0, 576, 640),     # 6 splits of 2 tiles, not 7
    (1, 129, 900, 32, 576, 512, 0, 576, 320),    # one workgroup per query rather than two rounds
    (1, 100, 900, 20, 576, 512, 0, 576, 449),    # two splits, the second one ragged
    (32, 1, 700, 32, 576, 512, 0, 576, 512),     # 8 splits, a wave merges a head
    (25, 1, 700, 31, 576, 512, 0, 576, 576),     # 9 splits, a workgroup does
    (60, 1, 700, 6, 576, 512, 0, 576, 640),      # a last workgroup of two heads
    (1, 300, 400, 3, 64, 64, 64, 128, 130),      # small-tile form, two workgroups per CU
]


@pytest.mark.parametrize("case", CASES)
def test_split_launches(oracle, case):
    import paper_2603_12201_amd as ic
    B, Tq, Lk, Hq, d_qk, d_v, v_off, row, ks = case
    print("[case] splits B=%d Tq=%d Lk=%d Hq=%d d_qk=%d k=%d" % (B, Tq, Lk, Hq, d_qk, ks), flush=True)
    g = torch.Generator().manual_seed(ks + Tq)
    Q = torch.randn((B, Tq, Hq, d_qk), generator=g).to(torch.bfloat16)
    KV = torch.randn((B, Lk, row), generator=g).to(torch.bfloat16)
    rng = np.random.default_rng(ks)
    idx = np.full((B, Tq, ks), -1, dtype=np.int32)
    for b in range(B):
        for t in range(Tq):
            n = ks if t else ks - 70                # a row whose last split holds nothing
            idx[b, t, :n] = np.sort(rng.choice(Lk, size=n, replace=False))
    scale = 1.0 / math.sqrt(d_qk)
    O, lse = ic.sparse_attn(Q.cuda(), KV.cuda(), torch.from_numpy(idx).cuda(), d_v, v_off, scale, want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.sparse_attn(synth.bits(Q), synth.bits(KV), idx, d_v, v_off, scale)
    parity.check_attn(O.float().cpu().numpy(), want)
    assert np.allclose(lse.cpu().numpy(), want_lse, rtol=0, atol=2e-2)


@pytest.mark.parametrize("nq, k", [(60, 2048), (40, 2048), (110, 1030), (3, 2048)])
def test_fewer_splits_are_no_less_exact(nq, k):
    """A query in fewer splits than one layer's launch may have keeps its partials in fp32: as far from 64-bit results as an
    unsplit launch (the same queries several times over), where two bf16 partials were 1.22 times as far.  In as many splits,
    or with the workspace that bf16 partials of those take, there is one more rounding to bf16: at most 2^-9 of a value,
    spread evenly over its binade 0.00166 (rms), so sqrt(whole^2 + 0.00166^2) with 2 % for the sample."""
    import paper_2603_12201_amd as ic
    print("[case] partials nq=%d k=%d" % (nq, k), flush=True)
    g = torch.Generator(device="cuda").manual_seed(nq)
    Lk, scale = 2500, 1 / 24.0
    Q = torch.randn((1, nq, 32, 576), generator=g, device="cuda", dtype=torch.bfloat16)
    KV = torch.randn((1, Lk, 576), generator=g, device="cuda", dtype=torch.bfloat16)
    idx = torch.rand((nq, Lk), generator=g, device="cuda").topk(k, dim=1).indices.sort(dim=1).values.to(torch.int32)[None].contiguous()
    want = torch.stack([torch.softmax((Q[0, t].double() @ KV[0, idx[0, t].long()].double().t()) * scale, -1)
                        @ KV[0, idx[0, t].long(), :512].double() for t in range(nq)])
    far = lambda O: ((O[0, :nq].double() - want).norm() / want.norm()).item()
    run = lambda *a, **kw: ic.sparse_attn(a[0], KV, a[1], 512, 0, scale, **kw)
    rep = -(-256 // nq)
    whole = far(run(Q.repeat(1, rep, 1, 1), idx.repeat(1, rep, 1)))
    tiles = -(-k // 64)
    per = -(-tiles // min(tiles, rep))
    parts = nq * -(-tiles // per)                     # of one layer's launch, in bf16
    least = -(-parts * 32768 // 256) * 256 + -(-parts * 256 // 256) * 256
    split = far(run(Q, idx))
    small = far(run(Q, idx, workspace=torch.empty(least, dtype=torch.uint8, device="cuda")))
    once_more = 1.02 * (whole ** 2 + 0.00166 ** 2) ** 0.5
    assert split <= (once_more if nq == 3 else 1.02 * whole) and small <= once_more, (split, small, whole)   # (3 queries: the 32 splits of before)
