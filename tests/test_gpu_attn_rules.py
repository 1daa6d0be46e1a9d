"""The launches that a forward pass of 576 / 512 rows is given by their estimated times: one launch for several layers or one each,
splits of what a row can hold, whole prefixes in the dense form, rows behind them.  Sizes on both sides of each rule, against a 64-bit reference."""
import pytest
import torch

import paper_2603_12201_amd as ic
from tests.test_gpu_attn_stream import D_QK, D_V, SCALE, _check, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,L,n,H,k", [
    (1, 1, 100, 3, 32, 2048), (1, 16, 500, 1, 32, 2048), (1, 16, 500, 3, 8, 2048), (4, 16, 300, 1, 32, 2048), (64, 2, 130, 2, 8, 2048),   # splits of held rows
    (1, 60, 60, 4, 32, 2048), (16, 4, 4, 4, 32, 2048), (2, 64, 64, 2, 5, 2048), (4, 70, 70, 4, 5, 2048), (1, 129, 129, 3, 8, 200),        # layers together
    (1, 256, 256, 2, 8, 2048), (1, 300, 300, 1, 32, 2048), (2, 257, 257, 1, 32, 2048), (16, 33, 33, 1, 32, 2048),                         # dense or not
    (2, 300, 400, 1, 16, 350), (1, 400, 400, 2, 32, 390), (4, 90, 290, 1, 32, 250), (1, 700, 800, 1, 4, 120),                             # rows behind
])
def test_forward(B, T, L, n, H, k):
    g = torch.Generator().manual_seed(B * T + L + n)
    layers = []
    for i in range(n):
        t = {"Q": torch.randn((B, T, H, D_QK), generator=g).to(torch.bfloat16).cuda(), "KV": torch.randn((B, L, D_QK), generator=g).to(torch.bfloat16).cuda()}
        if i == 0:
            t["q"] = (torch.randn((B, T, 4, 64), generator=g) / 8).to(torch.bfloat16).cuda()
            t["k"] = torch.randn((B, L, 64), generator=g).to(torch.bfloat16).cuda()
            t["w"] = torch.rand((B, T, 4), generator=g).cuda()
        layers.append(t)
    outs = [torch.full((B, T, H, D_V), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(n)]
    arr = ic.make_layers(layers, k, L - T, D_V, 0, SCALE, outs)
    idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
    ic.forward_stack(arr, [True] + [False] * (n - 1), idx, ws)
    held = torch.arange(L - T, L).clamp_max(k - 1) + 1
    assert torch.equal((idx >= 0).sum(-1).cpu(), held.expand(B, T))
    for t, out in zip(layers, outs):
        _check(out, None, _reference(t["Q"].cpu(), t["KV"].cpu(), idx.cpu()[..., :min(k, L)])[0], None)


def test_more_sequences_than_a_grid_dimension():
    # 65540 sequences of two rows: as many blocks of the dense form, whose numbers times sequences do not fit 32 bits
    B, T, L, H, k = 65540, 2, 2, 32, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    t = {"Q": rnd(B, T, H, D_QK), "KV": rnd(B, L, D_QK), "q": rnd(B, T, 4, 64), "k": rnd(B, L, 64), "w": torch.rand((B, T, 4), generator=g, device="cuda")}
    out = torch.full((B, T, H, D_V), 7.0, dtype=torch.bfloat16, device="cuda")
    arr = ic.make_layers([t], k, 0, D_V, 0, SCALE, [out])
    idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(ic.forward_stack_workspace(arr), 256), dtype=torch.uint8, device="cuda")
    ic.forward_stack(arr, [True], idx, ws)
    some = torch.cat([torch.arange(0, B, 331), torch.arange(B - 40, B)])
    _check(out.cpu()[some], None, _reference(t["Q"].cpu()[some], t["KV"].cpu()[some], idx.cpu()[some][..., :L])[0], None)
