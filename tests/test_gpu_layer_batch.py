"""Attention of a Full layer and its Shared layers in one launch: the same results as layer by layer, and layers whose
buffers overlap keep their order."""
import math

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _stack(ic, n, B, Tq, Lk, H_q, tiny, ks, seed, alias=False):
    cfg = synth.config("c0" if tiny else "c2", B=B, Tq=Tq, Lk=Lk, q_pos0=Lk - Tq, H_q=H_q, k_sel=ks, seed=seed, n_layers=n)
    layers = [{k: v.cuda() for k, v in l.items()} for l in synth.stack_layers(cfg)]
    outs = [torch.empty((B, Tq, H_q, cfg["d_v"]), dtype=torch.bfloat16, device="cuda") for _ in layers]
    if alias:                                    # layer 1 attends with what layer 0 wrote
        n_q = layers[1]["Q"].numel()
        flat = torch.zeros(max(n_q, outs[0].numel()), dtype=torch.bfloat16, device="cuda")
        flat[:n_q] = layers[1]["Q"].reshape(-1)
        layers[1]["Q"] = flat[:n_q].view(layers[1]["Q"].shape)
        outs[0] = flat[:outs[0].numel()].view(outs[0].shape)
    return cfg, layers, outs


@pytest.mark.parametrize("case", [
    # n, pattern, B, Tq, Lk, H_q, tiny, k, alias
    (4, "FSSS", 2, 1, 1500, 32, False, 700, False),      # splits over all four layers
    (10, "FSSSSSSSSS", 1, 1, 900, 20, False, 300, False),  # more layers than one launch takes
    (4, "FSFS", 1, 256, 256, 4, True, 64, False),        # small-tile form
    (3, "FSS", 1, 300, 700, 32, False, 256, False),      # chained queries of three layers
    (3, "FSS", 2, 2, 1000, 32, False, 256, True),        # overlapping buffers: one layer after the other
])
def test_layers_in_one_launch(case):
    import paper_2603_12201_amd as ic
    n, pattern, B, Tq, Lk, H_q, tiny, ks, alias = case
    print("[case] layer batch %s B=%d Tq=%d Lk=%d H_q=%d" % (pattern, B, Tq, Lk, H_q), flush=True)
    got = []
    for one_by_one in (False, True):
        cfg, layers, outs = _stack(ic, n, B, Tq, Lk, H_q, tiny, ks, 7, alias)
        scale = 1.0 / math.sqrt(cfg["d_qk"])
        idx = torch.empty((B, Tq, ks), dtype=torch.int32, device="cuda")
        if one_by_one:
            for t, o, c in zip(layers, outs, pattern):
                if c == "F":
                    idx = ic.indexer_topk(t["q"], t["k"], t["w"], ks, cfg["q_pos0"])
                ic.sparse_attn(t["Q"], t["KV"], idx, cfg["d_v"], cfg["v_off"], scale, out=o)
        else:
            arr = ic.make_layers(layers, ks, cfg["q_pos0"], cfg["d_v"], cfg["v_off"], scale, outs)
            ws = torch.empty(max(256, ic.forward_stack_workspace(arr)), dtype=torch.uint8, device="cuda")
            ic.forward_stack(arr, [c == "F" for c in pattern], idx, ws)
        torch.cuda.synchronize()
        got.append((idx.clone(), [o.float() for o in outs]))
    assert torch.equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1], got[1][1]):
        assert (a - b).norm() <= 5e-3 * b.norm()         # other splits round a partial differently
