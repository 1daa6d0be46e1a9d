"""Index tensors of the caller's own whose leading rows are whole prefixes (counted on the device, then the dense form and
the rest): where the count ends, what ends it, tails short and long, two sequences with counts of their own, a similarity
matrix of layers with different counts."""
import numpy as np
import pytest
import torch

from tests import parity
import synth

pytestmark = pytest.mark.gpu


def _selection(B, Tq, Lk, k, spoil, seed):
    rng = np.random.default_rng(seed)
    idx = np.full((B, Tq, k), -1, dtype=np.int32)
    for b in range(B):
        for t in range(Tq):
            n = Lk - Tq + t + 1
            idx[b, t, :min(n, k)] = np.arange(n) if n <= k else np.sort(rng.choice(n, k, replace=False))
    for b, t, how in spoil:
        n = Lk - Tq + t + 1
        if how == "swap":
            idx[b, t, [0, n - 1]] = idx[b, t, [n - 1, 0]]
        elif how == "short":
            idx[b, t, n - 1] = -1
        elif how == "long":
            idx[b, t, n] = n if n < Lk else 0
        elif how == "hole":
            idx[b, t, n // 2] = -1
        elif how == "behind":
            idx[b, t, k - 1] = 0
        elif how == "empty":
            idx[b, t] = -1
    return idx


CASES = [
    # B, Tq, Lk, k, H_q, spoiled (sequence, row, how)
    (1, 400, 400, 1024, 32, []),
    (1, 513, 513, 512, 32, []),                                        # one row behind the prefixes
    (1, 700, 700, 512, 32, []),                                        # a short tail
    (1, 900, 900, 512, 32, []),                                        # a long one
    (2, 300, 500, 1024, 32, [(1, 37, "swap")]),                        # behind a prefix, counts 300 and 37
    (1, 400, 400, 1022, 31, [(0, 0, "behind")]),                       # none; k not a multiple of four
    (1, 400, 400, 1024, 32, [(0, 15, "short"), (0, 300, "hole")]),     # last row of a chunk
    (1, 400, 400, 1024, 32, [(0, 16, "long")]),                        # first row of one
    (1, 600, 600, 512, 32, [(0, 320, "empty")]),
    (1, 400, 400, 1024, 32, [(0, 399, "hole")]),                       # the last row
    (1, 400, 400, 1022, 32, [(0, 333, "swap")]),                       # k not a multiple of four, rows counted
    (1, 1100, 1100, 1024, 32, []),                                     # rows behind, split on their own
    (3, 600, 600, 512, 32, [(0, 100, "hole"), (2, 0, "behind")]),      # rows behind go along; counts 100, 512 and 0
    (5, 600, 600, 512, 32, [(4, 200, "short")]),                       # more workgroups than rows left in four of five sequences
]


@pytest.mark.parametrize("case", CASES)
def test_leading_prefix_rows(oracle, case):
    import paper_2603_12201_amd as ic
    B, Tq, Lk, k, H_q, spoil = case
    print("[case] lead B=%d Tq=%d Lk=%d k=%d H_q=%d %s" % case, flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Lk, q_pos0=Lk - Tq, H_q=H_q, k_sel=k, row_elems=576, H_I=4, seed=Tq + k)
    t = synth.attn_layer(cfg, 0)
    idx = _selection(B, Tq, Lk, k, spoil, Tq)
    O, lse = ic.sparse_attn(t["Q"].cuda(), t["KV"].cuda(), torch.from_numpy(idx).cuda(), 512, 0, 1 / 24.0, want_lse=True)
    torch.cuda.synchronize()
    lb = synth.bits_layer(t)
    want, want_lse = oracle.sparse_attn(lb["Q"], lb["KV"], idx, 512, 0, 1 / 24.0)
    parity.check_attn(O.float().cpu().numpy(), want)
    got, ref = lse.cpu().numpy(), np.asarray(want_lse, dtype=np.float64).reshape(lse.shape)
    assert np.array_equal(np.isinf(got), np.isinf(ref))
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() < 1e-3


def test_similarity_of_layers_with_leading_rows(oracle):
    import paper_2603_12201_amd as ic
    B, Tq, k = 2, 600, 512
    print("[case] similarity with leading rows B=%d Tq=%d k=%d" % (B, Tq, k), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Tq, q_pos0=0, H_q=32, k_sel=k, row_elems=576, H_I=4, seed=5)
    spoil = [[], [(1, 100, "hole")], [(0, 0, "empty"), (1, 511, "swap")]]
    layers = [synth.attn_layer(cfg, l) for l in range(3)]
    g = [{n: v.cuda() for n, v in t.items()} for t in layers]
    idx = [torch.from_numpy(_selection(B, Tq, Tq, k, s, 10 + l)).cuda() for l, s in enumerate(spoil)]
    outs = [torch.empty((B, Tq, 32, 512), dtype=torch.bfloat16, device="cuda") for _ in g]
    arr = ic.make_layers(g, k, 0, 512, 0, 1 / 24.0, outs)
    # without room for the counts (3 tensors x 2 sequences x 512 / 16 chunks of 4 bytes) every row is computed
    need = int(ic.lib().ic_similarity_matrix_workspace(arr, 3))
    small = torch.empty(need - 3 * 2 * 32 * 4, dtype=torch.uint8, device="cuda")
    S_all = ic.similarity_matrix(arr, idx, workspace=small).cpu().numpy()
    S = ic.similarity_matrix(arr, idx).cpu().numpy()
    assert np.abs(S - S_all).max() < 2e-4                                  # bf16 outputs of two forms, averaged over 1200 rows
    none = torch.empty(0, dtype=torch.uint8, device="cuda")               # no room for the counts: row by row
    for i in range(3):
        own = ic.sparse_attn(g[i]["Q"], g[i]["KV"], idx[i], 512, 0, 1 / 24.0, workspace=none)
        parity.check_attn(outs[i].float().cpu().numpy(), own.double().cpu().numpy())
        for j in range(i):
            re = ic.sparse_attn(g[i]["Q"], g[i]["KV"], idx[j], 512, 0, 1 / 24.0, workspace=none)
            a, b = own.double().flatten(2), re.double().flatten(2)
            na, nb = a.norm(dim=-1), b.norm(dim=-1)
            cs = torch.where((na == 0) & (nb == 0), torch.ones_like(na), (a * b).sum(-1) / (na * nb).clamp_min(1e-300))
            assert abs(S[i, j] - cs.mean().item()) < 2e-4
        assert S[i, i] == 1.0 and all(S[i, j] == 0.0 for j in range(i + 1, 3))


@pytest.mark.parametrize("B, Tq, k", [(1, 400, 1024), (1, 700, 512), (2, 600, 512)])
def test_a_workspace_that_is_not_needed_is_not_written(oracle, B, Tq, k):
    """Where ic_sparse_attn needs no workspace the caller may be using it elsewhere, on any stream."""
    import ctypes as C
    import paper_2603_12201_amd as ic
    print("[case] unneeded workspace B=%d Tq=%d k=%d" % (B, Tq, k), flush=True)
    cfg = synth.config("c2", B=B, Tq=Tq, Lk=Tq, q_pos0=0, H_q=32, k_sel=k, row_elems=576, H_I=4, seed=Tq + k)
    t = synth.attn_layer(cfg, 0)
    g = {n: v.cuda() for n, v in t.items()}
    host = _selection(B, Tq, Tq, k, [], Tq)
    idx = torch.from_numpy(host).cuda()
    lb = synth.bits_layer(t)
    want, _ = oracle.sparse_attn(lb["Q"], lb["KV"], host, 512, 0, 1 / 24.0)
    ws = torch.full((64 << 20,), 0xA5, dtype=torch.uint8, device="cuda")
    d = ic.AttnDesc(B, Tq, Tq, 32, 576, 512, 0, 576, k, 1 / 24.0)
    L = ic.lib()
    assert L.ic_sparse_attn_workspace(C.byref(d)) == 0
    for where in ("binding", "aligned", "misaligned"):
        out = torch.full((B, Tq, 32, 512), 7.0, dtype=torch.bfloat16, device="cuda")
        if where == "binding":
            ic.sparse_attn(g["Q"], g["KV"], idx, 512, 0, 1 / 24.0, workspace=ws, out=out)
        else:
            p = ws.data_ptr() + (6 if where == "misaligned" else 0)
            st = L.ic_sparse_attn(C.byref(d), g["Q"].data_ptr(), g["KV"].data_ptr(), idx.data_ptr(), out.data_ptr(), None, p,
                                  ws.numel() - 256, torch.cuda.current_stream().cuda_stream)
            assert st == ic.Status.OK
        torch.cuda.synchronize()
        assert bool((ws == 0xA5).all()), where
        parity.check_attn(out.float().cpu().numpy(), want)


@pytest.mark.parametrize("gain", [1.0, 3.0, 6.0])
def test_lse_is_as_exact_as_the_row_forms(gain):
    """Both forms take a score in two accumulation chains of nine steps, so their lse differ from 64-bit sums alike; with one
    chain of eighteen the dense form's distance was 1.05 / 1.27 / 1.45 times the row form's at these gains."""
    import paper_2603_12201_amd as ic
    print("[case] lse gain=%g" % gain, flush=True)
    T, scale = 1024, 1 / 24.0
    gen = torch.Generator(device="cuda").manual_seed(3)
    Q = torch.randn((1, T, 32, 576), generator=gen, device="cuda", dtype=torch.bfloat16) * gain
    KV = torch.randn((1, T, 576), generator=gen, device="cuda", dtype=torch.bfloat16)
    t = torch.arange(T, device="cuda")
    idx = torch.where(t[None, :] <= t[:, None], t[None, :], -1).to(torch.int32)[None].contiguous()
    _, dense = ic.sparse_attn(Q, KV, idx, 512, 0, scale, want_lse=True)
    _, row = ic.sparse_attn(Q, KV, idx, 512, 0, scale, want_lse=True, workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
    K = KV[0].double()
    far = [0.0, 0.0]
    for h in range(0, 32, 4):
        z = (torch.matmul(Q[0, :, h].double(), K.t()) * scale).masked_fill(t[None, :] > t[:, None], float("-inf"))
        want = torch.logsumexp(z, -1)
        for i, got in enumerate((dense, row)):
            far[i] += (got[0, :, h].double() - want).pow(2).sum().item()
    assert not torch.equal(dense, row)                # (two forms, not one twice)
    # 8192 values each: the ratio of two such root mean squares scatters by about 2 %
    assert far[0] ** 0.5 <= 1.08 * far[1] ** 0.5, (far[0] ** 0.5, far[1] ** 0.5)


@pytest.mark.parametrize("B, Tq, Lk, k, taken", [(1, 400, 400, 1022, True), (1, 1100, 1100, 1024, True), (3, 600, 600, 512, True),
                                                 (2, 300, 500, 1024, True), (1, 2060, 2060, 2048, True), (4, 2100, 2100, 2048, True), (1, 32768, 32768, 2048, True),
                                                 (1, 700, 2400, 2048, False), (1, 256, 2048, 2048, False), (1, 600, 600, 512, False)])
def test_shapes_that_look_for_leading_rows(B, Tq, Lk, k, taken):
    """The cases above take the path that they mean to, and shapes with little to gain on causal rows do not."""
    import ctypes as C
    import paper_2603_12201_amd as ic
    d = ic.AttnDesc(B, Tq, Lk, 32, 576, 512, 0, 576, k, 1 / 24.0)
    assert ic.lib().ic_sparse_attn_workspace(C.byref(d)) == 0
    assert (ic.lib().ic_sparse_attn_lead_workspace(C.byref(d)) > 0) == taken


def test_similarity_with_rows_behind_the_prefixes_of_several_sequences(oracle):
    """Few rows behind the candidates in each of three sequences: split over the chip together where the workspace has room,
    whole where it has not; the same similarities."""
    import ctypes as C
    import paper_2603_12201_amd as ic
    B, T, k, n = 3, 1040, 1024, 3
    print("[case] similarity tails B=%d T=%d k=%d" % (B, T, k), flush=True)
    g = torch.Generator(device="cuda").manual_seed(8)
    layers = [{"Q": torch.randn((B, T, 32, 576), generator=g, device="cuda", dtype=torch.bfloat16),
               "KV": torch.randn((B, T, 576), generator=g, device="cuda", dtype=torch.bfloat16)} for _ in range(n)]
    idx = [torch.from_numpy(_selection(B, T, T, k, [(1, 900 + i, "hole")], i)).cuda() for i in range(n)]
    S, O = [], []
    for short in (False, True):
        outs = [torch.full((B, T, 32, 512), 7.0, dtype=torch.bfloat16, device="cuda") for _ in layers]
        arr = ic.make_layers(layers, k, 0, 512, 0, 1 / 24.0, outs)
        need = int(ic.lib().ic_similarity_matrix_workspace(arr, n))
        if short:
            need = B * T * 32 * 512 * 2                # one output
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        s = torch.empty((n, n), dtype=torch.float64, device="cuda")
        ptrs = (C.c_void_p * n)(*[i.data_ptr() for i in idx])
        assert ic.lib().ic_similarity_matrix(arr, n, ptrs, C.c_void_p(s.data_ptr()), C.c_void_p(ws.data_ptr()), need,
                                             C.c_void_p(torch.cuda.current_stream().cuda_stream)) == ic.Status.OK
        torch.cuda.synchronize()
        S.append(s.cpu().numpy())
        O.append([o.float() for o in outs])
    # bf16 outputs of sums in another order: a unit in the last place of a value here and there
    assert np.allclose(S[0], S[1], rtol=0, atol=2e-4), (S[0], S[1])
    for a, b in zip(*O):
        assert ((a - b).norm() / b.norm()).item() < 4e-3
