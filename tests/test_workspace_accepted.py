"""Workspaces that are enough for one layer at a time stay accepted where more would only make a call faster.  Host only:
a later argument error shows that a call got past its workspace check, and nothing is launched."""
import ctypes as C

import pytest


def _layers(n, Tq, Lk, k):
    import paper_2603_12201_amd as ic
    arr = (ic.Layer * n)()
    for l in range(n):
        arr[l].ix = ic.IndexerDesc(B=1, Tq=Tq, Lk=Lk, H_I=32, d_I=128, k_sel=k, q_pos0=Lk - Tq, dtype=0, flags=0, q_scale=None, k_scale=None)
        arr[l].at = ic.AttnDesc(B=1, Tq=Tq, Lk=Lk, H_q=32, d_qk=576, d_v=512, v_off=0, row_elems=576, k_sel=k, sm_scale=0.04)
        arr[l].q = arr[l].k = arr[l].w = arr[l].Q = arr[l].KV = arr[l].O = 4096
    return ic, arr


def _up(x):
    return (x + 255) // 256 * 256


def _bf16_partials(nq, k, H=32):
    """One layer's attention with its partials in bf16: as many splits of whole tiles as bring nq queries up to 256."""
    tiles = -(-k // 64)
    per = -(-tiles // min(tiles, -(-256 // nq)))
    parts = nq * -(-tiles // per)
    return 0 if nq >= 256 or per == tiles else _up(parts * H * 512 * 2) + _up(parts * H * 8)


@pytest.mark.parametrize("nq", [1, 12, 40, 100, 200, 255, 256])
def test_attention_with_bf16_partials_is_enough(nq):
    """The query asks for fp32 partials where a query is split in fewer; what the least took before is still accepted."""
    import paper_2603_12201_amd as ic
    L, S = ic.lib(), ic.Status
    one, k = C.c_void_p(4096), 2048
    d = ic.AttnDesc(nq, 1, 5000, 32, 576, 512, 0, 576, k, 1 / 24.0)
    least = _bf16_partials(nq, k)
    assert L.ic_sparse_attn_workspace(C.byref(d)) >= least and (L.ic_sparse_attn_workspace(C.byref(d)) > 0) == (least > 0)
    if least:
        assert L.ic_sparse_attn(C.byref(d), one, one, one, one, None, one, least - 256, None) == S.ERR_WORKSPACE


@pytest.mark.parametrize("n, Tq, Lk, k", [(4, 1, 10007, 2048), (3, 2, 100000, 2048), (8, 40, 5000, 2048), (2, 300, 4000, 512)])
def test_pattern_loss_and_greedy_search_need_one_layer(n, Tq, Lk, k):
    ic, arr = _layers(n, Tq, Lk, k)
    L, S = ic.lib(), ic.Status
    one, refs, buf = C.c_void_p(4096), (C.c_void_p * n)(*([8192] * n)), C.create_string_buffer(n)
    # one layer's attention, or the scores of every row (fewer than 64 MB here)
    attn = _bf16_partials(Tq, k)
    assert attn <= L.ic_sparse_attn_workspace(C.byref(arr[0].at))
    strip = Tq * _up(4 * Lk)
    need = _up(max(attn, strip)) + _up(8 * n) + 256
    assert strip < 64 << 20 and need <= L.ic_pattern_loss_workspace(arr, n)
    bad_mask = bytes([0] + [1] * (n - 1))                                # refused behind the workspace check
    loss = lambda b: L.ic_pattern_loss(arr, n, bad_mask, refs, one, one, one, b, None)
    assert loss(need) == S.ERR_PATTERN
    assert loss(need - 256) == S.ERR_WORKSPACE
    greedy = lambda b: L.ic_greedy_search_forward(arr, n, n, 1, refs, one, buf, None, None, one, b, None)   # n Shared layers: one too many
    assert greedy(need + _up(8 * n)) == S.ERR_SHAPE
    assert greedy(need + _up(8 * n) - 256) == S.ERR_WORKSPACE


def test_lead_entry_point_checks_its_workspace():
    import paper_2603_12201_amd as ic
    L, S = ic.lib(), ic.Status
    one = C.c_void_p(4096)
    for Tq, k in ((1100, 1024), (2100, 2048), (100, 256)):                   # a tail split over the chip; no leading rows looked for
        d = ic.AttnDesc(1, Tq, Tq, 32, 576, 512, 0, 576, k, 1 / 24.0)
        need = L.ic_sparse_attn_lead_workspace(C.byref(d))
        assert need > 0 and need % 256 == 0
        call = lambda w, n: L.ic_sparse_attn_lead(C.byref(d), one, one, one, one, None, w, n, None)
        assert call(None, need) == S.ERR_WORKSPACE and call(C.c_void_p(4096 + 8), need) == S.ERR_WORKSPACE
        assert call(one, need - 1) == S.ERR_WORKSPACE
        assert L.ic_sparse_attn_lead(C.byref(d), None, one, one, one, None, one, need, None) == S.ERR_NULL
    assert L.ic_sparse_attn_lead_workspace(None) == 0
