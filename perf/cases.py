"""The work this library is measured on.

Each case is a call, or the short sequence of calls, that a serving engine, a long-context prefill job, an indexer's
training step or a layer-pattern study makes, with the sizes of this repository's configurations (32 bf16 or 64 fp8
indexer heads of 128, k = 2048, 32 query heads on one 576-element MLA row) or generic ones.  A case lists its pattern of
Full (F: indexer + top-k) and Shared (S: indices reused) layers; every layer has inputs of its own.
"""
import math
import random

import torch

import paper_2603_12201_amd as ic

MLA = {"H_q": 32, "d_qk": 576, "d_v": 512, "v_off": 0, "row": 576}
BF16_INDEXER = {"H_I": 32, "d_I": 128, "k_sel": 2048, "dtype": "bf16"}
FP8_INDEXER = {"H_I": 64, "d_I": 128, "k_sel": 2048, "dtype": "fp8"}
TINY = {"H_I": 4, "d_I": 64, "k_sel": 64, "dtype": "bf16", "H_q": 4, "d_qk": 64, "d_v": 64, "v_off": 64, "row": 128}


def _case(kind, ix, at, **sizes):
    c = {"kind": kind}
    c.update(ix)
    c.update(at)
    c.update(sizes)
    return c


def listed():
    rows = [
        # the smallest stack: head dims of 64, separate K and V halves; a toy model's prefill, all launches
        ("tiny_stack", _case("stack", TINY, {}, B=1, Tq=512, Lk=512, pos0=0, pattern="FSFS")),
        # one user's chat: a single request at a short context, one token at a time
        ("decode_one_10k", _case("stack", BF16_INDEXER, MLA, B=1, Tq=1, Lk=10007, pos0=10006, pattern="FSSS")),
        # one user's long document: a single request at the longest context
        ("decode_one_200k", _case("stack", BF16_INDEXER, MLA, B=1, Tq=1, Lk=200000, pos0=199999, pattern="FSSS")),
        # offline generation: a full batch of equal contexts
        ("decode_batch_64k", _case("stack", BF16_INDEXER, MLA, B=32, Tq=1, Lk=65536, pos0=65535, pattern="FSSS")),
        # online serving with the cache filled (about 800K tokens): ragged lengths behind a page table
        ("decode_paged_800k", _case("paged", BF16_INDEXER, MLA, B=40, Tq=1, Lk=49152, pos0=0, low=700, page=64, pattern="FSSS")),
        # serving with an fp8 index cache and one drafted token, layer by layer as a model calls it
        ("decode_fp8_draft", _case("layers", FP8_INDEXER, MLA, B=12, Tq=2, Lk=30011, pos0=30009, pattern="FSSS")),
        # short prompts arriving together: most query rows see fewer keys than k
        ("prefill_short", _case("stack", BF16_INDEXER, MLA, B=3, Tq=1021, Lk=1021, pos0=0, pattern="FSSS")),
        # a piece of a prompt on top of a cached prefix (chunked prefill, a new turn), layer by layer
        ("prefill_chunk", _case("layers", BF16_INDEXER, MLA, B=1, Tq=700, Lk=41700, pos0=41000, pattern="FSSS")),
        # a long prompt
        ("prefill_32k", _case("stack", BF16_INDEXER, MLA, B=1, Tq=32768, Lk=32768, pos0=0, pattern="FSSS")),
        # the longest prompt, fp8 indexer
        ("prefill_fp8_131k", _case("stack", FP8_INDEXER, MLA, B=1, Tq=131072, Lk=131072, pos0=0, pattern="FS")),
        # the indexer's training step: a Full layer and the layers it serves, targets, both losses and the gradient
        ("distill_4k", _case("distill", BF16_INDEXER, MLA, B=1, Tq=4096, Lk=4096, pos0=0, pattern="FSSS")),
        # choosing the pattern: overlap of the layers' index sets and the output similarity matrix
        ("pattern_study", _case("study", BF16_INDEXER, MLA, B=1, Tq=3000, Lk=3000, pos0=0, pattern="FFFFFF")),
    ]
    return [dict(c, name=n) for n, c in rows]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["tiny", "decode", "decode", "paged", "layers", "prefill", "prefill", "chunk", "fp8", "distill", "study"])
    if kind == "tiny":
        L = _log(rng, 64, 2048)
        return _case("stack", TINY, {}, B=rng.randint(1, 3), Tq=L, Lk=L, pos0=0, pattern=rng.choice(["FSFS", "FSSS", "FFFF"]))
    if kind == "decode":
        B = _log(rng, 1, 64)
        L = _log(rng, 2500, min(262144, (1 << 21) // B))
        return _case("stack", BF16_INDEXER, MLA, B=B, Tq=1, Lk=L, pos0=L - 1, pattern=rng.choice(["FSSS", "FSFS"]))
    if kind == "paged":
        B = _log(rng, 2, 64)
        L = _log(rng, 4096, min(131072, (1 << 21) // B)) // 64 * 64
        return _case("paged", BF16_INDEXER, MLA, B=B, Tq=1, Lk=L, pos0=0, low=_log(rng, 64, L // 2), page=rng.choice([64, 128, 256]),
                     pattern="FSSS")
    if kind == "layers":
        B, Tq = _log(rng, 1, 32), rng.randint(1, 4)
        L = _log(rng, 2500, min(131072, (1 << 20) // B))
        return _case("layers", rng.choice([BF16_INDEXER, FP8_INDEXER]), MLA, B=B, Tq=Tq, Lk=L, pos0=L - Tq, pattern="FSSS")
    if kind == "prefill":
        B = rng.choice([1, 1, 1, 2, 4])
        L = _log(rng, 200, 32768 // B)
        return _case("stack", BF16_INDEXER, MLA, B=B, Tq=L, Lk=L, pos0=0, pattern=rng.choice(["FSSS", "FSFS"]))
    if kind == "chunk":
        Tq = _log(rng, 16, 4096)
        pos0 = _log(rng, 1000, 100000)
        return _case("layers", BF16_INDEXER, MLA, B=1, Tq=Tq, Lk=pos0 + Tq, pos0=pos0, pattern="FSSS")
    if kind == "fp8":
        L = _log(rng, 3000, 100000)
        return _case("stack", FP8_INDEXER, MLA, B=1, Tq=L, Lk=L, pos0=0, pattern="FS")
    if kind == "distill":
        L = _log(rng, 500, 8192)
        return _case("distill", BF16_INDEXER, MLA, B=rng.choice([1, 2]), Tq=L, Lk=L, pos0=0, pattern=rng.choice(["FS", "FSSS", "FSSSSS"]))
    L = _log(rng, 500, 6000)
    return _case("study", BF16_INDEXER, MLA, B=1, Tq=L, Lk=L, pos0=0, pattern="F" * rng.randint(3, 8))


# ---- inputs ------------------------------------------------------------------------------------------------------

def _e4m3(x):
    """One scale per token: the last dimension holds a token's features."""
    scale = x.abs().amax(dim=-1, keepdim=True).clamp_min(1e-12) / 448.0
    return (x / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn), scale.squeeze(-1).contiguous()


class State:
    pass


def prepare(case, seed):
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 1000003 + 17)
    B, Tq, Lk, k_sel = case["B"], case["Tq"], case["Lk"], case["k_sel"]
    H, d = case["H_I"], case["d_I"]

    def normal(*shape, dtype=torch.bfloat16):
        return torch.randn(shape, generator=gen, device=dev, dtype=dtype)

    s = State()
    s.case, s.full = case, [c == "F" for c in case["pattern"]]
    s.lens = s.pc = None
    n_rows = B * Lk
    if case["kind"] == "paged":
        # a sequence owns exactly the pages its length needs, in random physical order
        page, host = case["page"], torch.Generator().manual_seed(seed * 7919 + 3)
        lens = torch.randint(case["low"], Lk + 1, (B,), generator=host)
        pages = [-(-int(n) // page) for n in lens]
        order = torch.randperm(sum(pages), generator=host)
        table = torch.zeros((B, Lk // page + 1), dtype=torch.int32)
        at = 0
        for b, n in enumerate(pages):
            table[b, :n] = order[at:at + n].to(torch.int32)
            at += n
        n_rows = sum(pages) * page
        s.lens = lens.to(torch.int32).to(dev)
        s.pc = ic.paged_cache(s.lens, table.to(dev), page)

    s.layers = []
    for full in s.full:
        t = {"Q": normal(B, Tq, case["H_q"], case["d_qk"])}
        cache = (n_rows,) if case["kind"] == "paged" else (B, Lk)
        t["KV"] = normal(*cache, case["row"])
        if full:
            t["w"] = torch.rand((B, Tq, H), generator=gen, device=dev)
            if case["dtype"] == "bf16":
                t["q"] = normal(B, Tq, H, d) * (1.0 / math.sqrt(d))
                t["k"] = normal(*cache, d)
            else:
                q, t["q_scale"] = _e4m3(normal(B, Tq, H * d, dtype=torch.float32))
                t["q"] = q.reshape(B, Tq, H, d)
                t["k"], t["k_scale"] = _e4m3(normal(B, Lk, d, dtype=torch.float32))
        s.layers.append(t)
    s.scale = 1.0 / math.sqrt(case["d_qk"])
    s.outs = [torch.empty((B, Tq, case["H_q"], case["d_v"]), dtype=torch.bfloat16, device=dev) for _ in s.layers]
    s.arr = ic.make_layers(s.layers, k_sel, case["pos0"], case["d_v"], case["v_off"], s.scale, s.outs,
                           Lk=Lk if case["kind"] == "paged" else None)
    s.ws = torch.empty(max(ic.forward_stack_workspace(s.arr), 256), dtype=torch.uint8, device=dev)
    s.idx = torch.empty((B, Tq, k_sel), dtype=torch.int32, device=dev)
    if case["kind"] == "study":
        s.index_sets = [_indices(s, t) for t in s.layers]
    return s


def _indices(s, t, **more):
    return ic.indexer_topk(t["q"], t["k"], t["w"], s.case["k_sel"], s.case["pos0"], t.get("q_scale"), t.get("k_scale"),
                           workspace=s.ws, **more)


def run(s):
    c = s.case
    if c["kind"] == "stack":
        ic.forward_stack(s.arr, s.full, s.idx, s.ws)
        return [s.idx, s.outs]
    if c["kind"] == "paged":
        ic.forward_stack_paged(s.arr, s.full, s.pc, s.idx, s.ws)
        return [s.idx, s.outs]
    if c["kind"] == "layers":
        for t, full, out in zip(s.layers, s.full, s.outs):
            if full:
                _indices(s, t, idx=s.idx)
            ic.sparse_attn(t["Q"], t["KV"], s.idx, c["d_v"], c["v_off"], s.scale, workspace=s.ws, out=out)
        return [s.idx, s.outs]
    if c["kind"] == "distill":
        idx, logits = _indices(s, s.layers[0], want_scores=True)
        probs = []
        for t, out in zip(s.layers, s.outs):
            _, lse = ic.sparse_attn(t["Q"], t["KV"], idx, c["d_v"], c["v_off"], s.scale, want_lse=True, workspace=s.ws, out=out)
            probs.append(ic.attn_probs(t["Q"], t["KV"], idx, s.scale, lse))
        multi, avg, grad = ic.distill_loss(probs, logits, want_grad=True)
        return [idx, logits, probs, multi, avg, grad, s.outs]
    overlap, inter, sizes = ic.topk_overlap(s.index_sets, c["Lk"])
    S = ic.similarity_matrix(s.arr, s.index_sets)
    return [overlap, inter, sizes, S, s.outs]


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def _spans(case):
    """(keys visible, entries selected, distinct cache rows, sequences' keys) summed over the query rows / sequences."""
    B, Tq, Lk, k, p0 = case["B"], case["Tq"], case["Lk"], case["k_sel"], case["pos0"]
    if case["kind"] == "paged":
        mean = (case["low"] + Lk) / 2.0
        return B * mean, B * min(k, mean), B * min(k, mean), B * mean
    lo, hi = p0 + 1, p0 + Tq
    pairs = B * (lo + hi) * Tq / 2.0
    short = max(0, min(hi, k) - lo + 1)
    entries = B * (short * (2 * lo + short - 1) / 2.0 + (Tq - short) * k)
    return pairs, entries, min(entries, float(B * Lk)), float(B * Lk)


def work(case):
    pairs, entries, rows, keys = _spans(case)
    nq = case["B"] * case["Tq"]
    n, n_full = len(case["pattern"]), case["pattern"].count("F")
    elem = 2 if case["dtype"] == "bf16" else 1
    ix_bytes = keys * case["d_I"] * elem + nq * case["H_I"] * (case["d_I"] * elem + 4)
    ix_flops = 2.0 * case["H_I"] * case["d_I"] * pairs
    idx_bytes = nq * case["k_sel"] * 4
    qo_bytes = nq * case["H_q"] * (case["d_qk"] + case["d_v"]) * 2
    at_bytes = rows * case["row"] * 2 + qo_bytes
    at_flops = 2.0 * entries * case["H_q"] * (case["d_qk"] + case["d_v"])
    if case["kind"] == "distill":
        # scores and their indices once; per layer attention and its probabilities; losses' gradient
        return {"bytes": ix_bytes + 2 * idx_bytes + n * (at_bytes + idx_bytes) + idx_bytes,
                "flops": ix_flops + n * (at_flops + 2.0 * entries * case["H_q"] * case["d_qk"])}
    if case["kind"] == "study":
        # every index set and every layer's inputs and outputs once; one attention per pair of layers
        return {"bytes": n * (idx_bytes + at_bytes), "flops": n * (n + 1) / 2.0 * at_flops}
    return {"bytes": n_full * ix_bytes + idx_bytes + n * at_bytes, "flops": n_full * ix_flops + n * at_flops}


def tolerance(case):
    if case["kind"] == "study":
        return {"rel": 1e-2, "differ": 0.0}        # bf16 outputs; the counts are whole numbers of given sets
    # bf16 outputs; a score summed in another order in fp32 may swap a pair at the k-th place, which shifts the row's
    # ascending positions between the two
    return {"rel": 1e-2, "differ": 0.005}
