"""Rules of the top-k launches that no result shows (a row that a form cannot decide takes the radix select, exactly, but for
many times as long): the library's own arithmetic, and the kernels' thresholds and lists replayed on the CPU."""
import ctypes

import numpy as np
import pytest

import paper_2603_12201_amd as m


def rule(name, *args):
    """A host function ic::name(int, ...) of the library."""
    f = getattr(m.lib(), "_ZN2ic%d%sE%s" % (len(name), name, "i" * len(args)))
    f.restype = ctypes.c_int
    return f(*(ctypes.c_int(a) for a in args))


def keys_of(x):
    """Order-preserving keys of positive scores."""
    return x.view(np.uint32).astype(np.int64) + 0x80000000


def threshold(keys, runs, want):
    """The lower edge of the bin, of 4096 between the smallest and the largest of 4096 sampled keys, that `want` of them reach."""
    n = len(keys)
    at = (np.arange(runs) * n // runs & ~3)[:, None] + np.arange(4096 // runs)
    s = keys[at].ravel()
    shift = max(0, int(s.max() - s.min()).bit_length() - 12)
    ranks = np.cumsum(np.bincount((s - s.min()) >> shift, minlength=4096)[::-1])
    return s.min() + ((4095 - int(np.searchsorted(ranks, want))) << shift)


def test_lists_of_a_row_in_parts_hold_what_the_rule_admits():
    """A row that is let into the parts form leaves about 2 k + 1 / 128 of its keys as candidates.  Its lists together have room for a
    quarter more at any number of rows: the sampled threshold scatters by 8 (k = 2048, 131 073 keys) to 14 per cent."""
    seen = 0
    for rows in range(1, 513):
        for keys in (65537, 100000, 131073, 300000, 500000, 700000, 1000000, 1040000):
            parts = rule("select_parts", rows, keys)
            for k in (1, 64, 512, 2048):
                if parts and rule("select_parts_fit", k, keys):
                    seen += 1
                    assert parts * rule("select_parts_slots", rows, keys) >= 5 * (2 * k + keys // 128) // 4, (rows, keys, k)
    assert seen > 10000


@pytest.mark.parametrize("rows, keys", [(1, 200000), (6, 500000), (6, 700000), (7, 500000), (7, 800000), (15, 450000), (28, 600000), (100, 200000)])
def test_parts_decide_rows_of_independent_scores(rows, keys):
    k, parts, slots = 2048, rule("select_parts", rows, keys), rule("select_parts_slots", rows, keys)
    rng = np.random.default_rng(keys + rows)
    for _ in range(12):
        x = keys_of(np.maximum(rng.standard_normal(keys, dtype=np.float32) + 5, 0))
        cand = np.nonzero(x >= threshold(x, 32, 4096 * 2 * k // keys + 32))[0]
        assert len(cand) >= k
        assert np.bincount(cand // 32 % parts, minlength=parts).max() <= slots     # a part has every parts-th block of 32 keys
