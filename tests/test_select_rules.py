"""Rules of the top-k launches that no result shows (a row that a form cannot decide takes the radix select, exactly, but for
many times as long): the library's own arithmetic, and the kernels' thresholds and lists replayed on the CPU."""
import ctypes

import numpy as np
import pytest
from scipy.signal import lfilter

import paper_2603_12201_amd as m


def rule(name, *args):
    """A host function ic::name(int, ...) of the library."""
    f = getattr(m.lib(), "_ZN2ic%d%sE%s" % (len(name), name, "i" * len(args)))
    f.restype = ctypes.c_int
    return f(*(ctypes.c_int(a) for a in args))


def keys_of(x):
    """Order-preserving keys of scores."""
    u = (x + np.float32(0)).view(np.uint32)
    return np.where(u >> 31, ~u, u | 0x80000000).astype(np.int64)


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


def test_short_rows_of_a_ragged_launch_in_parts_are_read_once():
    """Sequences too short for the sample (less than 8192 keys, or 4 k) beside long ones keep their keys in LDS for the radix select's sweeps."""
    assert rule("select_parts_cache", 1) >= max(8192, 4 * 2048)


@pytest.mark.parametrize("keys, memory", [(41700, 0), (131072, 0), (41700, 64), (65536, 64), (131072, 64), (131072, 256), (131072, 1024)])
@pytest.mark.parametrize("mean", [5, 0])
def test_candidate_form_decides_rows_of_correlated_scores(keys, memory, mean):
    """Half of the variance in a component that decays over `memory` keys (neighbours score alike), all scores positive or around zero:
    at most 2 of 100 rows of a launch of more rows than CUs leave fewer than k candidates or more than the list holds."""
    k, many, rows, missed = 2048, 1, 100, 0
    rng = np.random.default_rng(keys + memory)
    rank, runs, room = rule("select_cand_rank", k, keys, many), rule("select_cand_runs", many), rule("select_cand_list", many)
    for _ in range(rows):
        x = rng.standard_normal(keys, dtype=np.float32)
        if memory:
            a = np.exp(-1 / memory)
            slow = lfilter([np.sqrt(1 - a * a)], [1, -a], rng.standard_normal(keys, dtype=np.float32))
            x = (np.sqrt(0.5) * (x + slow)).astype(np.float32)
        x = keys_of(x + np.float32(mean))
        n = int((x >= threshold(x, runs, rank)).sum())
        missed += n < k or n > room
    assert missed <= 2, missed
