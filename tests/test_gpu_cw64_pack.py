"""Constant-weight codes over uint64 words, packed by t-subsets or screened:
each instance of the packing kernel at its smallest length and at batch
remainders, both sides of its limits, and capacities around the code's size."""
import math
import sys

import numpy as np
import pytest

import oracle
import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu

# (n, w, d): every weight 2 .. 8 with one, two and three ones left out of a
# t-subset, n = w and w + 1, walks around 4096 positions, n = 64; then t-subsets
# just inside and outside 2^19, weight 9, three of weight 7, t = 0 and d = 2.
CASES = sorted({(n, w, d) for w in range(2, 9) for d in (3, 4, 5, 6, 7, 8) for n in (w, w + 1, w + 5)}) + [
    (29, 3, 4), (30, 3, 4), (64, 3, 6), (64, 4, 8), (64, 2, 3), (24, 4, 3), (21, 6, 4), (18, 8, 6), (40, 4, 4),
    (30, 5, 5), (60, 4, 6), (54, 5, 8), (17, 9, 6), (14, 7, 8), (16, 7, 6), (33, 3, 7), (12, 4, 2)]


def run(n, w, d, cap):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    words = torch.zeros(max(cap, 1), dtype=torch.int64, device="cuda")[:cap]
    count = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    rc = 0
    try:
        gc.greedy_code_cw64(n, w, d, words, count)
    except gc.GreedyCodeError as e:
        rc = e.rc
    return rc, int(count.item()), words.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n,w,d", CASES)
def test_words_and_capacities(n, w, d):
    print(f"[cw64] n={n} w={w} d={d}", flush=True)
    sys.stdout.flush()
    want = oracle.greedy_list64(n, d, oracle.weight_class64(n, w))[0]
    rc, m, words = run(n, w, d, min(math.comb(n, w), want.size + 5))
    assert rc == 0 and m == want.size
    assert np.array_equal(words[:m], want) and not words[m:].any()
    for cap in sorted({1, want.size - 1, want.size} - {0}):
        rc, m, words = run(n, w, d, cap)
        assert rc == (gc.GC_ECAPACITY if cap < want.size else 0), cap
        assert m == cap and np.array_equal(words, want[:cap]), cap


def test_both_sides_of_the_subset_limit():
    # t = 4: C(60, 4) = 487635 and C(62, 4) = 557845 around 2^19 = 524288.  The
    # words of length 60 are the first C(60, 5) positions of the longer walk.
    cap = 1 << 18
    rc, m, a = run(60, 5, 4, cap)
    assert rc == 0
    rc, n62, b = run(62, 5, 4, cap)
    assert rc == 0 and n62 > m
    assert np.array_equal(a[:m], b[:m]) and int(b[m]) >> 60
