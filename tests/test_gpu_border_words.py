"""B-ordering codes whose low-weight words are held in registers (up to 16384)
or listed in global memory: both sides of the line (n = 15, d = 8: 16383 words,
n = 25, d = 5: 15275; n = 16, d = 8: 26332, n = 26, d = 5: 17901), one word a
thread and fewer, against the screens.  Results are words, so they are equal."""
import sys

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu


def basis(n, seed):
    rng = np.random.default_rng(seed)
    while True:
        rows, pivots = [], []
        for _ in range(n):
            v = int(rng.integers(1, 1 << n))
            rows.append(v)
        for v in rows:
            for p in pivots:
                v = min(v, v ^ p)
            if v:
                pivots.append(v)
        if len(pivots) == n:
            return rows


@pytest.mark.parametrize("n,d", [(2, 2), (7, 3), (10, 4), (14, 8), (15, 8), (16, 8), (25, 5), (26, 5)])
def test_words_of_both_kinds(n, d):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    print(f"[linear] border n={n} d={d}", flush=True)
    sys.stdout.flush()
    p = gc.problem(n, d, "border", basis=basis(n, 10 * n + d))
    got = gc.device_problem_code(p)[0].cpu().numpy()
    assert np.array_equal(got, gc.device_problem_code(p, target_survivors=1000)[0].cpu().numpy())
