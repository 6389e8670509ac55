"""Graded codes around the line between windows and rounds (n = 18 and 19; at
distance 2 n = 9 and 10) and around the steps of the team's size (one
workgroup up to 512 words of 64 candidates, two from 1024; by rounds at
distance 2 from 512), against the screens: whole walks, a weight, a range after
a prefix.  Results are words, so they have to be equal."""
import sys

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
SCREENS = dict(target_survivors=1000)


def words(p, prefix_words=None, **tuning):
    return gc.device_problem_code(p, prefix_words=prefix_words, **tuning)[0].cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("o", ["grlex", "grevlex"])
@pytest.mark.parametrize("n,d", [(9, 2), (10, 2), (14, 2), (15, 2), (15, 3), (16, 3), (17, 4), (18, 3), (18, 4), (19, 3),
                                 (19, 4), (20, 5)])
def test_rule(n, d, o):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    print(f"[cover] n={n} d={d} {o}", flush=True)
    sys.stdout.flush()
    p = gc.problem(n, d, o)
    got = words(p)
    assert np.array_equal(got, words(p, **SCREENS))
    p = gc.problem(n, d, o, weight=n // 2)
    assert np.array_equal(words(p), words(p, **SCREENS))
    stop = (1 << n) // 3
    prefix = words(gc.problem(n, d, o, stop=stop))
    p = gc.problem(n, d, o, start=stop, prefix=len(prefix))
    assert np.array_equal(words(p, prefix_words=prefix), got)
