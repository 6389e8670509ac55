"""Self-orthogonal graded codes after given words.  Any words may be given:
odd ones, overlapping oddly, and enough of them to span n / 2 dimensions and
more, where the words of a code of its own would span all that is left."""
import sys

import numpy as np
import pytest

import oracle
import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
SCREENS = dict(target_survivors=1000)


@pytest.fixture(scope="module", autouse=True)
def cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    gc.load()


def both(p, given):
    """The code by cover windows and by the screens (any given words may leave
    more than the problem's capacity, which is for a code of its own)."""
    import torch
    out = []
    for tuning in ({}, SCREENS):
        words = torch.zeros(gc.problem_capacity(p) + len(given), dtype=torch.int32, device="cuda")
        words[: len(given)] = torch.from_numpy(given.view(np.int32).copy())
        count = torch.zeros(1, dtype=torch.int64, device="cuda")
        gc.greedy_code_problem_device(p, words, count, **tuning)
        out.append(words[: int(count.item())].cpu().numpy().view(np.uint32))
    return out


def by_definition(n, d, o, start, given):
    """The walk's even words from position `start` on, each kept when it is at
    distance d or more from, and overlaps evenly with, all words before it."""
    walk = np.concatenate([oracle.weight_class(n, w, oracle.ORDERINGS[o]) for w in range(0, n + 1, 2)])
    code = list(map(int, given))
    for x in map(int, walk[start:]):
        if all((x ^ c).bit_count() >= d and (x & c).bit_count() % 2 == 0 for c in code):
            code.append(x)
    return np.array(code, np.uint32)


def words_given(n, kind):
    rng = np.random.default_rng(n)
    if kind == "units":        # of the first n / 2 coordinates
        return np.array([1 << i for i in range(n // 2)], np.uint32)
    if kind == "more units":
        return np.array([1 << i for i in range(n // 2 + 2)], np.uint32)
    # n / 2 or more words with an even weight
    x = rng.integers(0, 1 << n, size=n // 2 + (kind == "many")).astype(np.uint32)
    return np.array([int(v) ^ (int(v).bit_count() & 1) for v in x], np.uint32)


@pytest.mark.parametrize("o", ["grlex", "grevlex"])
@pytest.mark.parametrize("kind", ["units", "more units", "even", "many"])
@pytest.mark.parametrize("n,d", [(8, 1), (8, 2), (9, 2), (11, 4)])
def test_spanning_prefixes_by_the_definition(n, d, kind, o):
    print(f"[so] n={n} d={d} {kind} {o}", flush=True)
    sys.stdout.flush()
    given = words_given(n, kind)
    got, _ = both(gc.problem(n, d, o, self_orthogonal=True, start=1, prefix=len(given)), given)
    assert np.array_equal(got, by_definition(n, d, o, 1, given))


@pytest.mark.parametrize("o", ["grlex", "grevlex"])
@pytest.mark.parametrize("kind", ["units", "more units", "even", "many"])
@pytest.mark.parametrize("n,d", [(14, 2), (16, 1), (17, 2), (20, 4)])
def test_spanning_prefixes(n, d, kind, o):
    print(f"[so] n={n} d={d} {kind} {o}", flush=True)
    sys.stdout.flush()
    given = words_given(n, kind)
    got, ref = both(gc.problem(n, d, o, self_orthogonal=True, start=1, prefix=len(given)), given)
    assert np.array_equal(got, ref)
