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


# More given words than a workgroup takes at a time (1024), with new dimensions
# among the later ones: those of a code, and any.
@pytest.mark.parametrize("o", ["grlex", "grevlex"])
@pytest.mark.parametrize("n,d", [(22, 2), (24, 4)])
def test_long_prefixes_of_a_code(n, d, o):
    full, _ = both(gc.problem(n, d, o, self_orthogonal=True), np.zeros(0, np.uint32))
    total = gc.problem_positions(gc.problem(n, d, o, self_orthogonal=True))
    for cut in (total // 2, total * 3 // 4):
        head, _ = both(gc.problem(n, d, o, self_orthogonal=True, stop=cut), np.zeros(0, np.uint32))
        print(f"[so] n={n} d={d} {o} cut {cut}: {len(head)} of {len(full)}", flush=True)
        sys.stdout.flush()
        assert np.array_equal(head, full[: len(head)])
        got, ref = both(gc.problem(n, d, o, self_orthogonal=True, start=cut, prefix=len(head)), head)
        assert np.array_equal(got, ref) and np.array_equal(got, full)


@pytest.mark.parametrize("o", ["grlex", "grevlex"])
@pytest.mark.parametrize("count", [1024, 1025, 2047, 3100])
def test_long_prefixes_of_any_words(count, o):
    n = 18
    rng = np.random.default_rng(count)
    # Each 1024 words add two dimensions to those before them.
    basis = rng.permutation(n)
    given = np.zeros(count, np.uint32)
    for i in range(count):
        for j in range(2 * (i // 1024) + 2):
            given[i] ^= np.uint32(int(rng.integers(2)) * (3 << int(basis[j]) & (1 << n) - 1))
    print(f"[so] {count} words {o}", flush=True)
    sys.stdout.flush()
    got, ref = both(gc.problem(n, 2, o, self_orthogonal=True, start=5, prefix=count), given)
    assert np.array_equal(got, ref)
