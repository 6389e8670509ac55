"""Parts of walks: short ones from the start, where a linear search has few levels,
and ranges after given words, where a rule on their number and the range's length
chooses the builder.  Against the screens, which a tuning asks for."""
import sys

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
SCREENS = dict(target_survivors=1000)


@pytest.fixture(scope="module", autouse=True)
def cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    gc.load()


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run(p, given, cap, **tuning):
    """The code, and whether the buffer past it is as it was."""
    import torch
    words = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    words[: len(given)] = torch.from_numpy(np.asarray(given, np.uint32).view(np.int32).copy())
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    gc.greedy_code_problem_device(p, words, count, **tuning)
    got, m = words.cpu().numpy().view(np.uint32), int(count.item())
    assert (got[m:] == 0xFFFFFFFF).all()
    return got[:m]


BASIS = [1 << j ^ (1 << j - 1 if j % 3 else 0) for j in range(20)]
STOPS = [1, 2, 3, 4, 5, 63, 64, 65, 1000, 4096, 4097, 65535, 65536, 65537, 200001]


@pytest.mark.parametrize("so", [False, True])
@pytest.mark.parametrize("o", ["lex", "gray", "border"])
@pytest.mark.parametrize("d", [2, 3, 6, 8, 13, 14])
def test_short_walks(d, o, so):
    if so and o == "border":
        return  # not a problem
    kw = dict(self_orthogonal=so, basis=BASIS if o == "border" else None)
    log(f"[parts] n=20 d={d} {o} {so}")
    for stop in STOPS:
        p = gc.problem(20, d, o, stop=stop, **kw)
        cap = stop + 4
        got = run(p, [], cap)
        assert np.array_equal(got, run(p, [], cap, **SCREENS)), stop
        # and on from there
        for end in (stop + 1, stop + 100, 262144):
            p = gc.problem(20, d, o, start=stop, stop=end, prefix=len(got), **kw)
            cap = len(got) + end - stop + 4
            assert np.array_equal(run(p, got, cap), run(p, got, cap, **SCREENS)), (stop, end)


@pytest.mark.parametrize("o", ["lex", "gray"])
@pytest.mark.parametrize("n,d", [(17, 2), (20, 3)])
def test_many_given_words(n, d, o):
    cut = (1 << n) * 3 // 4 + 7
    head = run(gc.problem(n, d, o, stop=cut), [], cut)
    assert len(head) > 20000
    for wrong in (None, 0, 1, len(head) // 2, 16384, len(head) - 1):
        given = head.copy()
        if wrong is not None:
            given[wrong] ^= 1 << n - 1
        log(f"[parts] n={n} d={d} {o} {len(given)} words, {wrong} wrong")
        p = gc.problem(n, d, o, start=cut, prefix=len(given))
        cap = len(given) + (1 << n) - cut + 4
        assert np.array_equal(run(p, given, cap), run(p, given, cap, **SCREENS)), wrong


# Given words without positions before them, and positions without words.
@pytest.mark.parametrize("o", ["lex", "gray", "grlex", "grevlex"])
def test_words_and_positions_that_do_not_belong_together(o):
    for p, given in ((gc.problem(12, 3, o, start=100), []), (gc.problem(12, 3, o, prefix=2), [5, 77]),
                     (gc.problem(12, 3, o, start=1, prefix=3), [0, 0, 9])):
        assert np.array_equal(run(p, given, 4100), run(p, given, 4100, **SCREENS))


@pytest.mark.parametrize("kw", [{}, dict(weight=10), dict(self_orthogonal=True)])
@pytest.mark.parametrize("n,d,o", [(20, 2, "grlex"), (21, 3, "grevlex"), (21, 4, "grlex"), (22, 6, "grlex"), (22, 8, "grevlex")])
def test_graded_ranges_after_given_words(n, d, o, kw):
    total = gc.problem_positions(gc.problem(n, d, o, **kw))
    for num in (1, 4, 7):
        cut = total * num // 8
        head = run(gc.problem(n, d, o, stop=cut, **kw), [], cut + 4)
        log(f"[parts] n={n} d={d} {o} {kw} {len(head)} words")
        for length in (1, 1000, 1 << 14, 1 << 18, total):
            stop = min(total, cut + length)
            p = gc.problem(n, d, o, start=cut, stop=stop, prefix=len(head), **kw)
            cap = len(head) + stop - cut + 4
            assert np.array_equal(run(p, head, cap), run(p, head, cap, **SCREENS)), (cut, length)
