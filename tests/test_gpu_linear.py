"""Linear codes built from their generators against the screens: lex, Gray,
B-ordering and self-orthogonal lex/Gray walks, at the edges of the search's
storage (one label word, one wave, LDS, global memory), of the word list of a
B-ordering, of ranges and of capacities.

The screens build the same code when a tuning asks for them (target_survivors
here), and are checked against the oracle elsewhere; results are words, so
they have to be equal."""
import sys

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
SCREENS = dict(target_survivors=1000)


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    gc.load()
    return torch


def both(p, prefix_words=None):
    a, _ = gc.device_problem_code(p, prefix_words=prefix_words)
    b, _ = gc.device_problem_code(p, prefix_words=prefix_words, **SCREENS)
    return a.cpu().numpy().view(np.uint32), b.cpu().numpy().view(np.uint32)


def basis(n, seed):
    rng = np.random.default_rng(seed)
    b = [1 << int(j) for j in rng.permutation(n)]
    for i in range(n):
        for j in range(i):
            if rng.random() < 0.5:
                b[i] ^= b[j]
    return [b[int(i)] for i in rng.permutation(n)]


# label bits 5, 6 and 7 (one word, then two); 14 and 15 (one wave, then the
# workgroup); 17 and 18 at d = 10 (past LDS, into global memory)
@pytest.mark.parametrize("o", ["lex", "gray"])
@pytest.mark.parametrize("n,d", [(1, 2), (2, 2), (5, 2), (16, 3), (17, 4), (14, 5), (20, 5), (16, 9), (18, 9), (21, 8),
                                 (22, 10), (24, 10), (19, 17), (20, 19), (17, 17), (16, 17)])
def test_walks(n, d, o):
    log(f"[linear] n={n} d={d} {o}")
    got, ref = both(gc.problem(n, d, o))
    assert np.array_equal(got, ref)


# listed low-weight words: 1, below and above one segment (4096), above the
# limit at which the screens take over (n = 25, d = 11)
@pytest.mark.parametrize("n,d", [(1, 2), (3, 2), (9, 9), (12, 6), (15, 5), (19, 5), (19, 6), (21, 8), (22, 12), (25, 11)])
def test_user_basis(n, d):
    log(f"[linear] border n={n} d={d}")
    got, ref = both(gc.problem(n, d, "border", basis=basis(n, 100 * n + d)))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("o", ["lex", "gray"])
@pytest.mark.parametrize("n,d", [(1, 1), (2, 1), (2, 2), (7, 1), (13, 2), (16, 3), (17, 4), (22, 6), (23, 8), (24, 12)])
def test_self_orthogonal(n, d, o):
    log(f"[linear] self-orthogonal n={n} d={d} {o}")
    got, ref = both(gc.problem(n, d, o, self_orthogonal=True))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("kw", [dict(ordering="lex"), dict(ordering="gray"), dict(ordering="border"),
                                dict(ordering="gray", self_orthogonal=True)], ids=["lex", "gray", "border", "so"])
def test_ranges_and_prefixes(kw):
    n, d = 15, 4
    if kw["ordering"] == "border":
        kw = dict(kw, basis=basis(n, 5))
    full, _ = both(gc.problem(n, d, **kw))
    total = gc.problem_positions(gc.problem(n, d, **kw))
    for cut in (1, 2, 77, total // 3, total // 2 + 1, total - 1):
        log(f"[linear] {kw['ordering']} cut {cut}")
        head, ref = both(gc.problem(n, d, stop=cut, **kw))
        assert np.array_equal(head, ref) and np.array_equal(head, full[: len(head)])
        rest = gc.problem(n, d, start=cut, prefix=len(head), **kw)
        got, ref = both(rest, prefix_words=head)
        assert np.array_equal(got, ref) and np.array_equal(got, full)
        # A prefix that is no beginning of the code: one word changed, one missing.
        for other in (np.concatenate([head[:-1], head[-1:] ^ np.uint32(3)]), head[:-1]):
            got, ref = both(gc.problem(n, d, start=cut, prefix=len(other), **kw), prefix_words=other)
            assert np.array_equal(got, ref)


def test_capacity_keeps_the_beginning_and_nothing_past_it(cuda):
    full, _ = both(gc.problem(16, 3, "gray"))
    for cap in (1, 3, 4, 1001, len(full) - 1):
        words = cuda.full((cap + 8,), -1, dtype=cuda.int32, device="cuda")
        count = cuda.zeros(1, dtype=cuda.int64, device="cuda")
        with pytest.raises(gc.GreedyCodeError) as e:
            gc.greedy_code_device(16, 3, "gray", words[:cap], count)
        assert e.value.rc == gc.GC_ECAPACITY and int(count.item()) == cap
        got = words.cpu().numpy().view(np.uint32)
        assert np.array_equal(got[:cap], full[:cap]) and (got[cap:] == 0xFFFFFFFF).all()


# In a batch the search has less room than alone: (24, 12) goes on to the screens.
@pytest.mark.parametrize("teams", [1, 8])
def test_batch(teams):
    jobs = [(n, d, o) for o in ("lex", "gray") for n, d in [(1, 2), (9, 3), (17, 4), (18, 9), (22, 10), (24, 12), (20, 20)]]
    log(f"[linear] batch teams={teams}")
    words, _, _ = gc.greedy_code_batch(jobs, teams=teams)
    for (n, d, o), w in zip(jobs, words):
        ref, _ = gc.device_code(n, d, o, **SCREENS)
        assert np.array_equal(w.cpu().numpy(), ref.cpu().numpy()), (n, d, o)
