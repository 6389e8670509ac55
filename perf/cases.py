"""The work that users of this library have it do, as measurable cases.

A case names one kind of call and its sizes; prepare() makes what a program
holds before the call (inputs from the seed), run() makes one pass through the
public entry points, work() says what the path cannot do without.

The plain walks (n, d, ordering) have no data of their own, so there the seed
picks the ordering within its family: lex or Gray ("positional"), graded
lexicographic or graded reverse lexicographic ("graded").  The other kinds
take real inputs: a basis, a checkpoint, a list of jobs.
"""
import math
import random

import numpy as np
import torch

import paper_1507_05398_amd as gc

FAMILY = {"positional": ("lex", "gray"), "graded": ("grlex", "grevlex")}


def listed():
    return [
        # The smallest calls: a textbook code (Hamming [15, 11]) straight into
        # host memory, where the latency of one call is all there is.
        {"name": "host_15_3", "kind": "host", "family": "positional", "n": 15, "d": 3},
        # An ordinary single code of each family, left on the device.
        {"name": "lin_20_4", "kind": "plain", "family": "positional", "n": 20, "d": 4},
        {"name": "graded_22_5", "kind": "plain", "family": "graded", "n": 22, "d": 5},
        # The dense screens: small distance, codes of 10^5 to 10^6 words.
        {"name": "graded_24_3", "kind": "plain", "family": "graded", "n": 24, "d": 3},
        {"name": "lin_26_3", "kind": "plain", "family": "positional", "n": 26, "d": 3},
        # The longest walk: 2^30 candidates, a small code.
        {"name": "lin_30_10", "kind": "plain", "family": "positional", "n": 30, "d": 10},
        # B-ordering with the user's own basis (the seed's), an odd length.
        {"name": "border_23_5", "kind": "border", "n": 23, "d": 5},
        # Self-orthogonal codes; at n = 24, d = 8 lex this is the extended Golay code.
        {"name": "so_24_8", "kind": "so", "family": "graded", "n": 24, "d": 8},
        # Constant weight: the weight-10 vectors of length 24.
        {"name": "weight_24_10_6", "kind": "weight", "n": 24, "w": 10, "d": 6},
        # A construction resumed from a checkpoint somewhere in the walk.
        {"name": "resume_21_4", "kind": "resume", "family": "graded", "n": 21, "d": 4},
        # Many codes of uneven size in one launch.
        {"name": "batch_30", "kind": "batch", "jobs": 30, "n_lo": 12, "n_hi": 22},
        # A burst of jobs through the job server, words back in host memory.
        {"name": "served_200", "kind": "served", "jobs": 200, "n_lo": 10, "n_hi": 20},
    ]


def draw(rng):
    kind = rng.choice(["host", "plain", "plain", "plain", "border", "so", "weight", "resume", "batch", "served",
                       "cw64"])
    fam = rng.choice(["positional", "graded"])
    # Distances up to a third of the length: beyond it codes have a few words.
    if kind in ("host", "plain"):
        if fam == "positional" and rng.random() < 0.3:
            return {"kind": kind, "family": fam, "n": rng.randint(25, 29), "d": rng.randint(7, 9)}
        n = rng.randint(9, 25 if fam == "positional" else 24)
        return {"kind": kind, "family": fam, "n": n, "d": rng.randint(3, n // 3)}
    if kind == "border":
        n = rng.randint(9, 25)
        return {"kind": kind, "n": n, "d": rng.randint(3, n // 3)}
    if kind == "so":
        n = rng.randint(14, 24)
        return {"kind": kind, "family": fam, "n": n, "d": rng.choice([4, 6, 8][: 1 + (n >= 18) + (n >= 22)])}
    if kind == "weight":
        n = rng.randint(14, 26)
        return {"kind": kind, "n": n, "w": rng.randint(4, n // 2), "d": rng.choice([4, 6])}
    if kind == "resume":
        n = rng.randint(14, 23)
        return {"kind": kind, "family": fam, "n": n, "d": rng.randint(3, n // 3)}
    if kind == "batch":
        lo = rng.randint(8, 14)
        return {"kind": kind, "jobs": rng.randint(5, 30), "n_lo": lo, "n_hi": rng.randint(lo + 4, 22)}
    if kind == "served":
        return {"kind": kind, "jobs": rng.randint(20, 300), "n_lo": 10, "n_hi": rng.randint(14, 21)}
    n = rng.randint(20, 40)
    return {"kind": "cw64", "n": n, "w": rng.randint(3, 4 if n > 30 else 5), "d": rng.choice([4, 6])}


def _ordering(case, seed):
    return FAMILY[case["family"]][seed % 2]


def _random_basis(n, rng):
    """An ordered basis of F_2^n: the unit vectors under random row additions
    and a random order."""
    b = [1 << j for j in range(n)]
    rng.shuffle(b)
    for i in range(n):
        for j in range(i):
            if rng.random() < 0.5:
                b[i] ^= b[j]
    rng.shuffle(b)
    return b


def _job_list(case, rng):
    """(n, d, ordering) jobs: lengths spread evenly over the range (served
    jobs skewed towards the short ones), distances 3 to 8, orderings from the
    seed."""
    lo, hi, jobs = case["n_lo"], case["n_hi"], case["jobs"]
    out = []
    for i in range(jobs):
        u = (i + 0.5) / jobs
        if case["kind"] == "served":
            u = min(1.0 - 1e-9, -math.log2(1.0 - u) / 6.0)  # half of the jobs in the lowest sixth
        n = lo + int(u * (hi - lo + 1))
        out.append((n, 3 + i * 5 % 6, rng.choice(["lex", "gray", "grlex", "grevlex"])))
    return out


def _buffers(capacity):
    return {"words": torch.zeros(capacity, dtype=torch.int32, device="cuda"),
            "count": torch.zeros(1, dtype=torch.int64, device="cuda")}


def prepare(case, seed):
    rng = random.Random(seed)
    kind, n, d = case["kind"], case.get("n"), case.get("d")
    if kind in ("border", "so", "weight"):
        if kind == "border":
            p = gc.problem(n, d, "border", basis=_random_basis(n, rng))
        elif kind == "so":
            p = gc.problem(n, d, _ordering(case, seed), self_orthogonal=True)
        else:
            p = gc.problem(n, d, FAMILY["graded"][seed % 2], weight=case["w"])
        return dict(case, problem=p, **_buffers(gc.problem_capacity(p)))
    if kind == "resume":
        # The checkpoint: what a run that stopped at `cut` returned.
        o = _ordering(case, seed)
        cut = rng.randrange((1 << n) // 5, (1 << n) // 3)
        words, _ = gc.device_problem_code(gc.problem(n, d, o, stop=cut))
        state = dict(case, problem=gc.problem(n, d, o, start=cut, prefix=words.numel()),
                     **_buffers(gc.greedy_code_capacity(n, d)))
        state["words"][: words.numel()] = words
        return state
    if kind == "batch":
        plan = gc.BatchPlan(_job_list(case, rng))
        for words, _ in plan.bufs:
            words.zero_()
        return dict(case, plan=plan)
    if kind == "served":
        jobs = _job_list(case, rng)
        return dict(case, list=jobs, words=[np.zeros(gc.greedy_code_capacity(n, d), np.uint32) for n, d, _ in jobs])
    if kind == "cw64":
        n += seed % 2  # a length or the next one
        cap = math.comb(case["n"] + 1, case["w"])
        return dict(case, n=n, words=torch.zeros(cap, dtype=torch.int64, device="cuda"),
                    count=torch.zeros(1, dtype=torch.int64, device="cuda"))
    state = dict(case, ordering=_ordering(case, seed))
    if kind == "host":
        return dict(state, words=np.zeros(gc.greedy_code_capacity(n, d), np.uint32))
    return dict(state, **_buffers(gc.greedy_code_capacity(n, d)))


def run(state):
    kind = state["kind"]
    if kind == "batch":
        state["plan"].run()
        return state["plan"].bufs
    if kind == "served":
        sizes = np.zeros(len(state["list"]), np.int64)
        with gc.Server(arena_bytes=32 << 20, teams=2) as srv:
            tickets = [srv.submit(*j) for j in state["list"]]
            pending = list(range(len(tickets)))
            while pending:
                rest = []
                for i in pending:
                    if srv.poll(tickets[i])[0] >= gc.GC_JOB_DONE:
                        code = srv.fetch(tickets[i])
                        state["words"][i][: len(code)] = code
                        sizes[i] = len(code)
                        srv.release(tickets[i])
                    else:
                        rest.append(i)
                pending = rest
        return {"words": np.concatenate(state["words"]).view(np.int32), "sizes": sizes}
    if kind == "host":
        code = gc.greedy_code(state["n"], state["d"], state["ordering"])
        state["words"][: len(code)] = code
        return {"words": state["words"].view(np.int32), "count": len(code)}
    words, count = state["words"], state["count"]
    if kind == "plain":
        gc.greedy_code_device(state["n"], state["d"], state["ordering"], words, count)
    elif kind == "cw64":
        gc.greedy_code_cw64(state["n"], state["w"], state["d"], words, count)
    else:
        gc.greedy_code_problem_device(state["problem"], words, count)
    return {"words": words, "count": count}


def _ball(n, r):
    return sum(math.comb(n, i) for i in range(r + 1))


def _code_size(n, d):
    """Sphere-packing bound on the words of one code."""
    if d > n:
        return 1
    nn, dd = (n - 1, d - 1) if d % 2 == 0 else (n, d)
    return (1 << nn) // _ball(nn, (dd - 1) // 2)


def work(case):
    """Bytes: the words written, once (sizes by the packing bound) and a
    checkpoint read once.  Operations: one comparison of n bits for each
    candidate of the walk."""
    kind = case["kind"]
    if kind in ("batch", "served"):
        jobs = _job_list(case, random.Random(0))
        return {"bytes": sum(4 * _code_size(n, d) for n, d, _ in jobs), "flops": sum(n << n for n, _, _ in jobs)}
    n, d = case["n"], case["d"]
    if kind in ("weight", "cw64"):
        e, w = (d + 1) // 2, case["w"]
        # Pairs of code words share at most w - e ones.
        words = math.comb(n, w - e + 1) // math.comb(w, w - e + 1) if w >= e else 1
        return {"bytes": (8 if kind == "cw64" else 4) * max(1, words), "flops": n * math.comb(n, w)}
    size = _code_size(n, d)
    if kind == "so":
        return {"bytes": 4 * min(size, 1 << n // 2), "flops": n << n - 1}
    return {"bytes": 4 * size, "flops": n << n}


def exact(case, seed):
    """The plain walks over at most 2^14 positions by the definition: walk the
    ordering, keep what is at distance d or more from everything kept."""
    if case["kind"] not in ("host", "plain") or case["n"] > 14:
        return None
    n, d, o = case["n"], case["d"], _ordering(case, seed)
    x = np.arange(1 << n, dtype=np.int64)
    weight = np.bitwise_count(x)
    if o == "gray":
        x = x ^ (x >> 1)
    elif o == "grlex":
        x = x[np.lexsort((x, weight))]
    elif o == "grevlex":  # equal weights: the word with a 1 at the lowest differing bit first
        back = sum(((x >> j) & 1) << (n - 1 - j) for j in range(n))
        x = x[np.lexsort((-back, weight))]
    covered = np.zeros(1 << n, dtype=bool)
    code = []
    every = np.arange(1 << n, dtype=np.int64)
    near = every[np.bitwise_count(every) < d]
    for v in x.tolist():
        if not covered[v]:
            code.append(v)
            covered[near ^ v] = True
    words = np.zeros(_code_size(n, d), np.int32)
    words[: len(code)] = code
    return {"words": words, "count": np.array([len(code)]) if case["kind"] == "plain" else len(code)}
