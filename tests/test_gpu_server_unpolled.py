"""A server whose jobs nobody polls: what was published runs to its end without
a further call, also where a wide job changes the teams in between, and words,
fetch and stats alone find it."""
import sys
import time

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
NARROW = [(12, 3, "grlex"), (16, 5, "grevlex"), (20, 4, "lex"), (24, 4, "grlex"), (18, 6, "grlex"), (22, 5, "grevlex")]
WIDE = [(25, 6, "grlex"), (25, 6, "grevlex")]


@pytest.fixture(scope="module", autouse=True)
def cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    gc.load()


@pytest.mark.parametrize("teams", [2, 4])
@pytest.mark.parametrize("how", ["fetch", "stats"])
def test_published_jobs_finish_without_polls(teams, how):
    want = {j: gc.device_code(*j)[0].cpu().numpy().view(np.uint32) for j in NARROW + WIDE}
    jobs = NARROW + WIDE[:1] + NARROW + WIDE[1:] + NARROW
    with gc.Server(arena_bytes=32 << 20, teams=teams) as srv:
        for turn in range(2):
            t0 = time.perf_counter()
            tickets = []
            for j in jobs:
                t = time.perf_counter()
                tickets.append(srv.submit(*j))
                if j in WIDE:
                    print(f"[server] teams={teams} submit of {j}: {1e3 * (time.perf_counter() - t):.2f} ms", flush=True)
            print(f"[server] teams={teams}: {len(jobs)} jobs submitted in {1e3 * (time.perf_counter() - t0):.1f} ms",
                  flush=True)
            sys.stdout.flush()
            time.sleep(1.0)
            for t, j in zip(tickets, jobs):  # the first call on each ticket
                if how == "stats":
                    assert srv.stats(t)["count"] == len(want[j]), j
                assert np.array_equal(srv.fetch(t), want[j]), j
                srv.release(t)


def test_a_finished_wide_job_that_nobody_asks_for():
    want = {j: gc.device_code(*j)[0].cpu().numpy().view(np.uint32) for j in NARROW + WIDE}
    with gc.Server(arena_bytes=32 << 20, teams=2) as srv:
        wide = [srv.submit(*j) for j in WIDE]
        for turn in range(3):
            tickets = [srv.submit(*j) for j in NARROW]
            time.sleep(0.3)
            for t, j in zip(tickets, NARROW):
                assert srv.poll(t)[0] == gc.GC_JOB_DONE, j
                assert np.array_equal(srv.fetch(t), want[j]), j
                srv.release(t)
        for t, j in zip(wide, WIDE):
            assert np.array_equal(srv.fetch(t), want[j]), j
