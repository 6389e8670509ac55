"""Linear codes whose search needs hundreds of KiB of label bitmaps, in batches
and on a server: built from their generators (no windows), beside graded jobs
that use the same workspace, and those that a team has no room for."""
import sys

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
LINEAR = [(24, 11, "lex"), (28, 10, "lex"), (22, 13, "gray"), (30, 10, "gray"), (26, 12, "lex")]
GRADED = [(20, 4, "grlex"), (18, 5, "grevlex"), (21, 3, "grevlex"), (22, 7, "grlex")]
SCREENED = [(25, 14, "gray"), (24, 13, "lex")]  # no room, and none found to be left


@pytest.fixture(scope="module")
def want():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    gc.load()
    return {j: gc.device_code(*j)[0].cpu().numpy().view(np.uint32) for j in LINEAR + GRADED + SCREENED}


def mixed():
    return [j for pair in zip(LINEAR, GRADED + SCREENED) for j in pair] + SCREENED + GRADED


@pytest.mark.parametrize("teams", [0, 1, 4, 8])
def test_batch(want, teams):
    print(f"[team] batch teams={teams}", flush=True)
    sys.stdout.flush()
    words, info, _ = gc.greedy_code_batch(mixed(), teams=teams)
    for j, w, i in zip(mixed(), words, info):
        assert i["status"] == 0 and np.array_equal(w.cpu().numpy().view(np.uint32), want[j]), j


@pytest.mark.parametrize("teams", [1, 2, 4, 8])
def test_served(want, teams):
    with gc.Server(arena_bytes=16 << 20, teams=teams) as srv:
        for turn in range(2):
            print(f"[team] served teams={teams}", flush=True)
            sys.stdout.flush()
            tickets = [srv.submit(*j) for j in mixed()]
            srv.drain(timeout_ms=30000)
            for t, j in zip(tickets, mixed()):
                assert np.array_equal(srv.fetch(t), want[j]), j
                if j in LINEAR:
                    assert srv.stats(t)["windows"] == 0, j
                srv.release(t)
