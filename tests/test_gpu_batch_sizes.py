"""Batches around the number of jobs whose records fit the pinned block of a
launch (128 KiB of 360-byte records: 364 jobs): words and counts of each job."""
import sys

import numpy as np
import pytest

import oracle
import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
KINDS = [(7, 3, "grlex"), (8, 3, "lex"), (6, 1, "gray"), (9, 4, "grevlex"), (5, 2, "grlex"), (9, 5, "gray")]


@pytest.mark.parametrize("njobs", [1, 2, 364, 365, 700])
def test_batch_of_njobs(njobs):
    print(f"[batch] {njobs} jobs", flush=True)
    sys.stdout.flush()
    jobs = [KINDS[i % len(KINDS)] for i in range(njobs)]
    want = {j: oracle.greedy_ball(j[0], j[1], oracle.ORDERINGS[j[2]])[0] for j in KINDS}
    words, info, _ = gc.greedy_code_batch(jobs)
    for j, w, i in zip(jobs, words, info):
        assert i["status"] == 0
        assert np.array_equal(w.cpu().numpy().view(np.uint32), want[j]), j
