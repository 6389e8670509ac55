"""Single graded codes have a launch of their own: calls that overlap on
several streams and threads, teams of one and of many workgroups, and an
expired wait followed by further calls on the same workspace."""
import os
import sys
import threading

import numpy as np
import pytest

import oracle
import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
KINDS = [(18, 4, "grlex"), (9, 3, "grevlex"), (16, 5, "grevlex"), (17, 3, "grlex"), (18, 7, "grlex"), (12, 2, "grevlex")]


def build(job, stream=None, noalloc=False):
    import torch
    n, d, o = job
    words = torch.zeros(gc.greedy_code_capacity(n, d), dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    call = gc.greedy_code_device_noalloc if noalloc else gc.greedy_code_device
    call(n, d, o, words, count, stream=stream)
    return words[:int(count.item())].cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("threads", [1, 4])
def test_overlapping_calls(threads):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    print(f"[cover] {threads} threads", flush=True)
    sys.stdout.flush()
    want = {j: oracle.greedy_ball(j[0], j[1], oracle.ORDERINGS[j[2]])[0] for j in KINDS}
    bad = []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            for i in range(12):
                job = KINDS[(i + k) % len(KINDS)]
                if not np.array_equal(build(job, stream), want[job]):
                    bad.append((k, job))
        except Exception as e:  # reported by the main thread
            bad.append((k, e))

    pool = [threading.Thread(target=work, args=(k,)) for k in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    assert not bad, bad
    for job in KINDS:
        assert np.array_equal(build(job, noalloc=True), want[job]), job


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("job", [(18, 4, "grlex"), (18, 7, "grevlex")])
def test_expired_wait_then_further_calls(job, noalloc):
    os.environ["GC_SPIN_LIMIT"] = "0"
    try:
        with pytest.raises(gc.GreedyCodeError) as e:
            build(job, noalloc=noalloc)
        assert e.value.rc == gc.GC_ETIMEOUT
    finally:
        del os.environ["GC_SPIN_LIMIT"]
    want = oracle.greedy_ball(job[0], job[1], oracle.ORDERINGS[job[2]])[0]
    assert np.array_equal(build(job, noalloc=noalloc), want)
