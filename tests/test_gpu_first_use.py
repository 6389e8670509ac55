"""The first call that needs a workspace makes it without waiting for other
streams: with long work on the null stream, a call on a stream of its own is back
before that work ends.  In a process of its own, whose pool is empty."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import time
import torch
assert torch.cuda.is_available(), "GPU tests need a ROCm device"
import paper_1507_05398_amd as gc
gc.greedy_code_device(9, 3, "lex", torch.zeros(64, dtype=torch.int32, device="cuda"),
                      torch.zeros(1, dtype=torch.int64, device="cuda"))  # the kernels are loaded
words = torch.zeros(gc.greedy_code_capacity(16, 5), dtype=torch.int32, device="cuda")
count = torch.zeros(1, dtype=torch.int64, device="cuda")
stream = torch.cuda.Stream()
torch.cuda._sleep(1000)
torch.cuda.synchronize()
t = time.perf_counter()
torch.cuda._sleep(1000000)
torch.cuda.synchronize()
per_second = 1000000 / (time.perf_counter() - t)
done = torch.cuda.Event()
torch.cuda._sleep(int(per_second))
done.record()
t = time.perf_counter()
gc.greedy_code_device(16, 5, "grlex", words, count, stream=stream)
dt = time.perf_counter() - t
busy = not done.query()
torch.cuda.synchronize()
print("first call %.1f ms, other stream busy: %s, words %d" % (1e3 * dt, busy, count.item()), flush=True)
assert busy
"""


def test_first_call_waits_for_no_other_stream():
    print("[first use]", flush=True)
    got = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    print(got.stdout, flush=True)
    assert got.returncode == 0, got.stderr[-2000:]
