"""The server changes teams when a wide job (built by the screens) opens or
closes: every result is the code that the device entry point builds."""
import sys
import time

import numpy as np
import pytest

import paper_1507_05398_amd as gc

pytestmark = pytest.mark.gpu
NARROW = [(12, 3, "grlex"), (16, 5, "grevlex"), (20, 4, "lex"), (11, 7, "gray"), (18, 6, "grlex")]
WIDE = [(25, 6, "grlex"), (25, 6, "grevlex")]


@pytest.mark.parametrize("teams", [2, 4])
def test_wide_jobs_between_narrow_ones(teams):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    want = {j: gc.device_code(*j)[0].cpu().numpy().view(np.uint32) for j in NARROW + WIDE}
    with gc.Server(arena_bytes=16 << 20, teams=teams) as srv:
        for order in (NARROW + WIDE[:1] + NARROW + WIDE[1:] + NARROW, WIDE + NARROW, NARROW):
            print(f"[server] teams={teams}: {len(order)} jobs", flush=True)
            sys.stdout.flush()
            tickets = [(srv.submit(*j), j) for j in order]
            t0 = time.time()
            while tickets:
                rest = []
                for t, j in tickets:
                    state, _ = srv.poll(t)
                    assert state != gc.GC_JOB_FAILED
                    if state == gc.GC_JOB_DONE:
                        assert np.array_equal(srv.fetch(t), want[j]), j
                        srv.release(t)
                    else:
                        rest.append((t, j))
                tickets = rest
                assert time.time() - t0 < 60
