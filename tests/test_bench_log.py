"""bench.py's launch log: the screens' rates come from the launches that executed
checks, the others' bytes from the rest."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_mixed_launches_are_kept_apart():
    log = bench.LaunchLog()
    stats = dict(kernel_ms=2.0, checks_near=3 * 10**8, checks_deep=10**8, checks_pairs=10**8, count=7)
    log.add("25_4_grlex", stats, 11)
    log.add("24_4_grlex", dict(stats, kernel_ms=8.0, checks_near=0, checks_deep=0, checks_pairs=0, count=10**6), 13)
    assert log.launches == {True: 1, False: 1} and log.w_ee == 24 and log.executed == 5 * 10**8
    assert abs(log.gchecks() - 250.0) < 1e-9          # 5e8 in 2 ms
    assert abs(log.tops() - 250.0 * 50 / 1e3) < 1e-9  # 2 n = 50 operations each
    assert abs(log.gbytes() - 4e6 / 8e-3 / 1e9) < 1e-9
