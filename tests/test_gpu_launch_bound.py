"""Plans that commit one migration a ranking pass over lists long enough for the bound on the launches of the loop kernel to
count (more than 8192 candidates): every one of them has to come to its end.  Against the oracle; every comparison is exact."""
import numpy as np
import pytest

from paper_2310_09443_amd.traces import Trace, Workload
from test_gpu_loop_edges import _equal_tensors
from test_gpu_parity import assert_plan_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [9000, 30000])
def test_equal_candidates_all_committed(g10, n):
    """More candidates of one benefit than a list holds: every other pass is ranked by an arg-max over the threads, and
    nothing on its list clears the others' bound."""
    h, v, args = run_both(g10, _equal_tensors(n, 300, 5_000_000))
    a = dict(args, gpu_cap=64_000, host_cap=v.peak, bw_out=(10**6, 10**6), bw_in=(10**6, 10**6))
    p = v.plan(**a)
    assert len(p.records) == n - 1
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches <= n // 64 + 4        # (a launch takes 64 rounds, and each commits a migration)
    h.close()


def test_host_memory_tested_slot_by_slot_in_every_pass(g10):
    """Periods that lie side by side, flash too slow for any of them, host memory for one tensor and a half: the bound of a
    chunk's host occupancy never suffices, so every migration waits for the exact test of a pass of its own."""
    n = 18000
    K, i = 5 * n + 8, np.arange(n, dtype=np.int64)
    tr = Trace("side_by_side", np.full(K, 1000, np.uint64), (64_000 + 2 * ((i * 7919) % n)).astype(np.uint64), np.zeros(n, np.uint8),
               np.concatenate([4 + 5 * i, 8 + 5 * i]).astype(np.uint32), np.concatenate([i, i]).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.1, host_cap_frac=0.3))
    a = dict(args, gpu_cap=32_000, host_cap=150_000, bw_out=(1, 10**6), bw_in=(1, 10**6), max_iters=9800)
    p = v.plan(**a)
    assert len(p.records) == 9800
    assert_plan_equal(h.plan(**a), p)
    h.close()
