"""The two walks behind a plan, smart prefetching and the replay, at the sizes where their forms change: windows that go
around the timeline and end in one chunk, chunks of one strip and of several, many events at one point, iteration times
at the limit of the replay's arithmetic in doubles.  Against the oracle; every comparison is exact."""
import numpy as np
import pytest

from paper_2310_09443_amd import traces
from paper_2310_09443_amd.traces import Trace, Workload
from test_gpu_parity import assert_plan_equal, assert_prefetch_equal, g10, run_both  # noqa: F401  (g10 is a fixture)
from test_gpu_replay import both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_chunks", [0, 1, 2])
@pytest.mark.parametrize("K", [130, 256, 257, 1000, 1537])
def test_prefetch_windows_around_the_timeline(g10, K, max_chunks):
    """Global tensors used twice, close together: their other period goes around, nearly a whole iteration long."""
    i = np.arange(6 * K, dtype=np.uint64)
    at = traces.rand_int(7, 1, i, 0, K - 8).astype(np.uint32)
    tr = Trace(f"around{K}", traces.rand_int(7, 2, np.arange(K, dtype=np.uint64), 2000, 90000).astype(np.uint64),
               traces.rand_int(7, 3, i, 4096, 4 << 20).astype(np.uint64), np.ones(len(i), np.uint8),
               np.concatenate([at, at + 1 + (i % 5).astype(np.uint32)]), np.concatenate([i, i]).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.5, host_cap_frac=0.3))
    for cap in (0.4, 0.8, 0.95):
        a = dict(args, gpu_cap=int(v.peak * cap))
        p = v.plan(**a)
        assert len(p.records)
        assert_plan_equal(h.plan(max_chunks=max_chunks, **a), p)
        assert_prefetch_equal(h.prefetch(), p.prefetch())
    h.close()


@pytest.mark.parametrize("total", [(1 << 48) // 10 - 1, (1 << 48) // 10, (1 << 48) // 10 + 1])
def test_replay_times_at_the_limit_of_doubles(g10, total):
    """From 2^48 / 10 ns of kernel time on, of the plan's or of the replay's durations, the replay works in whole numbers."""
    w = traces.stress(K=400, N=3000, seed=21)
    d = np.full(400, total // 400, np.uint64)
    d[7] += np.uint64(total - int(d.sum()))
    h, v, args = run_both(g10, Workload(traces.with_durations(w.trace, d), cap_frac=0.3, host_cap_frac=0.1))
    a = dict(args, bw_out=(1, 3), bw_in=(1, 2))
    p = v.plan(**a)
    assert len(p.records)
    assert_plan_equal(h.plan(**a), p)
    both(h, p, (None, d // np.uint64(3), d + np.uint64(5)))
    h.close()


@pytest.mark.parametrize("n", [1, 10, 11, 21, 22, 64, 200])
def test_replay_of_many_events_at_one_point(g10, n):
    """All evictions at one point, all prefetches at one, all uses at one: whole wavefronts of one kind, on one channel and two."""
    K = 200
    uk = np.concatenate([np.full(n, 3), np.full(n, 190)]).astype(np.uint32)
    ut = np.concatenate([np.arange(n), np.arange(n)]).astype(np.uint32)
    tr = Trace(f"point{n}", np.full(K, 40_000, np.uint64), (1000 + np.arange(n) % 7).astype(np.uint64), np.zeros(n, np.uint8), uk, ut)
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.05, host_cap_frac=0.4))
    for host in (0.0, 0.4, 1.0):
        a = dict(args, host_cap=int(v.peak * host), bw_out=(200, 300), bw_in=(200, 300))
        p = v.plan(**a)
        assert len(p.records)
        assert_plan_equal(h.plan(**a), p)
        both(h, p, (None, np.full(K, 1, np.uint64), np.full(K, 90_000, np.uint64)))
    h.close()


@pytest.mark.parametrize("n", [63, 65, 128, 129, 191, 192, 193, 255, 256, 257, 320, 513])
def test_replay_of_predecessors_at_every_distance(g10, n):
    """n events between an event and the one it waits for: among the 64 events that are walked at a time, among the last 192, in memory."""
    test_replay_of_many_events_at_one_point(g10, n)
