"""The picking of several migrations per round: transfer windows that meet on one channel, in one chunk and across many, in
both iterations; lists longer than a wavefront; times at the limit of the arithmetic in doubles.  Against the oracle through
the C ABI; integer work: every comparison is exact."""
import numpy as np
import pytest

from paper_2310_09443_amd import traces
from paper_2310_09443_amd.traces import Trace, Workload
from test_gpu_parity import assert_plan_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_chunks", [0, 1])
@pytest.mark.parametrize("bw", [(40, 130), (300, 300), (1500, 6000), (20000, 50000)])
@pytest.mark.parametrize("K", [300, 1100])
def test_windows_that_meet(g10, K, bw, max_chunks):
    """Slow channels: windows of a good part of the timeline, most of which meet, also around its end (a fifth of the
    tensors live across iterations); fast ones: windows of a slot or two."""
    w = traces.stress(K=K, N=9 * K, seed=K + bw[0])
    rng = np.random.default_rng(K)
    tr = w.trace
    tr = Trace(tr.name, tr.dur_ns, tr.size_bytes // np.uint64(64) + np.uint64(1), (rng.random(tr.N) < 0.2).astype(np.uint8), tr.use_kernel, tr.use_tensor)
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.3, host_cap_frac=0.2))
    for cap, host, b in ((0.3, 0.2, bw), (0.6, 0.03, bw), (0.15, 1.0, bw[::-1])):
        a = dict(args, gpu_cap=int(v.peak * cap), host_cap=int(v.peak * host), bw_out=b, bw_in=b)
        assert_plan_equal(h.plan(max_chunks=max_chunks, **a), v.plan(**a))
    h.close()


@pytest.mark.parametrize("n", [64, 65, 255, 256, 257, 600])
def test_long_lists(g10, n):
    """n candidates of nearly one benefit in 40 different places, some equal: more than a wavefront holds, more than a list holds."""
    i = np.arange(n, dtype=np.int64)
    K, at = 900, i % 40
    tr = Trace(f"near{n}", traces.rand_int(3, 1, np.arange(K, dtype=np.uint64), 900, 1100).astype(np.uint64), (64_000 + 2 * (i % 3)).astype(np.uint64),
               (i % 5 == 0).astype(np.uint8), np.concatenate([1 + 3 * at, K - 2 - 2 * at]).astype(np.uint32), np.concatenate([i, i]).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.1, host_cap_frac=0.4))
    for bw in ((6000, 25000), (300, 1000)):
        a = dict(args, bw_out=bw, bw_in=bw)
        assert_plan_equal(h.plan(**a), v.plan(**a))
        assert_plan_equal(h.plan(max_iters=n // 3 + 1, **a), v.plan(max_iters=n // 3 + 1, **a))
    h.close()


@pytest.mark.parametrize("total", [(1 << 48) - 1, 1 << 48, (1 << 48) + 1])
def test_iteration_times_at_the_limit_of_doubles(g10, total):
    """Below 2^48 ns of kernel time the rounds work in doubles, from there on in whole numbers, one migration a pass."""
    w = traces.stress(K=500, N=4000, seed=12)
    d = np.full(500, total // 500, np.uint64)
    d[250] += np.uint64(total - int(d.sum()))
    h, v, args = run_both(g10, Workload(traces.with_durations(w.trace, d), cap_frac=0.3, host_cap_frac=0.1))
    for bw in ((1, 3), (7, 2)):
        a = dict(args, bw_out=bw, bw_in=bw)
        p = v.plan(**a)
        assert len(p.records)
        assert_plan_equal(h.plan(**a), p)
    h.close()
