"""The greedy loop at the sizes where its chunk jobs, its list of a pass and its 32-bit sums can go wrong, against the
oracle through the C ABI.  Integer work: every comparison is exact."""
import numpy as np
import pytest

from paper_2310_09443_amd import traces
from paper_2310_09443_amd.traces import Trace, Workload
from test_gpu_parity import assert_plan_equal, assert_prefetch_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_chunks", [0, 1, 2])
@pytest.mark.parametrize("K", [8, 63, 64, 65, 255, 256, 257, 321, 512, 513, 767])
def test_ragged_chunks(g10, K, max_chunks):
    """A chunk's slots go to the lanes 64 apart: last chunks of one slot, of one and of several rounds of lanes."""
    w = traces.stress(K=K, N=12 * K, seed=K)
    h, v, args = run_both(g10, w)
    for cap, host in ((0.25, 0.25), (0.6, 0.02), (0.9, 2.0)):
        a = dict(args, gpu_cap=int(v.peak * cap), host_cap=int(v.peak * host))
        p = v.plan(**a)
        assert_plan_equal(h.plan(max_chunks=max_chunks, **a), p)
    assert_prefetch_equal(h.prefetch(), p.prefetch())
    h.close()


def _equal_tensors(n, K, dur):
    """n tensors of one size, used at the same two kernels of their group: every ranking ends in ties."""
    g = np.arange(n, dtype=np.int64) % 3
    first, last = 1 + g, K - 2 - g
    uk = np.concatenate([first, last]).astype(np.uint32)
    ut = np.concatenate([np.arange(n), np.arange(n)]).astype(np.uint32)
    tr = Trace(f"equal{n}", np.full(K, dur, np.uint64), np.full(n, 64_000, np.uint64), np.zeros(n, np.uint8), uk, ut)
    return Workload(tr, cap_frac=0.1, host_cap_frac=0.3)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 700])
def test_list_of_equal_candidates(g10, n):
    """Ties by the dozen: the list of a pass is full of them, or overflows (64 entries)."""
    h, v, args = run_both(g10, _equal_tensors(n, 300, 5000))
    for host in (0.3, 1.0):
        a = dict(args, host_cap=int(v.peak * host))
        assert_plan_equal(h.plan(**a), v.plan(**a))
        assert_plan_equal(h.plan(max_iters=n // 2 + 1, **a), v.plan(max_iters=n // 2 + 1, **a))
    h.close()


@pytest.mark.parametrize("dur", [16_777_215, 16_777_216, 16_777_217, 1 << 33, 1 << 45])
def test_long_kernels(g10, dur):
    """Chunk totals (256 slots) a little below and above 2^32 ns, and far above."""
    w = traces.stress(K=600, N=6000, seed=9)
    tr = w.trace
    d = np.where(np.arange(tr.K) % 2 == 0, np.uint64(dur), np.uint64(max(dur - 3, 1))).astype(np.uint64)
    d[300:] = np.uint64(dur)
    w = Workload(traces.with_durations(tr, d), cap_frac=0.3, host_cap_frac=0.1, bw_out_Bpus=(1, 3), bw_in_Bpus=(1, 2))
    h, v, args = run_both(g10, w)
    for bw in ((1, 3), (700, 2000), (6000, 25000)):
        a = dict(args, bw_out=bw, bw_in=bw)
        assert_plan_equal(h.plan(**a), v.plan(**a))
    h.close()


@pytest.mark.parametrize("total", [(1 << 32) - 1, 1 << 32, (1 << 32) + 1])
def test_chunk_totals_at_32_bits(g10, total):
    """Every full chunk's total exactly at the last value that its jobs sum in 32 bits, and one and two above it."""
    w = traces.stress(K=700, N=7000, seed=10)
    d = np.full(w.trace.K, 1 << 24, np.uint64)
    d[100:512:256] = np.uint64(total - 255 * (1 << 24))
    assert d[:256].sum() == total and d[256:512].sum() == total
    w = Workload(traces.with_durations(w.trace, d), cap_frac=0.3, host_cap_frac=0.1)
    h, v, args = run_both(g10, w)
    for bw in ((1, 3), (700, 2000), (6000, 25000)):
        a = dict(args, bw_out=bw, bw_in=bw)
        p = v.plan(**a)
        assert len(p.records)
        assert_plan_equal(h.plan(**a), p)
    h.close()


@pytest.mark.parametrize("K,n", [(131_072, 7899 * 256), (131_072, 7899 * 256 + 1), (131_072, 8192 * 256), (127_232, 8192 * 256), (127_233, 8192 * 256)])
def test_most_chunks_and_most_tiles(g10, K, n):
    """497, 498 and 512 chunks of 256 slots with as many tiles of 256 candidates as fit the LDS beside them, and one more:
    the first passes of the plan, with both ranking keys (every tensor is one candidate with a window either way)."""
    i = np.arange(n, dtype=np.uint64)
    first = traces.rand_int(5, 1, i, 0, K // 2 - 1).astype(np.uint32)
    last = traces.rand_int(5, 2, i, K // 2 + 64, K - 1).astype(np.uint32)
    tr = Trace(f"limits{n}", np.full(K, 1000, np.uint64), traces.rand_int(5, 3, i, 4096, 65536).astype(np.uint64), np.zeros(n, np.uint8),
               np.concatenate([first, last]), np.concatenate([i, i]).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.5, host_cap_frac=0.1))
    for rank in (0, 1):
        a = dict(args, max_iters=24, rank=rank)
        assert_plan_equal(h.plan(**a), v.plan(**a))
        assert h._counters(0).score_full_cands == n
    h.close()


@pytest.mark.parametrize("cap,host", [(0.15, 0.02), (0.3, 0.25), (0.6, 0.05), (0.85, 2.0)])
@pytest.mark.parametrize("K,N", [(90, 300), (257, 1500), (600, 2600)])
def test_clipped_areas_that_are_their_bands_and_others(g10, K, N, cap, host):
    """Plans by the clipped area, in the form that commits several migrations a pass where their areas are bands: excesses above and
    below the tensors' sizes, limits in the middle of a round; alone and beside a plan that stays in the other form."""
    w = traces.stress(K=K, N=N, seed=K + N)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * cap), host_cap=int(v.peak * host), area=1)
    p = v.plan(**a)
    assert_plan_equal(h.plan(**a), p)
    for limit in (9, 40, 77):
        assert_plan_equal(h.plan(max_iters=limit, **a), v.plan(max_iters=limit, **a))
    b = dict(a, gpu_cap=int(v.peak * 0.97))
    rs = h.plan_batch([a, b])
    assert_plan_equal(rs[0], p)
    assert_plan_equal(rs[1], v.plan(**b))
    h.close()


@pytest.mark.parametrize("host", [0.02, 0.4])
@pytest.mark.parametrize("K,N,max_chunks", [(1024, 9000, 0), (1025, 9000, 0), (11264, 14000, 0), (11265, 14000, 0), (3000, 20000, 3)])
def test_chunk_test_of_few_and_many_chunks(g10, K, N, max_chunks, host):
    """Up to 44 chunks a round of eight picks or more is tested a row of lanes per chunk: rows left over, one chunk more, both destinations."""
    w = traces.stress(K=K, N=N, seed=K)
    h, v, args = run_both(g10, w)
    for cap in (0.3, 0.7):
        a = dict(args, gpu_cap=int(v.peak * cap), host_cap=int(v.peak * host))
        p = v.plan(max_iters=600, **a)
        assert_plan_equal(h.plan(max_iters=600, max_chunks=max_chunks, **a), p)
    h.close()


def test_rounds_of_many_picks_on_few_chunks(g10):
    """23 chunks and, on average, more than the eight migrations a round from which rows of lanes test the chunks."""
    w = traces.resnet152()
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.4), host_cap=int(v.peak * 0.25), bw_out=(12000, 25000), bw_in=(12000, 25000))
    r = h.plan(**a)
    assert_plan_equal(r, v.plan(**a))
    assert r.n_migrations > 8 * (r.loop_passes + r.loop_more_rounds)
    h.close()


def test_no_change_of_form_near_the_limit(g10):
    """A plan by the clipped area whose limit leaves it a few passes stays in the form it is in (a change is another launch)."""
    w = traces.stress(K=90, N=300)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.3), host_cap=int(v.peak * 0.25), bw_out=(12000, 25000), bw_in=(12000, 25000), area=1)
    p = v.plan(**a)
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches > 1 and r.loop_more_rounds > 0          # it changes where nothing limits it
    for limit in (10, 13, 16):
        r = h.plan(max_iters=limit, **a)
        assert_plan_equal(r, v.plan(max_iters=limit, **a))
        assert r.n_iterations == limit and r.loop_launches == 1
    h.close()


def test_change_of_form_in_a_batch(g10):
    """Beside other plans a plan ends its launch for the first change of form only: it is not held at every one until theirs end."""
    w = traces.stress(K=600, N=2600)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.4), host_cap=int(v.peak * 0.25), bw_out=(12000, 25000), bw_in=(12000, 25000), area=1)
    p = v.plan(**a)
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches > 2                         # (alone: a launch for every change)
    for r in h.plan_batch([a, a]):
        assert_plan_equal(r, p)
        assert r.loop_launches == 2                    # (1.5 ms; a launch may take 2)
    h.close()


def test_batch_of_all_forms(g10):
    """Both keys, both readings, plans that refuse candidates and plans with lists: launches side by side, several of each."""
    w = traces.encoder12()
    h, v, args = run_both(g10, w)
    tight = dict(args, gpu_cap=int(v.peak * 0.3), host_cap=int(v.peak * 0.004), bw_out=(400, 25000), bw_in=(400, 25000))
    clip = dict(args, gpu_cap=int(v.peak * 0.6), area=1)
    ps = [clip, tight, dict(args), dict(args, rank=1, max_iters=300), dict(clip, rank=1, max_iters=40), dict(clip, gpu_cap=int(v.peak * 0.9), max_iters=40),
          dict(tight, host_cap=0), dict(tight, area=1, max_iters=30)]
    want = [v.plan(**dict(a, max_iters=a.get("max_iters", 2 ** 64 - 1))) for a in ps]
    for _ in range(2):
        rs = h.plan_batch(ps)
        for r, p in zip(rs, want):
            assert_plan_equal(r, p)
    assert rs[1].loop_launches > 1 and rs[1].loop_passes < len(want[1].records) + len(want[1].null_cands)      # (it refuses several a round)
    h.close()


@pytest.mark.parametrize("N,flash,host,limit", [(14000, 800, 0.005, 60), (8000, 32000, 0.25, 120)])
def test_lists_of_the_clipped_area_on_many_chunks(g10, N, flash, host, limit):
    """46 chunks, more than rows of lanes take: candidates that host memory refuses while the plan makes lists; lists that commit several."""
    w = traces.stress(K=11600, N=N)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.3), host_cap=int(v.peak * host), bw_out=(flash, 25000), bw_in=(flash, 25000), area=1, max_iters=limit)
    p = v.plan(**a)
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches >= 3                        # (into the form with lists and out of it)
    if host < 0.01:
        assert len(p.null_iters) > 40
    else:
        assert r.loop_more_rounds > 0 and r.loop_passes < r.n_iterations
    h.close()
