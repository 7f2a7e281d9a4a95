"""Plans whose host memory refuses candidates by the hundred: several of them go in one round of the loop kernel, in a form of
its own that a plan changes to after its eighth.  Against the oracle, record by record."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2310_09443_amd import traces
from test_gpu_parity import assert_plan_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


def _args(args, v, cap, host, flash):
    return dict(args, gpu_cap=int(v.peak * cap), host_cap=int(v.peak * host), bw_out=(flash, 25000), bw_in=(flash, 25000))


@pytest.mark.parametrize("trace, cap, host, flash", [("encoder", 0.3, 0.0, 400), ("encoder", 0.3, 0.004, 400), ("encoder", 0.3, 0.05, 400),
                                                     ("stress", 0.2, 0.0, 6000), ("stress", 0.2, 0.004, 6000), ("stress", 0.5, 0.004, 300)])
def test_many_refusals(g10, trace, cap, host, flash):
    w = traces.encoder12() if trace == "encoder" else traces.stress(K=1403, N=5003, seed=19)
    h, v, args = run_both(g10, w)
    a = _args(args, v, cap, host, flash)
    p = v.plan(**a)
    assert len(p.null_cands) > 40
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches > 1 and 2 * r.loop_passes < len(p.records) + len(p.null_cands)      # (in the form for it, several a round)
    # chunks of several strips of 256 slots; one tile
    assert_plan_equal(h.plan(max_tiles=1, max_chunks=2, **a), p)
    # ends in the middle of a round, before and behind the change of form
    first = int(p.null_iters[0])
    for limit in (first + 1, first + 8, first + 9, first + 37):
        assert_plan_equal(h.plan(max_iters=limit, **a), v.plan(max_iters=limit, **a))
    h.close()


def test_many_refusals_on_many_chunks(g10):
    """46 chunks: room looked up by more chunks than there are wavefronts, periods over all of them."""
    w = traces.stress(K=11600, N=14000)
    h, v, args = run_both(g10, w)
    a = _args(args, v, 0.3, 0.01, 300)
    p = v.plan(max_iters=1500, **a)
    r = h.plan(max_iters=1500, **a)
    assert_plan_equal(r, p)
    assert len(p.null_cands) > 1000 and 2 * r.loop_passes < 1500
    h.close()


def test_batch_of_plans_with_and_without_refusals(g10):
    w = traces.stress(K=2011, N=9001, seed=23)
    h, v, args = run_both(g10, w)
    sweep = [_args(args, v, 0.3, host, 6000) for host in (0.5, 0.01, 0.03, 1.0)]
    for d, r in zip(sweep, h.plan_batch(sweep)):
        assert_plan_equal(r, v.plan(**d))
    h.close()


def early_refusals(K, N, flash):
    """A stress trace in which the twelve tensors with the longest periods are too slow for the flash and the smallest of them one byte
    too large for the host: they win first and are refused, and nothing is behind them."""
    w = traces.stress(K=K, N=N)
    v = O.Vitality(w.trace, O.PREFIX)
    start, L, R = np.asarray(v.start).astype(np.int64), v.per_L.astype(np.int64), v.per_R.astype(np.int64)
    window = start[R % K] + (R // K) * start[K] - start[L + 1]
    longest = {}
    for i in np.argsort(-window, kind="stable"):
        longest.setdefault(int(v.per_tensor[i]), int(window[i]))
        if len(longest) == 12:
            break
    for t, ns in longest.items():
        w.trace.size_bytes[t] = ns * flash // 1000 * 6 // 10          # (out and in take 1.2 windows)
    sizes = [int(w.trace.size_bytes[t]) for t in longest]
    return w, dict(gpu_cap=sum(sizes) + v.peak // 10, host_cap=min(sizes) - 1, bw_out=(flash, 10 * flash), bw_in=(flash, 10 * flash))


def test_refusals_at_the_start_only(g10):
    """A plan leaves the form for refused candidates once none has been for long."""
    w, a = early_refusals(1100, 4200, 2_400_000)
    h, v, _ = run_both(g10, w)
    p = v.plan(**a)
    assert list(p.null_iters) == list(range(12)) and len(p.records) > 800
    r = h.plan(**a)
    assert_plan_equal(r, p)
    assert r.loop_launches == 3 and r.score_full_cands <= 8192      # (to that form and back; a list that is not re-tiled)
    for q in h.plan_batch([a, dict(a, host_cap=2 ** 50)]):
        if q.n_dropped:
            assert_plan_equal(q, p)
    h.close()


def test_refusals_of_a_plan_that_commits_one_migration_a_pass(g10):
    """With a tensor so large that several a round are not picked, the form for refused candidates has nothing to offer."""
    w, a = early_refusals(1500, 3000, 3_200_000)
    assert int(w.trace.size_bytes.max()) * 1000 >= 1 << 48
    h, v, _ = run_both(g10, w)
    p = v.plan(max_iters=200, **a)
    r = h.plan(max_iters=200, **a)
    assert_plan_equal(r, p)
    assert r.n_dropped >= 8 and r.loop_launches == 1 and r.loop_more_rounds == 0
    h.close()
