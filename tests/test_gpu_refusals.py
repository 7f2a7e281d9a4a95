"""Plans whose host memory refuses candidates by the hundred: several of them go in one round of the loop kernel, in a form of
its own that a plan changes to after its eighth.  Against the oracle, record by record."""
import pytest

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
    assert_plan_equal(h.plan(**a), p)
    # chunks of several strips of 256 slots; one tile
    assert_plan_equal(h.plan(max_tiles=1, max_chunks=2, **a), p)
    # ends in the middle of a round, before and behind the change of form
    first = int(p.null_iters[0])
    for limit in (first + 1, first + 8, first + 9, first + 37):
        assert_plan_equal(h.plan(max_iters=limit, **a), v.plan(max_iters=limit, **a))
    h.close()


def test_batch_of_plans_with_and_without_refusals(g10):
    w = traces.stress(K=2011, N=9001, seed=23)
    h, v, args = run_both(g10, w)
    sweep = [_args(args, v, 0.3, host, 6000) for host in (0.5, 0.01, 0.03, 1.0)]
    for d, r in zip(sweep, h.plan_batch(sweep)):
        assert_plan_equal(r, v.plan(**d))
    h.close()
