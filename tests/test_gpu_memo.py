"""The scoring kernel of the ratio key keeps every candidate's key and scores again only what a migration to flash may have
moved to host: plans with many migrations to flash, against the oracle, record by record."""
import pytest

from paper_2310_09443_amd import traces
from test_gpu_parity import assert_plan_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flash, host, host_share", [
    (30000, 12000, 1.0),      # flash is the cheaper destination: every migration goes there
    (2000, 2000, 1.0),        # equal costs, long windows: the destination changes with every second migration
    (9000, 12000, 0.02),      # host memory for a few hundred of the 1500
])
def test_keys_kept_between_passes(g10, flash, host, host_share):
    w = traces.stress(K=8000, N=100000, seed=0x67100016)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.2), host_cap=int(v.peak * host_share), bw_out=(flash, host), bw_in=(flash, host))
    for limit in (1500, 130):        # (re-tiled in between; a limit between two re-tilings)
        r = h.plan(rank=1, max_iters=limit, **a)
        assert r.loop_wide_rounds > 0            # (the scoring kernel took part; where bound and key are one, lists are soon short)
        assert_plan_equal(r, v.plan(rank=1, max_iters=limit, **a))
    h.close()
