"""The scoring kernel of the ratio key, and the keys it keeps between passes on lists of 2^19 candidates and more, of which it
scores again only those that a migration to flash may have moved to host: plans with many migrations to flash, against the
oracle, record by record."""
import numpy as np
import pytest

from paper_2310_09443_amd import traces
from paper_2310_09443_amd.traces import Trace, Workload
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


@pytest.mark.parametrize("flash, host, taken_again", [
    (6000, 25000, False),     # keys on flash a little under a quarter of those to host
    (12000, 96000, True),     # ... an eighth: migrations to flash and to host by turns, rounds whose best lies under a kept key
    (300, 2400, True),        # the same with long windows, most of which meet: too many such rounds, nothing is kept any more
    (30000, 12000, False),    # bound and key are one
])
def test_keys_kept_on_long_lists(g10, flash, host, taken_again):
    w = traces.stress(K=20000, N=640000, seed=0x67100017)
    h, v, args = run_both(g10, w)
    a = dict(args, gpu_cap=int(v.peak * 0.2), host_cap=v.peak, bw_out=(flash, host), bw_in=(flash, host), rank=1, max_iters=300)
    r = h.plan(**a)
    assert h._counters(0).score_full_cands >= 1 << 19
    assert r.loop_wide_rounds > 128
    if taken_again:
        assert r.loop_second_rounds > 0
    assert_plan_equal(r, v.plan(**a))
    h.close()


def _struck_between_long_rounds():
    """A candidate `c` that the policy keeps on flash when a long round scores it, that a migration to flash (`w`) then pushes
    to host, and that a short round of the loop kernel's own finds pushed out before the next long round comes to it.

    Slots of 1 ms; a common tensor takes 0.9 of one on flash and an eighth of that to host, so its key is 0.05 a ns of
    over-capacity time on flash and 0.4 to host; in slots of that time, 1 and 8:
      pass 1  tile 0 alone: z (host only, 1160), whose size takes all pressure over the capacity out of [100, 244]
      pass 2  long: tile 0 and the tiles of A (bounds 1152, dead behind z).  c 74 on flash, 592 to host; w 980 on flash wins
      pass 3  short, tiles 0 and 35: w has taken the eviction slot of c and the prefetch slot of x; both go to host now; x 976 wins
      pass 4  short, tile 35 alone: nothing left there; then long: tile 0 and the tiles of B (bounds 600, 75 on flash).
              Two migrations lie between this round and the last one that scored c, and c wins with 592.
    """
    s, slot = 90_000, 1_000_000
    uses, size = [], []

    def add(n, first, last, sz=s):
        size.extend([sz] * n)
        uses.extend([(first, last)] * n)

    add(1, 129, 1226)                     # w: absent 131 .. 1224
    add(1, 129, 320)                      # c: absent 131 .. 318
    add(1, 79, 265, 16_000_000)           # z: 20 slots of transfer each way to host, too long on flash; absent 100 .. 244
    add(9000, 98, 245)                    # A: absent 100 .. 243
    add(1, 1101, 1226)                    # x: absent 1103 .. 1224
    add(212, 120, 222)                    # fills x's tile: absent 122 .. 220, dead behind z
    add(520_000, 400, 478)                # B: absent 402 .. 476 (so many that keys are kept)
    N, K = len(size), 1300
    i = np.arange(N)
    at = np.array(uses)
    # used by every kernel: no period, pressure everywhere but in [100, 244], where it is nearly flat
    ballast = [(N, 0, 99), (N + 1, 245, K - 1), (N + 2, 100, 119), (N + 3, 223, 244)]
    ut = np.concatenate([i, i] + [np.full(b - a + 1, t) for t, a, b in ballast])
    uk = np.concatenate([at[:, 0], at[:, 1]] + [np.arange(a, b + 1) for _, a, b in ballast])
    size = np.array(size + [600_000 * s] * 2 + [212 * s] * 2, np.uint64)
    tr = Trace("struck_between", np.full(K, slot, np.uint64), size, np.zeros(N + 4, np.uint8), uk.astype(np.uint32), ut.astype(np.uint32))
    return tr, s


def test_flash_struck_between_two_long_rounds(g10):
    tr, s = _struck_between_long_rounds()
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.5, host_cap_frac=1.0))
    a = dict(args, gpu_cap=int(v.pressure[150]) - 100 * s, host_cap=v.peak, bw_out=(100, 800), bw_in=(100, 800), rank=1, max_iters=12)
    p = v.plan(**a)
    assert p.records["tensor"][:4].tolist() == [2, 0, 9003, 1]             # z, w, x, c
    assert p.records["dest"][:4].tolist() == [1, 0, 1, 1]
    r = h.plan(**a)
    assert r.loop_wide_rounds >= 2 and h._counters(0).score_full_cands >= 1 << 19
    assert_plan_equal(r, p)
    h.close()
