"""The sorts and scans at the sizes where they change form - sorts in one workgroup up to 8192 keys and in tiles of 2048
above, scans whose tile sums every workgroup adds up itself up to 2048 tiles and that scan them first above - through the
analysis, whose arrays are compared with the oracle's, element by element."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2310_09443_amd import binding, traces
from paper_2310_09443_amd.traces import Trace, Workload
from test_gpu_parity import assert_plan_equal, g10, run_both  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


def _trace(P, K, N, seed):
    i = np.arange(P, dtype=np.uint64)
    return Trace(f"pairs{P}", np.full(K, 1000, np.uint64), traces.rand_int(seed, 1, np.arange(N), 1, 1 << 20).astype(np.uint64),
                 (traces.rand_unit(seed, 2, np.arange(N)) < 0.2).astype(np.uint8),
                 traces.rand_int(seed, 3, i, 0, K - 1).astype(np.uint32), traces.rand_int(seed, 4, i, 0, N - 1).astype(np.uint32))


@pytest.mark.parametrize("K,N", [(3, 2), (300, 70000), (70000, 40)])
@pytest.mark.parametrize("P", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 8191, 8192, 8193, 10241, 30000])
def test_sorted_uses_and_periods(P, K, N):
    tr = _trace(P, K, N, seed=P)
    v = O.Vitality(tr, O.PREFIX)
    dt = binding.DeviceTrace(tr)
    h = binding.g10_vitality(dt)
    s = binding.g10_vitality_static(dt)
    for x in (h, s):
        assert (x.n_uses, x.C, x.peak) == (v.n_uses, len(v.per_L), v.peak)
        for f in ("use_off", "use_k", "per_tensor", "per_L", "per_R", "start", "pressure"):
            assert np.array_equal(getattr(x, f), np.asarray(getattr(v, f))), f
    h.close()


TILES = 2048 * 2048            # elements in 2048 tiles


@pytest.mark.parametrize("P", [TILES, TILES + 1, 2 * TILES + 70_001])
def test_tile_sums_scanned_first(g10, P):
    """2048 tiles of pairs, one more, and so many that the periods and the candidates of a plan fill more than 2048 too;
    with duplicate pairs, and periods that run into the next iteration."""
    n, K = P * 100 // 201, 5000
    i = np.arange(n, dtype=np.uint64)
    first, last = traces.rand_int(6, 1, i, 0, 2000).astype(np.uint32), traces.rand_int(6, 2, i, 2500, K - 1).astype(np.uint32)
    tr = Trace(f"pairs{P}", traces.rand_int(6, 3, np.arange(K), 500, 1500).astype(np.uint64), traces.rand_int(6, 4, i, 512, 4096).astype(np.uint64),
               (i % 1001 == 1000).astype(np.uint8), np.concatenate([last, first, first[:P - 2 * n]]),
               np.concatenate([i, i, i[:P - 2 * n]]).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.5, host_cap_frac=0.1))
    assert len(tr.use_kernel) == P and v.n_uses == 2 * n and len(v.per_L) > n
    assert P <= TILES + 1 or n > TILES
    a = dict(args, max_iters=8)
    assert_plan_equal(h.plan(**a), v.plan(**a))
    h.close()


@pytest.mark.parametrize("K", [TILES, TILES + 1, TILES + 2047])
def test_many_kernels(g10, K):
    """The same for the start times and the pressure, whose scan also takes the peak."""
    i = np.arange(4000, dtype=np.uint64)
    tr = Trace(f"kernels{K}", traces.rand_int(8, 1, np.arange(K), 500, 1500).astype(np.uint64), traces.rand_int(8, 2, np.arange(400), 1 << 20, 1 << 24).astype(np.uint64),
               (np.arange(400) % 10 == 9).astype(np.uint8), traces.rand_int(8, 3, i, 0, K - 1).astype(np.uint32), (i % 400).astype(np.uint32))
    h, v, args = run_both(g10, Workload(tr, cap_frac=0.5, host_cap_frac=0.1))
    a = dict(args, max_iters=40)
    assert_plan_equal(h.plan(**a), v.plan(**a))
    h.close()
