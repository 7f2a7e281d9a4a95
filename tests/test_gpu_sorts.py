"""The sorts at the sizes where they change form - one workgroup up to 8192 keys, tiles of 2048 above - through the
analysis, whose arrays are compared with the oracle's, element by element."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2310_09443_amd import binding, traces
from paper_2310_09443_amd.traces import Trace

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
