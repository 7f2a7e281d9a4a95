"""The analysis at the sizes where it changes form: one launch for a tile of pairs with few kernels and tensors; sorts that
add their tiles' counts up in the scatter.  Against the oracle; every comparison is exact."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2310_09443_amd import traces
from paper_2310_09443_amd.traces import Trace
from test_gpu_parity import assert_vitality_equal, g10  # noqa: F401  (g10 is a fixture)

pytestmark = pytest.mark.gpu


def _trace(K, N, P, seed):
    i, k, n = (np.arange(x, dtype=np.uint64) for x in (P, K, N))
    return Trace(f"small{K}_{N}_{P}", traces.rand_int(seed, 1, k, 1, 90000).astype(np.uint64), traces.rand_int(seed, 2, n, 1, 1 << 30).astype(np.uint64),
                 (traces.rand_int(seed, 3, n, 0, 4) == 0).astype(np.uint8), traces.rand_int(seed, 4, i, 0, K - 1).astype(np.uint32),
                 traces.rand_int(seed, 5, i, 0, N - 1).astype(np.uint32))


@pytest.mark.parametrize("K,N,P", [(1, 1, 1), (2, 3, 5), (40, 7, 255), (40, 7, 256), (40, 7, 257), (300, 200, 2047), (300, 200, 2048), (300, 200, 2049),
                                   (4096, 4096, 2048), (4097, 4096, 2048), (4096, 4097, 2048), (2048, 1, 2048), (2049, 2, 2000),
                                   (500, 3000, 8192), (500, 3000, 8193), (700, 9000, 64 * 2048 - 1), (700, 9000, 64 * 2048), (700, 9000, 64 * 2048 + 1)])
@pytest.mark.parametrize("no_wrap", [False, True])
def test_analysis_at_its_limits(g10, K, N, P, no_wrap):
    tr = _trace(K, N, P, K + N + P)
    v = O.Vitality(tr, O.PREFIX, no_wrap=no_wrap)
    h = g10.g10_vitality(g10.DeviceTrace(tr), no_wrap=no_wrap)
    assert_vitality_equal(h, v)
    h.close()
