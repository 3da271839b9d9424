"""Dense 4- to 6-qubit gates on 512 MiB states, the first that stream from HBM: non-temporal tiles handed out in runs per
XCD, and for k = 4 groups in registers where neither a target nor a control lies inside a 128-byte line."""
import pytest

from test_gpu_mfma_edges import _check

pytestmark = pytest.mark.gpu


# targets above the lines and inside them; controls: none, above the lines, inside them (accesses through the cache)
@pytest.mark.parametrize("n,dtype", [(25, "c128"), (26, "c64")])
@pytest.mark.parametrize("k", [4, 5, 6])
def test_streaming_states(gpu, n, dtype, k):
    high, low = (4, 13, 7, n - 1, 10, n - 2)[:k], (0, 13, 7, n - 1, 3, n - 2)[:k]
    for i, (t, c) in enumerate([(high, ()), (low, ()), (high, (15,)), (high, (1, 18)), (low, (5,))]):
        print(n, dtype, t, c, flush=True)
        _check(gpu, n, dtype, k, t, c, seed=80 + 10 * k + i)
