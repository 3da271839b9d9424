"""Dense 5- and 6-qubit gates on both sides of the number of tiles from which these are whole: fewer tiles than compute
units are half as large."""
import pytest

from test_gpu_mfma_edges import _check

pytestmark = pytest.mark.gpu


# 256 whole tiles: 18 qubits for k = 5 complex128, 19 for complex64
@pytest.mark.parametrize("n,dtype", [(17, "c128"), (18, "c128"), (18, "c64"), (19, "c64")])
@pytest.mark.parametrize("k", [5, 6])
def test_both_tile_sizes(gpu, n, dtype, k):
    for i, (t, c) in enumerate([((0, 1, 2, 3, 4, 5), ()), ((n - 1, 2, 9, 0, 12, 5), ()), ((4, 13, 7, n - 1, 10, n - 2), (3,)),
                                ((1, 2, 3, n - 1, 6, 11), (0,))]):
        _check(gpu, n, dtype, k, t[:k], c, seed=140 + 10 * k + i)
