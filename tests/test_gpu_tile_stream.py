"""Plain runs on states that stream from HBM: passes over tiles with non-temporal accesses, the tiles handed out in runs
per XCD, bit for bit the single calls' results; the last cached size beside them."""
import numpy as np
import pytest

import circuits as C

from test_gpu_tile_runs import _narrow_op, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [(24, "c128"), (25, "c128"), (25, "c64"), (26, "c64")])
def test_matches_single_calls(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(980 + n))
    ops = [_narrow_op(rng, n, ("dense", "move", "diag", "cdense", "cmove")) for _ in range(24)]
    ops.insert(12, C.Op("fswap", p=2, q=n - 5, s=4))
    got, calls = _run(gpu, n, dtype, ops, C.random_state(n, 981 + n))
    assert got.tobytes() == calls.tobytes()
