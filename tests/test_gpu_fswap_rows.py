"""Fused-swaps within the lowest bits on both sides of the line between the wide-row form and tiles (up to 64 tiles, spans of
3 to 9 bits, up to 1024 work items), against the oracle, bit for bit."""
import pytest

import circuits as C

from test_gpu_fswap_forms import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [11, 12, 14, 15, 17, 18, 19])
def test_both_forms(gpu, n, dtype):
    psi = C.random_state(n, 1230 + n)
    psi[::5] = complex(-0.0, 0.0)
    st = gpu.State(n, dtype)
    for span in (2, 3, 4, 5, 7, 8, 9, 10):
        for lo in range(0, 4):
            for s in sorted({1, 2, (span - lo) // 2}):
                if s >= 1 and lo + 2 * s <= span:
                    _check(st, psi, lo, span - s, s)
    st.close()
