"""Fused-swaps in every form the launcher picks, against the oracle, bit for bit: within the lowest index bits (one tile,
and the first size past it), complex64 pairs with bit 0 left alone, in cache and streaming."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


def _check(st, psi, lo, hi, s):
    st.set(psi)
    st.fused_swap(lo, hi, s)
    ref = psi.copy()
    oracle.fused_swap(ref, lo, hi, s)
    assert st.get().tobytes() == ref.astype(st.get().dtype).tobytes(), (lo, hi, s)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [10, 11, 12, 13, 16])
def test_every_swap_of_small_states(gpu, n, dtype):
    psi = C.random_state(n, 1200 + n)
    psi[::5] = complex(-0.0, 0.0)
    st = gpu.State(n, dtype)
    for s in (1, 2, 3, 4, 5, 6, 8):
        for lo in range(0, n - 2 * s + 1, 1 if n < 13 else 2):
            for hi in sorted({lo + s, lo + s + 1, n - s, min(11, n) - s, min(12, n) - s, min(13, n) - s}):
                if lo + s <= hi <= n - s:
                    _check(st, psi, lo, hi, s)
    st.close()


@pytest.mark.parametrize("n,dtype", [(24, "c128"), (25, "c128"), (25, "c64"), (26, "c64")])
def test_both_sides_of_the_cache_line(gpu, n, dtype):
    psi = C.random_state(n, 1220)
    st = gpu.State(n, dtype)
    for lo, hi, s in ((0, 1, 1), (1, 2, 1), (2, 8, 3), (0, 6, 5), (1, 14, 2), (3, 12, 6), (4, 9, 2), (5, n - 4, 4),
                      (0, n - 6, 6), (2, n - 8, 8)):
        _check(st, psi, lo, hi, s)
    st.close()
