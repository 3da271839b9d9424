"""Streaming one-pass kernels (diagonals of every width, scaling, lane-exchange gates, sparse diagonals, lane-order moves)
at the sizes where they change form: fewer vectors than lanes, the table in kernel arguments and in device memory, both
sides of the 256 MiB line between cached and non-temporal accesses, targets inside and above a block's vectors."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd import binding as B

pytestmark = pytest.mark.gpu


def _psi(n, dtype, seed):
    psi = C.random_state(n, seed)
    return psi.astype(np.complex64).astype(np.complex128) if dtype == "c64" else psi


# one product of a rounded entry and an amplitude below 1 (complex64: entry, two products, one sum: 4 half units)
EPS = {"c128": 4 * 2.0 ** -53, "c64": 4 * 2.0 ** -24}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 3, 6, 9, 10, 13, 17])
def test_diagonals(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(800 + n))
    for k in sorted({1, 2, 3, 6, 7, 12} & set(range(1, n + 1))):
        for unit in (0.0, 0.3, 0.8):  # entries of exactly 1 and -1 among them
            t = tuple(int(v) for v in rng.permutation(n)[:k])
            d = np.exp(1j * rng.uniform(0, 2 * np.pi, size=1 << k))
            u = rng.random(1 << k)
            d[u < unit] = 1.0
            d[u < unit / 2] = -1.0
            psi = _psi(n, dtype, 810 + k)
            psi[::5] = 0.0
            psi[1::7] = complex(-0.0, 0.0)
            st = gpu.State(n, dtype)
            st.set(psi)
            st.apply_diag(t, d)
            got = st.get()
            st.close()
            a = np.zeros(1 << n, dtype=np.int64)
            for j, q in enumerate(t):
                a |= ((np.arange(1 << n) >> q) & 1) << j
            same = d[a] == 1.0  # untouched: the same bits
            assert got[same].tobytes() == psi[same].astype(got.dtype).tobytes()
            ref = psi.copy()
            oracle.apply_diag(ref, t, d)
            assert np.max(np.abs(got - ref)) <= EPS[dtype]


@pytest.mark.parametrize("n,dtype", [(24, "c128"), (25, "c128"), (25, "c64"), (26, "c64")])
def test_both_sides_of_the_cache_line(gpu, n, dtype):
    """256 MiB (cached accesses) and 512 MiB (non-temporal) of state."""
    rng = np.random.Generator(np.random.PCG64(820))
    ph = np.exp(1j * rng.uniform(0, 6, size=512))
    psi = _psi(n, dtype, 821)
    X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
    U = C._random_unitary(rng, 2)
    st = gpu.State(n, dtype)
    cases = [("diag", (n - 1,), ph[:2]), ("diag", (3, 11), ph[:4]), ("diag", (2, 13, 20), ph[:8]),
             ("diag", (1, 4, 9, 12, 15, 18, 2), ph[:128]), ("diag", (5, 9), np.array([1, 1, 1, -1])),
             ("diag", (0, 1), np.array([1, 1, 1, -1])), ("ctrl", ((0,), (1,)), X), ("ctrl", ((20,), (9,)), X),
             ("gate", (2,), U), ("gate", (n - 2,), U)]
    for kind, t, m in cases:
        st.set(psi)
        ref = psi.copy()
        if kind == "diag":
            st.apply_diag(t, m)
            oracle.apply_diag(ref, t, m)
        elif kind == "ctrl":
            st.apply_controlled(*t, m)
            oracle.apply_controlled(ref, *t, m)
        else:
            st.apply_gate(t, m)
            oracle.apply_dense(ref, t, m)
        assert np.max(np.abs(st.get() - ref)) <= 2 * EPS[dtype], (kind, t)
    st.set(psi)
    B.qs_scale(st.h, 0.75)
    assert np.array_equal(st.get(), (psi * 0.75).astype(st.get().dtype))
    st.close()
