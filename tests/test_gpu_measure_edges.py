"""Measurement and sampling where their kernels change form: the smallest states, both halves of a complex64 vector,
one and many partial sums, one and many chunks and scan tiles, few and many shots, states with massless regions."""
import numpy as np
import pytest

import circuits as C
from oracle import measure as M

pytestmark = pytest.mark.gpu


def _state(gpu, n, dtype, seed, sparse=False):
    psi = C.random_state(n, seed)
    if sparse:  # mass on a few scattered runs only
        keep = np.zeros(1 << n, dtype=bool)
        rng = np.random.Generator(np.random.PCG64(seed))
        for i in rng.integers(0, 1 << n, size=5):
            keep[int(i):int(i) + 3] = True
        psi = np.where(keep, psi, 0.0)
    if dtype == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    st = gpu.State(n, dtype)
    st.set(psi)
    return st, psi


# n = 1, 2: fewer vectors than lanes; 12, 13: one and two partial sums; 19: remainders of the four-load loop;
# 23: the largest number of partial sums
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 7, 12, 13, 19, 23])
def test_measure_edges(gpu, n, dtype):
    # the masses are FP64 sums of at most 2^11 terms per thread, then compensated: 2^11 eps relative is a bound on
    # each; the state's rounding to FP32 bounds the complex64 collapse (amplitudes below 1: one half unit, 2^-24)
    for q in sorted({0, 1 % n, n // 2, n - 1}):
        for u in (0.03, 0.97):
            st, psi = _state(gpu, n, dtype, 100 + n)
            out, p1 = st.measure(q, u)
            o_ref, p_ref, ref = M.measure(psi, q, u)
            assert out == o_ref and abs(p1 - p_ref) <= 2.0 ** -41
            assert np.max(np.abs(st.get() - ref)) <= (2.0 ** -41 if dtype == "c128" else 2.0 ** -23)
            st.close()


# chunks of 2048: n = 10 a part of one, 11 one, 12 two; n = 22 one scan tile, 23 two; shots 32768 / 32769: the two ways
# uniforms and indices travel
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,shots,sparse", [(1, 1, False), (2, 64, False), (5, 300, True), (10, 500, False),
                                            (11, 32769, False), (12, 32768, True), (16, 40000, True),
                                            (22, 3000, False), (23, 3000, True)])
def test_sample_edges(gpu, n, shots, sparse, dtype):
    st, psi = _state(gpu, n, dtype, 200 + n, sparse)
    u = np.random.Generator(np.random.PCG64(300 + n)).uniform(size=shots)
    u[0] = 0.0
    u[-1] = np.nextafter(1.0, 0.0)
    for _ in range(2):  # the second call reuses the state's scratch
        idx = st.sample(u)
        assert M.samples_valid(psi, u, idx).all()
        # an index may differ from the oracle's only where a cumulative sum ties with the target to rounding
        assert int(np.sum(idx != M.samples(psi, u))) <= 2
    st.close()


def test_measure_refuses_a_state_without_finite_mass_and_leaves_it(gpu):
    for bad in (0.0, np.nan, np.inf):
        st = gpu.State(6, "c64")
        psi = np.full(64, bad, dtype=np.complex64)
        st.set(psi)
        with pytest.raises(gpu.binding.QSError):
            st.measure(3, 0.5)
        with pytest.raises(gpu.binding.QSError):
            st.sample([0.5])
        assert st.get().tobytes() == psi.tobytes()
        st.close()
