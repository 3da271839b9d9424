"""Sampling next to chunks without mass (a collapsed qubit above the chunk's bits): wherever a target falls, also on the
very sums of the prefix, the index has mass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 2048 chunks of 2048 amplitudes, one scan tile (n = 22), and two tiles (n = 23); runs of 8, 1 and 512 empty chunks: within
# the share of a scan thread, on its borders, many threads
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,bit", [(22, 3), (22, 0), (23, 3), (23, 9)])
def test_no_index_without_mass(gpu, n, bit, dtype):
    rng = np.random.Generator(np.random.PCG64(1000 * n + bit))
    nch = 1 << (n - 11)
    c = np.flatnonzero(((np.arange(nch) >> bit) & 1) == 0)
    psi = np.zeros(1 << n, dtype=np.complex128 if dtype == "c128" else np.complex64)
    # one amplitude per chunk, of magnitudes that make the sums round
    at = c * 2048 + rng.integers(0, 2048, size=c.size)
    psi[at] = rng.standard_normal(c.size) * 10.0 ** rng.uniform(-1.5, 0.0, size=c.size)
    mass = np.zeros(nch)
    mass[c] = psi[at].real.astype(np.float64) ** 2
    prefix = np.cumsum(mass.astype(np.longdouble)).astype(np.float64)
    total = prefix[-1]
    # targets on and around the prefix in front of each run of empty chunks. A prefix is rounded 3 + 8 times within its tile
    # and twice beyond: it lies within 13 half units of the true one, and so does the total.
    ends = np.unique(prefix[np.flatnonzero(np.diff((mass > 0).astype(int)) == -1)])
    u0 = ends / total
    u = (u0[:, None] + np.spacing(u0)[:, None] * np.arange(-24, 25)[None, :]).ravel()
    u = np.clip(u, 0.0, np.nextafter(1.0, 0.0))
    st = gpu.State(n, dtype)
    st.set(psi)
    idx = st.sample(u)
    st.close()
    assert (np.abs(psi[idx]) > 0).all()
    # and it is the amplitude that the target meets, to the same rounding
    where = np.searchsorted(prefix, u * total, side="right")
    got = idx >> 11
    off = 16 * np.spacing(total)  # both, and the product
    low = prefix[got] - mass[got]
    assert ((low <= u * total + off) & (u * total <= prefix[got] + off)).all(), int(np.sum(got != where))
