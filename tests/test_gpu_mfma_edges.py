"""Dense 4- to 6-qubit gates on the matrix cores at the edges of their tiles, element by element against the oracle:
states of fewer groups than a tile has columns, one tile, several; targets in, around and above the lines; controls
beside them, on qubit 0 too."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


def _check(gpu, n, dtype, k, targets, controls=(), seed=0):
    rng = np.random.Generator(np.random.PCG64(700 + seed))
    U = C._random_unitary(rng, 1 << k)
    psi = C.random_state(n, 710 + seed)
    if dtype == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    st = gpu.State(n, dtype)
    st.set(psi)
    if controls:
        st.apply_controlled(controls, targets, U)
        oracle.apply_controlled(psi, controls, targets, U)
    else:
        st.apply_gate(targets, U)
        oracle.apply_dense(psi, targets, U)
    got = st.get()
    st.close()
    # a row's products sum to at most 1 in modulus (unit rows, unit state): 2 2^k real terms, each rounded once on its
    # way into the sum, on both sides; complex64 also rounds the matrix entries and the result
    eps = 2.0 ** -53 if dtype == "c128" else 2.0 ** -24
    assert np.max(np.abs(got - psi)) <= 2 * (2 * (1 << k) + 4) * eps


# a tile holds 16 groups (k = 6 complex128) up to 128 (k = 4 complex64): n - k = 0..8 covers a part of one, one and two
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("k", [4, 5, 6])
def test_few_groups(gpu, k, dtype):
    rng = np.random.Generator(np.random.PCG64(720 + k))
    for extra in range(0, 9):
        n = k + extra
        _check(gpu, n, dtype, k, tuple(int(v) for v in rng.permutation(n)[:k]), seed=extra)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("k", [4, 5, 6])
def test_target_positions(gpu, k, dtype):
    n = 17
    for i, t in enumerate([range(k), range(1, k + 1), range(3, 3 + k), range(n - k, n), [0] + list(range(n - k + 1, n)),
                           [16, 0, 9, 4, 13, 2][:k]]):
        _check(gpu, n, dtype, k, tuple(t), seed=20 + i)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("k,targets,controls", [(4, (1, 2, 3, 4), (0,)), (4, (8, 2, 11, 5), (0, 3)), (5, (0, 1, 2, 3, 4), (6,)),
                                                (5, (9, 8, 7, 6, 5), (0, 1, 2, 3, 4)), (6, (1, 3, 5, 7, 9, 11), (0, 2)),
                                                (6, (11, 10, 9, 8, 7, 6), (5, 1)), (6, (0, 1, 2, 3, 4, 5), (12,))])
def test_controls(gpu, k, targets, controls, dtype):
    _check(gpu, 13, dtype, k, targets, controls, seed=40 + k)


@pytest.mark.parametrize("n,dtype", [(24, "c128"), (25, "c64")])
def test_non_temporal_sizes(gpu, n, dtype):
    """256 MiB states: the first that take non-temporal accesses."""
    for k in (4, 5, 6):
        _check(gpu, n, dtype, k, (0, 13, 7, n - 1, 3, n - 2)[:k], seed=60 + k)
