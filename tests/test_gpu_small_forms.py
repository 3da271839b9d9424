"""Circuits that run in LDS in one launch: wide diagonals, gates with many controls and moves on 11 and 12 qubits, the
largest that do (complex128 with 12 where many operations are wide), two and four amplitudes a thread."""
import numpy as np
import pytest

import circuits as C
import oracle

from test_gpu_small_circuit import _run

pytestmark = pytest.mark.gpu
SIZES = [(11, "c128"), (12, "c128"), (11, "c64"), (12, "c64")]


def _check(gpu, n, dtype, ops, psi, tol):
    got, calls = _run(gpu, n, dtype, ops, psi)
    if dtype == "c64" or tol == 0.0:
        assert got.tobytes() == calls.tobytes()
    ref = psi.astype(got.dtype).astype(np.complex128)
    for op in ops:
        oracle.apply_op(ref, op)
    # at most 8 terms per amplitude and operation, 13 operations, amplitudes below 0.1
    assert np.max(np.abs(got - ref)) <= (1e-14 if dtype == "c128" else 1e-5)
    assert np.max(np.abs(got - calls)) <= tol


@pytest.mark.parametrize("n,dtype", SIZES)
def test_wide_diagonals_and_many_controls(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(560 + n))
    ops = []
    for k in (3, 6, 7, 9, n):
        t = tuple(int(v) for v in rng.permutation(n)[:k])
        d = np.exp(1j * rng.uniform(0, 2 * np.pi, size=1 << k))
        d[::4], d[1::4] = 1.0, -1.0
        ops.append(C.Op("diag", t, mat=d))
        phases = rng.choice([1, -1, 1j, -1j], size=1 << k).astype(np.complex128)
        ops.append(C.Op("diag", t[::-1], mat=phases))
    for k, nc in ((1, n - 1), (2, 5), (3, n - 3)):
        q = [int(v) for v in rng.permutation(n)[:k + nc]]
        ops.append(C.Op("ctrl", tuple(q[:k]), tuple(q[k:]), C._random_unitary(rng, 1 << k)))
    _check(gpu, n, dtype, ops, C.random_state(n, 561 + n), 1e-14 if dtype == "c128" else 1e-6)


@pytest.mark.parametrize("n,dtype", SIZES)
def test_moves(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(570 + n))
    ops = []
    for k in (1, 2, 3, 4, 5, 6, 3, 5):
        q = [int(v) for v in rng.permutation(n)]
        m = np.eye(1 << k, dtype=np.complex128)[rng.permutation(1 << k)]
        ops.append(C.Op("dense", tuple(q[:k]), mat=m * rng.choice([1, -1, 1j, -1j], size=1 << k)))
        ops.append(C.Op("ctrl", tuple(q[:k]), tuple(q[k:k + 3]), m))
        s = 1 + k % 4
        ops.append(C.Op("fswap", p=k % 2, q=n - s, s=s))
    psi = C.random_state(n, 571 + n)
    psi[::3] = 0.0
    psi[1::5] = complex(-0.0, 0.0)
    _check(gpu, n, dtype, ops, psi, 0.0)
