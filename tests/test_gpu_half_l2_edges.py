"""One-pass gates on states of 8, 16 and 32 MiB, of which the middle one takes non-temporal accesses: lane-exchange and
group forms, moves, controls inside and above a cache line."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [(19, "c128"), (20, "c128"), (21, "c128"), (20, "c64"), (21, "c64"), (22, "c64")])
def test_one_pass_gates(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(1200 + n))
    psi = C.random_state(n, 1201 + n)
    if dtype == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    # amplitudes below 2^-6 = 0.0156; 2^k products of 2 terms each and the entry's rounding: 2^(k+1) + 2 half units of it
    assert np.max(np.abs(psi)) < 2.0 ** -6
    unit = 2.0 ** (-6 - (53 if dtype == "c128" else 24))
    X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
    ops = [C.Op("dense", t, mat=C._random_unitary(rng, 1 << len(t)))
           for t in ((0,), (4,), (n - 1,), (0, n - 1), (5, n - 2), (6, 11, n - 1), (1, 9, n - 1))]
    ops += [C.Op("ctrl", (t,), (c,), m) for t, c in ((n - 1, 0), (0, n - 1), (9, n - 2), (5, 6))
            for m in (X, C._random_unitary(rng, 2))]
    ops += [C.Op("dense", (8,), mat=X)]
    st = gpu.State(n, dtype)
    for op in ops:
        st.set(psi)
        st.apply_op(op)
        got = st.get()
        ref = psi.copy()
        oracle.apply_op(ref, op)
        err = np.max(np.maximum(np.abs(got.real - ref.real), np.abs(got.imag - ref.imag)))
        assert err <= (2 ** (len(op.targets) + 1) + 2) * 2 * unit, (op.kind, op.targets, op.controls)
    st.close()
