"""Probabilities, norm and reset at the sizes where their kernels change form: fewer vectors than lanes, one and several
partial sums, the remainder of the four-load loop, both sides of the 256 MiB line between cached and non-temporal
accesses."""
import math

import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


# complex128: 256 MiB is 24 qubits; complex64: 25
@pytest.mark.parametrize("n,dtype", [(n, d) for d in ("c128", "c64") for n in (1, 2, 5, 9, 10, 12, 13, 22)] +
                         [(23, "c128"), (24, "c128"), (24, "c64"), (25, "c64")])
def test_probs_norm_and_reset(gpu, n, dtype):
    import torch
    psi = C.random_state(n, 600 + n)
    if dtype == "c64":
        psi = psi.astype(np.complex64)
    st = gpu.State(n, dtype)
    st.set(psi)
    P, norm = st.probs()
    re, im = psi.real.astype(np.float64), psi.imag.astype(np.float64)
    want = re * re + im * im
    # one multiply, one fused multiply-add against two multiplies and an add: at most two roundings of the result
    assert np.max(np.abs(P.cpu().numpy() - want) / np.where(want > 0, want, 1.0)) <= 2.0 ** -51
    # compensated sums per thread, then a tree over at most 256 threads and 1024 blocks: 18 roundings and the terms' own
    exact = math.fsum(want.tolist()) if n < 20 else float(torch.from_numpy(want).sum())
    assert abs(norm - exact) <= 2.0 ** -46 * exact
    assert st.norm() == norm and st.probs(want_norm=False)[1] is None
    assert abs(st.renormalize() - norm) == 0.0
    st.init_zero()
    got = st.get()
    assert got[0] == 1.0 and not np.any(got[1:])
    st.close()
