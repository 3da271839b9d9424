"""Probabilities into an array of doubles that does not start on a 16-byte boundary (a slice at an odd place): the same
values as into one that does, and nothing written around it."""
import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


# one vector, remainders, many blocks; 25 qubits complex64: non-temporal stores
@pytest.mark.parametrize("n,dtype", [(n, d) for d in ("c128", "c64") for n in (1, 2, 9, 13, 20)] + [(25, "c64")])
def test_probs_at_an_odd_place(gpu, n, dtype):
    import torch
    psi = C.random_state(n, 70 + n)
    st = gpu.State(n, dtype)
    st.set(psi if dtype == "c128" else psi.astype(np.complex64))
    want, norm = st.probs()
    assert want.data_ptr() % 16 == 0
    out = torch.full(((1 << n) + 3,), -1.0, dtype=torch.float64, device="cuda")
    at = out.data_ptr() + 8
    assert at % 16 == 8
    assert gpu.binding.qs_probs(st.h, at, True) == norm
    assert torch.equal(out[1:-2], want) and (out[[0, -2, -1]] == -1.0).all()
    out.fill_(-1.0)
    norm_dev = torch.zeros(3, dtype=torch.float64, device="cuda")
    gpu.binding.qs_probs_noalloc(st.buf.data_ptr(), n, st.qs_dtype, at, norm_dev.data_ptr() + 8, st.stream.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out[1:-2], want) and (out[[0, -2, -1]] == -1.0).all()
    assert norm_dev.tolist() == [0.0, norm, 0.0]
    st.close()
