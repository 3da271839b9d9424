"""Complex128 block passes in both forms (few blocks: one at a time through LDS whole; four blocks per compute unit and
more: four side by side, one component through LDS at a time) against the oracle, for every block size, ops on one to
three of a block's qubits, and on both sides of the size from which the state streams."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd.plan import Circuit, Plan

pytestmark = pytest.mark.gpu


def _ops(n, seed, count):
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(count):
        k = int(rng.integers(1, 4))
        t = tuple(int(v) for v in rng.permutation(n)[:k])
        out.append(C.Op("dense", t, mat=C._random_unitary(rng, 1 << k)))
    return out


# 256 compute units: 1,024 blocks are 20 qubits in blocks of 10, 21 in 11, 22 in 12, 23 in 13
@pytest.mark.parametrize("b,n", [(10, 19), (10, 20), (11, 20), (11, 21), (12, 21), (12, 22), (13, 22), (13, 23)])
@pytest.mark.parametrize("low", [3, 4])
def test_against_the_oracle(gpu, b, n, low):
    ops = _ops(n, 1000 + b, 24)
    psi = C.random_state(n, 1010 + b)
    st = gpu.State(n, "c128")
    st.set(psi)
    p = Plan(Circuit.from_ops(n, ops), "block", b, low, "c128")
    p.run(st)
    got = st.get()
    p.close()
    st.close()
    for op in ops:
        oracle.apply_op(psi, op)
    # 24 ops of at most 8 terms on amplitudes below 0.02
    assert np.max(np.abs(got - psi)) <= 1e-14


def test_streaming_states_take_every_block_once(gpu):
    """25 qubits (512 MiB): blocks are handed out in runs per XCD."""
    n = 25
    ops = _ops(n, 1020, 10)
    psi = C.random_state(n, 1021)
    st = gpu.State(n, "c128")
    st.set(psi)
    c = Circuit.from_ops(n, ops)
    p = Plan(c, "block", 12, 3, "c128")
    p.run(st)
    got = st.get()
    st.set(psi)
    c.run_plain(st)
    plain = st.get()
    for op in ops:
        oracle.apply_op(psi, op)
    assert np.max(np.abs(got - psi)) <= 1e-14
    assert np.max(np.abs(plain - psi)) <= 1e-14
    p.close()
    st.close()
