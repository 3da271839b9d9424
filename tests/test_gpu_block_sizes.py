"""Complex128 block passes of every block size on states of 2^22 amplitudes and more, where each block is a workgroup of
the kernel that keeps four on a compute unit: cached, and streaming with the blocks handed out in runs per XCD."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd.plan import Circuit, Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [21, 22, 25])
@pytest.mark.parametrize("bits", [10, 11, 12, 13])
def test_every_block_size(gpu, n, bits):
    rng = np.random.Generator(np.random.PCG64(1050 + n))
    ops = []
    for i in range(18 if n < 25 else 10):  # 1, 2 and 3 qubits, anywhere
        k = 1 + i % 3
        t = tuple(int(v) for v in rng.permutation(n)[:k])
        ops.append(C.Op("dense", t, mat=C._random_unitary(rng, 1 << k)))
    psi = C.random_state(n, 1051 + n)
    c = Circuit.from_ops(n, ops)
    p = Plan(c, "block", bits, 3, "c128")
    st = gpu.State(n, "c128")
    st.set(psi)
    p.run(st)
    got = st.get()
    p.close()
    c.close()
    st.close()
    for op in ops:
        oracle.apply_op(psi, op)
    # 18 operations of at most 8 terms on amplitudes below 0.02
    assert np.max(np.abs(got - psi)) <= 1e-14


@pytest.mark.parametrize("bits", [10, 11, 12, 13])
def test_persistent_workgroups_on_request(gpu, bits):
    """With block_wg_per_cu set, 22 qubits run the kernel whose workgroups walk several blocks; at its default, the one
    with a workgroup per block. Both agree with the oracle."""
    n = 22
    rng = np.random.Generator(np.random.PCG64(1070))
    ops = [C.Op("dense", tuple(int(v) for v in rng.permutation(n)[:2]), mat=C._random_unitary(rng, 4)) for _ in range(12)]
    psi = C.random_state(n, 1071)
    ref = psi.copy()
    for op in ops:
        oracle.apply_op(ref, op)
    c = Circuit.from_ops(n, ops)
    p = Plan(c, "block", bits, 3, "c128")
    st = gpu.State(n, "c128")
    before = gpu.binding.qs_get_tunable("block_wg_per_cu")
    try:
        for wg in (1, 4, before):
            gpu.binding.qs_set_tunable("block_wg_per_cu", wg)
            st.set(psi)
            p.run(st)
            assert np.max(np.abs(st.get() - ref)) <= 1e-14, wg
    finally:
        gpu.binding.qs_set_tunable("block_wg_per_cu", before)
    p.close()
    c.close()
    st.close()
