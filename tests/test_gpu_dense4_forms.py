"""Complex128 4-qubit gates on states that stream from HBM: groups in registers where no target lies inside a 128-byte
line, matrix-core tiles otherwise, with and without controls, on both sides of the line between the two and of the cache."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [24, 25])
def test_against_the_oracle(gpu, n):
    rng = np.random.Generator(np.random.PCG64(1300))
    psi = C.random_state(n, 1301)
    U = C._random_unitary(rng, 16)
    st = gpu.State(n, "c128")
    for t in ((3, 4, 5, 6), (2, 9, 13, 20), (23, 5, 14, 9), (20, 21, 22, 23), (0, 1, 2, 3)):
        for controls in ((), (11,), (1, 17)):
            if set(t) & set(controls):
                continue
            st.set(psi)
            ref = psi.copy()
            if controls:
                st.apply_controlled(controls, t, U)
                oracle.apply_controlled(ref, controls, t, U)
            else:
                st.apply_gate(t, U)
                oracle.apply_dense(ref, t, U)
            # 16 terms on amplitudes below 0.01
            assert np.max(np.abs(st.get() - ref)) <= 1e-15, (t, controls)
    st.close()
