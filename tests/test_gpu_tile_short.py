"""Short plain runs, on both sides of the number of operations from which passes over tiles pay for the copy of their
records: the same bits as the operations one call at a time, alone, between wide gates and after the circuit has grown
across the line."""
import numpy as np
import pytest

import circuits as C
from paper_2203_16044_amd.plan import Circuit

from test_gpu_tile_runs import _narrow_op, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [(12, "c128"), (13, "c128"), (16, "c128"), (20, "c128"), (13, "c64"), (16, "c64"),
                                     (20, "c64")])
def test_short_runs_match_single_calls(gpu, n, dtype):
    rng = np.random.Generator(np.random.PCG64(960 + n))
    psi = C.random_state(n, 961 + n)
    eye = C.Op("dense", (1,), mat=np.eye(2, dtype=np.complex128))
    wide = C.Op("dense", (0, 3, n - 1), mat=C._random_unitary(rng, 8))
    for nops in range(1, 10):
        ops = [_narrow_op(rng, n, ("dense", "diag", "cdense", "cmove")) for _ in range(nops)]
        for seq in (ops, [wide] + ops, ops + [eye, wide] + ops[::-1], [eye] * nops):
            got, calls = _run(gpu, n, dtype, seq, psi)
            if n == 12:  # the LDS form, where many operations are wide: sums in another order
                assert np.max(np.abs(got - calls)) <= 1e-14
            else:
                assert got.tobytes() == calls.tobytes(), (nops, len(seq))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_a_circuit_grows_across_the_line(gpu, dtype):
    n = 14
    rng = np.random.Generator(np.random.PCG64(970))
    psi = C.random_state(n, 971)
    st = gpu.State(n, dtype)
    c, ops = Circuit.from_ops(n, []), []
    for _ in range(12):
        op = _narrow_op(rng, n, ("dense", "cdense", "diag"))
        c.add(op)
        ops.append(op)
        st.set(psi)
        c.run_plain(st)
        got = st.get()
        st.set(psi)
        st.run(ops)
        assert got.tobytes() == st.get().tobytes()
    st.close()
