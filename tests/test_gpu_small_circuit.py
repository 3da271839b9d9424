"""Plain runs of circuits on states that fit one workgroup's LDS (one launch for the whole circuit) against the same
operations one call at a time and against the oracle, for every operation kind and state size, and up to and past the
sizes where the program needs several chunks or the state no longer fits."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd.plan import Circuit

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 2e-5}


def _run(gpu, n, dtype, ops, psi):
    assert len(ops) >= 6  # fewer run as single calls
    st = gpu.State(n, dtype)
    st.set(psi)
    c = Circuit.from_ops(n, ops)
    c.run_plain(st)
    got = st.get()
    st.set(psi)
    st.run(ops)
    calls = st.get()
    c.close()
    st.close()
    return got, calls


# c128: 12 and 13 qubits are 4 and 8 amplitudes per thread, 14 does not fit; c64: 14 is 16 per thread, 15 does not fit
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [2, 3, 5, 6, 7, 8, 10, 11, 12, 13, 14, 15])
def test_every_kind_matches_single_calls(gpu, n, dtype):
    circ = C.random_circuit(n, 500 + n, num_ops=60, kmax=6)
    psi = C.random_state(n, 510 + n)
    got, calls = _run(gpu, n, dtype, circ.ops, psi)
    # both sides round each amplitude once or twice per term of at most 64, over 60 operations, amplitudes below 1
    assert np.max(np.abs(got - calls)) <= TOL[dtype]
    if dtype == "c64":  # the same roundings in the same order
        assert got.tobytes() == calls.tobytes()
    ref = psi.astype(got.dtype).astype(np.complex128)
    for op in circ.ops:
        oracle.apply_op(ref, op)
    assert np.max(np.abs(got - ref)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 4, 9, 13])
def test_moves_are_exact(gpu, n, dtype):
    """Permutations with phases, phase diagonals, controlled moves and fused-swaps: the same bits as single calls,
    signed zeros and unchanged amplitudes included."""
    rng = np.random.Generator(np.random.PCG64(520 + n))
    ops = []
    for _ in range(40):
        k = int(rng.integers(1, min(6, n) + 1))
        t = tuple(int(v) for v in rng.choice(n, size=k, replace=False))
        phase = rng.choice([1, -1, 1j, -1j], size=1 << k)
        kind = int(rng.integers(0, 4))
        if kind == 0:
            ops.append(C.Op("dense", t, mat=np.eye(1 << k, dtype=np.complex128)[rng.permutation(1 << k)] * phase))
        elif kind == 1:
            phase[0] = 1
            ops.append(C.Op("diag", t, mat=phase.astype(np.complex128)))
        elif kind == 2 and k > 1:
            m = np.eye(1 << (k - 1), dtype=np.complex128)[rng.permutation(1 << (k - 1))]
            ops.append(C.Op("ctrl", t[1:], t[:1], m))
        elif n > 1:
            s = int(rng.integers(1, n // 2 + 1))
            p = int(rng.integers(0, n - 2 * s + 1))
            ops.append(C.Op("fswap", p=p, q=int(rng.integers(p + s, n - s + 1)), s=s))
    psi = C.random_state(n, 530 + n)
    psi[::3] = 0.0
    psi[1::5] = complex(-0.0, 0.0)
    got, calls = _run(gpu, n, dtype, ops, psi)
    assert got.tobytes() == calls.tobytes()


def test_large_diagonals_and_many_controls(gpu):
    n = 13
    rng = np.random.Generator(np.random.PCG64(540))
    ops = []
    for k in (3, 7, 12):
        t = tuple(int(v) for v in rng.choice(n, size=k, replace=False))
        d = np.exp(1j * rng.uniform(0, 2 * np.pi, size=1 << k))
        d[::4], d[1::4] = 1.0, -1.0
        ops.append(C.Op("diag", t, mat=d))
    for k, nc in ((1, 12), (2, 5), (3, 9)):
        q = [int(v) for v in rng.choice(n, size=k + nc, replace=False)]
        ops.append(C.Op("ctrl", tuple(q[:k]), tuple(q[k:]), C._random_unitary(rng, 1 << k)))
    psi = C.random_state(n, 541)
    got, calls = _run(gpu, n, "c128", ops, psi)
    assert np.max(np.abs(got - calls)) <= 1e-14  # at most 8 terms per amplitude, 6 operations, amplitudes below 0.1


def test_long_circuits_and_additions(gpu):
    """Programs of one chunk, of many, and past the staging limit (which run one call at a time); a circuit that grows
    after it has run."""
    n = 8
    psi = C.random_state(n, 550)
    for reps in (1, 5, 200, 3000):
        ops = C.u3_cnot_layers(n, seed=551, layers=5).ops * reps
        got, calls = _run(gpu, n, "c128", ops, psi)
        assert np.max(np.abs(got - calls)) <= 1e-15 * len(ops) + 1e-14
    base = C.u3_cnot_layers(n, seed=552, layers=2).ops
    st = gpu.State(n, "c128")
    c = Circuit.from_ops(n, base)
    for extra in C.random_circuit(n, 553, num_ops=8).ops:
        c.add(extra)
        base = base + [extra]
        st.set(psi)
        c.run_plain(st)
        got = st.get()
        st.set(psi)
        st.run(base)
        assert np.max(np.abs(got - st.get())) <= 1e-13
    st.close()


def test_capture_takes_the_launches_themselves(gpu):
    """Under stream capture a plain run records kernels that read nothing from the host: replays after other work on
    the state repeat the circuit."""
    import torch
    n = 9
    ops = C.u3_cnot_layers(n, seed=560, layers=3).ops
    psi = C.random_state(n, 561)
    s = torch.cuda.Stream()
    st = gpu.State(n, "c128", stream=s)
    c = Circuit.from_ops(n, ops)
    st.set(psi)
    c.run_plain(st)
    want = st.get()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run_plain(st)
    for _ in range(3):
        st.set(psi)
        other = C.random_circuit(n, 562, num_ops=20).ops
        Circuit.from_ops(n, other).run_plain(st)
        st.set(psi)
        with torch.cuda.stream(s):
            g.replay()
        st.sync()
        assert np.max(np.abs(st.get() - want)) <= 1e-13
    st.close()
