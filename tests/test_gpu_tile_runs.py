"""Plain runs of circuits beyond one workgroup's LDS (consecutive operations in one pass over tiles of the state) against
the same operations one call at a time, bit for bit, and against the oracle: targets within, across and above a tile's
lowest qubits, controls and diagonals inside and outside the tile, every matrix form, and programs of many passes with
calls between them."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd.plan import Circuit

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 2e-5}
PHASES = [1, -1, 1j, -1j]


def _run(gpu, n, dtype, ops, psi):
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


def _narrow_op(rng, n, kinds):
    """An operation with at most two targets to mix (diagonals: up to 7), on qubits drawn anywhere."""
    kind = kinds[int(rng.integers(len(kinds)))]
    q = [int(v) for v in rng.permutation(n)]
    k = int(rng.integers(1, 3))
    if kind == "diag":
        k = int(rng.integers(1, 8))
        form = int(rng.integers(4))
        d = np.exp(1j * rng.uniform(0, 2 * np.pi, size=1 << k))
        if form:
            d = rng.choice(PHASES[:2] if form == 1 else PHASES if form == 2 else [1, -1, 1j, 0.6 + 0.8j], size=1 << k)
        return C.Op("diag", tuple(q[:k]), mat=d.astype(np.complex128))
    if kind.endswith("move"):
        m = np.eye(1 << k, dtype=np.complex128)[rng.permutation(1 << k)]
        if rng.random() < 0.5:
            m = m * rng.choice(PHASES, size=1 << k)
    else:
        m = C._random_unitary(rng, 1 << k)
    if kind.startswith("c"):
        return C.Op("ctrl", tuple(q[:k]), tuple(q[k:k + int(rng.integers(1, 5))]), m)
    return C.Op("dense", tuple(q[:k]), mat=m)


# tiles are 2^12 complex128 and 2^13 complex64 amplitudes; 13 and 14 qubits still fit LDS from 6 operations on
@pytest.mark.parametrize("n,dtype", [(12, "c128"), (13, "c128"), (14, "c128"), (15, "c128"), (18, "c128"),
                                     (13, "c64"), (14, "c64"), (15, "c64"), (16, "c64"), (19, "c64")])
@pytest.mark.parametrize("kinds", [("dense", "dense", "diag", "cdense"), ("move", "cmove", "diag"),
                                   ("dense", "move", "diag", "cdense", "cmove")])
def test_matches_single_calls(gpu, n, dtype, kinds):
    rng = np.random.Generator(np.random.PCG64(900 + n))
    psi = C.random_state(n, 901 + n)
    psi[::7] = 0.0
    psi[1::11] = complex(-0.0, 0.0)
    for nops in (2, 5, 60):
        ops = [_narrow_op(rng, n, kinds) for _ in range(nops)]
        got, calls = _run(gpu, n, dtype, ops, psi)
        assert got.tobytes() == calls.tobytes(), (n, dtype, kinds, nops)
        ref = psi.astype(got.dtype).astype(np.complex128)
        for op in ops:
            oracle.apply_op(ref, op)
        assert np.max(np.abs(got - ref)) <= TOL[dtype]


@pytest.mark.parametrize("n,dtype", [(16, "c128"), (17, "c64")])
def test_one_target_at_a_time(gpu, n, dtype):
    """Every qubit as the target, alone in its stage and beside three others, gates and moves."""
    rng = np.random.Generator(np.random.PCG64(910))
    psi = C.random_state(n, 911)
    ops = []
    for q in range(n):
        others = [int(v) for v in rng.permutation(n) if v != q]
        ops += [C.Op("dense", (q,), mat=C._random_unitary(rng, 2)),
                C.Op("ctrl", (q,), (others[0],), np.array([[0, 1], [1, 0]], dtype=np.complex128)),
                C.Op("ctrl", (q,), tuple(others[:2]), C._random_unitary(rng, 2)),
                C.Op("diag", (q, others[1]), mat=np.array([1, 1, 1, -1], dtype=np.complex128)),
                C.Op("diag", (others[2], q), mat=np.exp(1j * rng.uniform(0, 6, size=4)))]
    for seq in (ops, ops[::-1], [ops[i] for i in rng.permutation(len(ops))]):
        got, calls = _run(gpu, n, dtype, seq, psi)
        assert got.tobytes() == calls.tobytes()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_wide_operations_between_passes(gpu, dtype):
    """Gates on 3 to 6 targets, wide diagonals and fused-swaps are calls of their own among the passes."""
    n = 16
    circ = C.random_circuit(n, 920, num_ops=120, kmax=6)
    psi = C.random_state(n, 921)
    got, calls = _run(gpu, n, dtype, circ.ops, psi)
    assert got.tobytes() == calls.tobytes()


def test_long_programs_share_the_staging_ring(gpu):
    """Records and the matrices of wide gates, together several times the ring, in the order they are needed."""
    n = 14
    rng = np.random.Generator(np.random.PCG64(930))
    wide = [C.Op("dense", tuple(int(v) for v in rng.permutation(n)[:6]), mat=C._random_unitary(rng, 64))
            for _ in range(4)]
    narrow = [_narrow_op(rng, n, ("dense", "diag", "cdense", "cmove")) for _ in range(40)]
    ops = []
    for r in range(240):
        ops += narrow + [wide[r % 4]] * (1 + r % 2)
    psi = C.random_state(n, 931)
    got, calls = _run(gpu, n, "c128", ops, psi)
    assert got.tobytes() == calls.tobytes()


def test_special_values_stay_where_calls_leave_them(gpu):
    """Infinities and NaN pass through moves, sign flips and unit entries untouched, and spread as the calls spread them."""
    n = 15
    rng = np.random.Generator(np.random.PCG64(940))
    psi = C.random_state(n, 941)
    psi[5], psi[4097], psi[77] = complex(np.inf, 0.0), complex(np.nan, 1.0), complex(0.0, -np.inf)
    ops = [_narrow_op(rng, n, ("move", "cmove", "diag", "cdense")) for _ in range(12)]
    for dtype in ("c128", "c64"):
        got, calls = _run(gpu, n, dtype, ops, psi)
        a, b = got.view(got.real.dtype), calls.view(got.real.dtype)
        assert np.array_equal(a, b, equal_nan=True)


def test_growing_and_capture(gpu):
    """A circuit that grows after a run; under stream capture each operation is a launch that reads nothing of the
    host's."""
    import torch
    n = 15
    ops = C.u3_cnot_layers(n, seed=950, layers=2).ops
    psi = C.random_state(n, 951)
    s = torch.cuda.Stream()
    st = gpu.State(n, "c128", stream=s)
    c = Circuit.from_ops(n, ops[:20])
    st.set(psi)
    c.run_plain(st)
    for op in ops[20:]:
        c.add(op)
    st.set(psi)
    c.run_plain(st)
    want = st.get()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run_plain(st)
    for _ in range(3):
        Circuit.from_ops(n, C.random_circuit(n, 952, num_ops=20).ops).run_plain(st)
        st.set(psi)
        with torch.cuda.stream(s):
            g.replay()
        assert st.get().tobytes() == want.tobytes()
    st.close()
