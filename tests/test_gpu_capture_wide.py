"""Captured wide gates, whose matrices a graph reads from host memory at each replay, beside eager plain runs and
sampling, which write to host memory of their own: before the capture and between the replays, round the ring they use."""
import numpy as np
import pytest
import torch

import circuits as C
import oracle
from paper_2203_16044_amd.plan import Circuit

pytestmark = pytest.mark.gpu


def _ops(n, num, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return [C.Op("dense", (q % n,), mat=C._random_unitary(rng, 2)) for q in range(num)]


def _after(psi, ops):
    ref = psi.copy()
    for op in ops:
        oracle.apply_op(ref, op)
    return ref


def _capture(st, stream, ops):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        for op in ops:
            st.apply_op(op)
    return g


def _replayed(st, stream, g, psi):
    st.set(psi)
    with torch.cuda.stream(stream):
        g.replay()
    st.sync()
    return st.get()


def _wide(n, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    t = [int(v) for v in rng.permutation(n)]
    return [C.Op("dense", tuple(t[:5]), mat=C._random_unitary(rng, 32))]


# 11: in LDS, 14: tiles (complex128 12 qubits). Errors: 32 terms an amplitude, amplitudes below 0.2
@pytest.mark.parametrize("n", [11, 14])
def test_plain_run_before_the_capture(gpu, n):
    psi = C.random_state(n, 571)
    wide = _wide(n, 572)
    s = torch.cuda.Stream()
    st = gpu.State(n, "c128", stream=s)
    st.sample(np.linspace(0, 0.99, 100))
    Circuit.from_ops(n, _ops(n, 60, 573)).run_plain(st)
    g = _capture(st, s, wide)
    ref = _after(psi, wide)
    for _ in range(3):
        assert np.max(np.abs(_replayed(st, s, g, psi) - ref)) <= 1e-13
    st.close()


@pytest.mark.parametrize("n", [11, 14])
@pytest.mark.parametrize("what", ["runs", "shots"])
def test_eager_work_between_replays(gpu, n, what):
    psi = C.random_state(n, 574)
    wide = _wide(n, 575)
    s = torch.cuda.Stream()
    st = gpu.State(n, "c128", stream=s)
    g = _capture(st, s, wide)
    ref = _after(psi, wide)
    c = Circuit.from_ops(n, _ops(n, 2000, 576))
    u = np.random.Generator(np.random.PCG64(577)).random(30000)
    for _ in range(3):
        for _ in range(60):
            st.set(psi)
            if what == "runs":
                c.run_plain(st)
            else:
                st.sample(u)
        assert np.max(np.abs(_replayed(st, s, g, psi) - ref)) <= 1e-13
    st.close()
