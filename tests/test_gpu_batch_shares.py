"""Batches whose small circuits are dealt out over the levels of the large ones, at the edges of that rule: shares of
one stage and of many, circuits without gates, more small circuits than compute units, no large circuit at all; every
block size, both precisions, replayed from the graph and launched directly."""
import numpy as np
import pytest

import circuits as C
import oracle
from paper_2203_16044_amd.batch import Batch

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 1e-5}  # probabilities below 1 after at most 300 gates


class _Circ:
    def __init__(self, n, ops):
        self.n, self.ops = n, ops


def _circ(n, seed, gates):
    rng = np.random.Generator(np.random.PCG64(seed))
    ops = []
    for _ in range(gates):
        k = int(rng.integers(1, 3))
        t = tuple(int(v) for v in rng.permutation(n)[:k])
        ops.append(C.Op("dense", t, mat=C._random_unitary(rng, 1 << k)))
    return _Circ(n, ops)


def _check(circs, dtype, **params):
    want = []
    for c in circs:
        psi = np.zeros(1 << c.n, dtype=np.complex128)
        psi[0] = 1.0
        for op in c.ops:
            oracle.apply_op(psi, op)
        want.append(np.abs(psi) ** 2)
    b = Batch(circs, dtype, **params)
    for graph in (False, True, True):
        b.run(graph)
        for i, w in enumerate(want):
            assert np.max(np.abs(b.probs(i) - w)) <= TOL[dtype], (i, circs[i].n, graph)
    b.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("bits", [10, 11, 12])
def test_shares(gpu, dtype, bits):
    circs = [_circ(bits + 2, 1100, 120), _circ(bits + 1, 1101, 40), _circ(8, 1102, 3), _circ(8, 1103, 300),
             _circ(9, 1104, 0), _circ(bits, 1105, 150), _circ(bits, 1106, 9), _circ(bits - 1, 1107, 60)]
    _check(circs, dtype, block_bits=bits, low_bits=3, wg_per_cu=8)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_more_small_circuits_than_compute_units(gpu, dtype):
    circs = [_circ(8, 1110 + i, 8) for i in range(300)] + [_circ(12, 1109, 60)]
    _check(circs, dtype, block_bits=10, low_bits=3, wg_per_cu=1)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_small_circuits_alone(gpu, dtype):
    _check([_circ(n, 1500 + n, 30) for n in (8, 9, 10, 11, 12)], dtype, block_bits=12, low_bits=4, wg_per_cu=2)
