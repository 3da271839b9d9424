"""Complex128 batch levels on both sides of the line between the two block kernels (one 12-qubit block's worth per compute
unit, 2^20 amplitudes on 256): levels of one side each and a batch whose levels cross it, every block size, few and many
blocks per workgroup, small circuits beside them."""
import numpy as np
import pytest

import oracle
from paper_2203_16044_amd.batch import Batch

from test_gpu_batch_shares import _circ

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [10, 11, 12])
@pytest.mark.parametrize("sizes", [(13, 15), (19, 18, 9), (20, 9), (19, 19, 12), (20, 13, 8)])
def test_levels_on_both_sides(gpu, bits, sizes):
    # the second circuit of a pair is shorter: later levels hold the first alone
    circs = [_circ(n, 40 * n + i, 60 >> (2 * i)) for i, n in enumerate(sizes)]
    want = []
    for c in circs:
        psi = np.zeros(1 << c.n, dtype=np.complex128)
        psi[0] = 1.0
        for op in c.ops:
            oracle.apply_op(psi, op)
        want.append(np.abs(psi) ** 2)
    for wg in (1, 32):
        b = Batch(circs, "c128", bits, 3, wg)
        for graph in (False, True, True):
            b.run(graph)
            for i, w in enumerate(want):
                # at most 60 gates of 4 products and sums each, on probabilities that sum to 1: 60 * 8 half units
                assert np.max(np.abs(b.probs(i) - w)) <= 1e-12, (sizes[i], wg, graph)
        b.close()


@pytest.mark.parametrize("bits", [10, 12])
def test_levels_that_stream(gpu, bits):
    """25 qubits, 512 MiB: non-temporal accesses; a small circuit beside it."""
    circs = [_circ(25, 1025, 12), _circ(9, 1026, 30)]
    b = Batch(circs, "c128", bits, 3, 32)
    for graph in (False, True, True):
        b.run(graph)
    for i, c in enumerate(circs):
        psi = np.zeros(1 << c.n, dtype=np.complex128)
        psi[0] = 1.0
        for op in c.ops:
            oracle.apply_op(psi, op)
        assert np.max(np.abs(b.probs(i) - np.abs(psi) ** 2)) <= 1e-12
    b.close()
