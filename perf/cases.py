"""Performance cases of the state-vector engine: what its users run, from the smallest call to the largest.

Every case starts from a seeded synthetic circuit of one of the families the repository's benchmark, batches and paper
workloads use (U3 + CNOT layers, U3 + CZ + RZ + Toffoli + fused-swap layers, QSB rotation / CNOT sets, SU(4) pairings,
quantum volume, one RX per qubit, random operations of every kind), in complex128 or complex64, and goes through the
public Python entry points: gate by gate (`Circuit.run_plain`), through a plan of block passes or fused dense blocks
(`Plan`), through a complex64 plan with periodic renormalisation (`LazyRenormPlan`), as a batch of circuits replayed
from a graph (`Batch`), by sampling (`State.sample`) or by measuring and resetting qubits in mid-circuit
(`State.measure`, `State.reset`).

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what a program holds before the call (circuit, plan, state, uniforms), from the seed
  run(state)           one pass; returns the state vector and what was computed from it
  work(case)           bytes and floating-point operations one pass cannot do without
  exact(case, seed)    the same outputs from plain torch in complex128
"""
import math
import random

import numpy as np
import torch

from paper_2203_16044_amd.batch import Batch
from paper_2203_16044_amd.binding import qs_batch_probs
from paper_2203_16044_amd.plan import Circuit, LazyRenormPlan, Plan
from paper_2203_16044_amd.state import State


def listed():
    return [
        # the smallest call: a 10-qubit circuit of 10 U3 + CNOT layers gate by gate, as an optimiser's inner loop or a
        # unit test runs it; launches and latency count
        dict(name="gates_u3cnot_n10_c128", kind="gates", family="u3_cnot", n=10, layers=10, dtype="c128"),
        # an ordinary gate-by-gate run that still fits the last-level cache, of odd width: RZ.RX.RZ + CNOT ring
        dict(name="gates_qsb_n21_c64", kind="gates", family="qsb", n=21, layers=4, dtype="c64"),
        # a large gate-by-gate run: U3, CZ, RZ on every qubit, Toffolis, a fused-swap between the ends; HBM-bound
        dict(name="gates_mixed_n28_c128", kind="gates", family="mixed", n=28, layers=3, dtype="c128"),
        # operations of every kind and width the entry points take: dense and controlled gates of 1 to 6 qubits,
        # diagonals, permutations, fused-swaps of any range
        dict(name="gates_random_n25_c64", kind="gates", family="random", n=25, layers=48, dtype="c64", form=25),
        # a planned circuit of ordinary size (quantum volume, depth 10): the state fits in cache, few blocks per pass
        dict(name="plan_qv_n19_c128", kind="plan", family="qv", n=19, layers=10, dtype="c128", bits=12, low=4),
        # the benchmark's own form near the largest that leaves room for a second state: SU(4) pairings + U3, planned
        dict(name="plan_su4_n31_c128", kind="plan", family="su4", n=31, layers=10, dtype="c128", bits=12, low=3),
        # the complex64 form of the benchmark: one plan, renormalised every 10 layers
        dict(name="lazy_su4_n27_c64", kind="lazy", family="su4", n=27, layers=20, dtype="c64", bits=12, low=4),
        # the same circuits through fused dense blocks of up to 6 qubits (the matrix-core gate kernel)
        dict(name="fuse6_su4_n27_c128", kind="fuse", family="su4", n=27, layers=6, dtype="c128", bits=6),
        # serving: a batch of independent circuits of 10 to 20 qubits, graph replay, in both precisions
        dict(name="batch_n10_20_c128", kind="batch", count=24, nmin=10, nmax=20, dtype="c128", bits=12, low=3, wg=32,
             form=512),
        dict(name="batch_n10_17_c64", kind="batch", count=40, nmin=10, nmax=17, dtype="c64", bits=12, low=4, wg=32,
             form=513),
        # reading a result out: 4,096 shots from a 27-qubit state
        dict(name="sample_n27_c128", kind="sample", n=27, shots=4096, dtype="c128"),
        # mid-circuit measurement: rotate and entangle an ancilla, measure it, reset it, 4 cycles
        dict(name="measure_n23_c64", kind="measure", n=23, layers=4, dtype="c64"),
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["gates", "gates", "plan", "plan", "lazy", "fuse", "batch", "sample", "measure"])
    dtype = rng.choice(["c128", "c64"])
    if kind == "gates":
        family = rng.choice(["u3_cnot", "qsb", "mixed", "random", "rx"])
        n = rng.randint(8, 28)
        if family == "random":
            return dict(kind=kind, family=family, n=min(n, 27), layers=rng.randint(8, 48), dtype=dtype,
                        form=rng.randrange(1 << 20))
        layers = 1 if family == "rx" else rng.randint(1, 4 if n > 24 else 10)
        return dict(kind=kind, family=family, n=n, layers=layers, dtype=dtype)
    if kind == "plan":
        n = rng.randint(8, 30)
        return dict(kind=kind, family=rng.choice(["su4", "qv", "mixed", "u3_cnot"]), n=n,
                    layers=rng.randint(2, 10 if n > 26 else 20), dtype=dtype, bits=rng.choice([10, 11, 12, 12, 13]),
                    low=rng.choice([3, 4]))
    if kind == "lazy":
        n = rng.randint(12, 30)
        return dict(kind=kind, family="su4", n=n, layers=rng.randint(11, 20 if n > 28 else 40), dtype="c64",
                    bits=rng.choice([11, 12, 12, 13]), low=rng.choice([3, 4]))
    if kind == "fuse":
        return dict(kind=kind, family=rng.choice(["su4", "qv", "u3_cnot"]), n=rng.randint(8, 28),
                    layers=rng.randint(2, 6), dtype=dtype, bits=rng.randint(3, 6))
    if kind == "batch":
        nmin = rng.randint(8, 14)
        return dict(kind=kind, count=_log_int(rng, 4, 40), nmin=nmin, nmax=rng.randint(nmin + 2, 20), dtype=dtype,
                    bits=rng.choice([10, 11, 12, 12]), low=rng.choice([3, 4]), wg=rng.choice([2, 8, 32]),
                    form=rng.randrange(1 << 20))
    if kind == "sample":
        return dict(kind=kind, n=rng.randint(6, 29), shots=_log_int(rng, 1, 200000), dtype=dtype)
    return dict(kind=kind, n=rng.randint(4, 28), layers=rng.randint(1, 6), dtype=dtype)


# ----------------------------------------------------------------------------------------------------------
# circuits
# ----------------------------------------------------------------------------------------------------------
class Op:
    """One operation, as `Circuit.add` reads it: dense / diag / ctrl matrices in FP64, or a fused-swap."""

    def __init__(self, kind, targets=(), mat=None, controls=(), p=0, q=0, s=0, layer=0):
        self.kind, self.layer = kind, layer
        self.targets = tuple(int(t) for t in targets)
        self.controls = tuple(int(c) for c in controls)
        self.mat = None if mat is None else np.ascontiguousarray(mat, dtype=np.complex128)
        self.p, self.q, self.s = int(p), int(q), int(s)


X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
CZ = np.array([1, 1, 1, -1], dtype=np.complex128)


def _u3(rng):
    t, p, m = rng.uniform(0.0, 2.0 * math.pi, size=3)
    c, s = math.cos(t / 2), math.sin(t / 2)
    return np.array([[c, -np.exp(1j * m) * s], [np.exp(1j * p) * s, np.exp(1j * (p + m)) * c]])


def _rx(rng):
    t = rng.uniform(0.0, 2.0 * math.pi)
    c, s = math.cos(t / 2), math.sin(t / 2)
    return np.array([[c, -1j * s], [-1j * s, c]])


def _rz(rng):
    t = rng.uniform(0.0, 2.0 * math.pi)
    return np.array([np.exp(-0.5j * t), np.exp(0.5j * t)])


def _unitary(rng, dim):
    z = rng.standard_normal((dim, dim)) + 1j * rng.standard_normal((dim, dim))
    q, r = np.linalg.qr(z)
    d = np.diag(r)
    return q * (d / np.abs(d))


def _random_op(shape, rng, n):
    """One operation of a kind and on qubits that `shape` picks, with values from `rng`."""
    kind = shape.choice(["dense", "dense", "diag", "ctrl", "fswap"])
    if kind == "fswap":
        s = shape.randint(1, min(8, n // 2))
        p = shape.randint(0, n - 2 * s)
        return Op("fswap", p=p, q=shape.randint(p + s, n - s), s=s)
    k = shape.randint(1, min(6 if kind == "dense" else 4, n - 2))
    qubits = shape.sample(range(n), k + shape.randint(1, 2))
    t, c = qubits[:k], qubits[k:]
    if kind == "diag":
        d = np.exp(1j * rng.uniform(0, 2 * math.pi, size=1 << k))
        if shape.random() < 0.3:  # a controlled phase: every entry 1 but the last
            d[:-1] = 1.0
        return Op("diag", t, d)
    if shape.random() < 0.25:
        m = np.eye(1 << k)[shape.sample(range(1 << k), 1 << k)]
    else:
        m = _unitary(rng, 1 << k)
    return Op(kind, t, m, c if kind == "ctrl" else ())


def _circuit(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    family, n, layers = case["family"], case["n"], case["layers"]
    ops = []
    if family == "random":
        shape = random.Random(case["form"])
        return [_random_op(shape, rng, n) for _ in range(layers)]
    for L in range(1, layers + 1):
        if family == "rx":
            ops += [Op("dense", (q,), _rx(rng), layer=L) for q in range(n)]
        elif family == "qsb":
            for q in range(n):
                ops += [Op("diag", (q,), _rz(rng), layer=L), Op("dense", (q,), _rx(rng), layer=L),
                        Op("diag", (q,), _rz(rng), layer=L)]
            ops += [Op("ctrl", (q,), X, ((q + 1) % n,), layer=L) for q in range(n)]
        elif family in ("su4", "qv"):
            perm = rng.permutation(n)
            ops += [Op("dense", (perm[2 * j], perm[2 * j + 1]), _unitary(rng, 4), layer=L) for j in range(n // 2)]
            if family == "su4":
                ops += [Op("dense", (q,), _u3(rng), layer=L) for q in range(n)]
        else:
            ops += [Op("dense", (q,), _u3(rng), layer=L) for q in range(n)]
            pairs = [(a, a + 1) for a in range((L - 1) % 2, n - 1, 2)]
            if family == "u3_cnot":
                ops += [Op("ctrl", (b,), X, (a,), layer=L) for a, b in pairs]
            else:
                ops += [Op("diag", ab, CZ, layer=L) for ab in pairs]
                ops += [Op("diag", (q,), _rz(rng), layer=L) for q in range(n)]
                for _ in range(2):
                    a, b, c = rng.choice(n, size=3, replace=False)
                    ops.append(Op("ctrl", (c,), X, (a, b), layer=L))
    if family == "mixed":
        s = min(6, n // 2)
        ops.append(Op("fswap", p=0, q=n - s, s=s, layer=layers))
    elif family == "u3_cnot":
        ops.append(Op("fswap", p=0, q=n - 4, s=4, layer=layers))
    return ops


def _batch_sizes(case):
    shape = random.Random(case["form"])
    return [(shape.randint(case["nmin"], case["nmax"]), shape.randint(10, 40)) for _ in range(case["count"])]


def _batch_circuits(case, seed):
    """(n, operations) of each circuit: U3 on all, CNOT or CZ on alternating pairs, RZ on all, per layer."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for j, (n, depth) in enumerate(_batch_sizes(case)):
        ops = []
        for L in range(1, depth + 1):
            ops += [Op("dense", (q,), _u3(rng), layer=L) for q in range(n)]
            for a in range((L - 1) % 2, n - 1, 2):
                ops.append(Op("ctrl", (a + 1,), X, (a,), layer=L) if (j + L) % 2 else Op("diag", (a, a + 1), CZ, layer=L))
            ops += [Op("diag", (q,), _rz(rng), layer=L) for q in range(n)]
        out.append((n, ops))
    return out


def _ancilla(case, seed):
    """Measurement cycles: (ancilla, its U3, the qubit it controls, that qubit's U3, two uniforms)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(case["layers"]):
        a, t = (int(v) for v in rng.choice(case["n"], size=2, replace=False))
        out.append((a, _u3(rng), t, _u3(rng), rng.uniform(0.02, 0.98, size=2)))
    return out


# ----------------------------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------------------------
def _torch_dtype(case):
    return torch.complex128 if case["dtype"] == "c128" else torch.complex64


def _random_vector(n, seed):
    """A normalised complex128 state with Gaussian components, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = torch.randn(2 << n, dtype=torch.float64, device="cuda", generator=g)
    v /= torch.linalg.vector_norm(v)
    return torch.view_as_complex(v.view(-1, 2))


class _DeviceArray:
    """A float64 device buffer of `owner` (kept alive with the tensor) as the array interface torch reads."""

    def __init__(self, owner, ptr, count):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<f8", "data": (ptr, False), "version": 3}


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "batch":
        circuits = [Circuit.from_ops(n, ops) for n, ops in _batch_circuits(case, seed)]
        s["batch"] = Batch(circuits, case["dtype"], case["bits"], case["low"], case["wg"])
        s["probs"] = [torch.as_tensor(_DeviceArray(s["batch"], qs_batch_probs(s["batch"].h, i)[0], 1 << c.n),
                                      device="cuda") for i, c in enumerate(circuits)]
        return s
    n = case["n"]
    s["state"] = State(n, case["dtype"])
    if kind in ("sample", "measure"):
        s["state"].buf.copy_(_random_vector(n, seed))
        if kind == "sample":
            s["u"] = np.random.Generator(np.random.PCG64(seed)).random(case["shots"])
        else:
            s["cycles"] = _ancilla(case, seed)
        return s
    ops = _circuit(case, seed)
    if kind == "lazy":
        marks = range(10, case["layers"] + 1, 10)
        s["plan"] = LazyRenormPlan(n, ops, marks, "block", case["bits"], case["low"], case["dtype"])
        return s
    s["circuit"] = Circuit.from_ops(n, ops)
    if kind == "plan":
        s["plan"] = Plan(s["circuit"], "block", case["bits"], case["low"], case["dtype"])
    elif kind == "fuse":
        s["plan"] = Plan(s["circuit"], "fuse", case["bits"], 0, case["dtype"])
    return s


def run(state):
    kind = state["kind"]
    if kind == "batch":
        state["batch"].run(graph=True)
        return state["probs"]
    st = state["state"]
    if kind == "sample":
        return st.sample(state["u"])
    if kind == "measure":
        seen = []
        for a, ua, t, ut, (u, v) in state["cycles"]:
            st.apply_gate((a,), ua)
            st.apply_controlled((a,), (t,), ut)
            seen.append(st.measure(a, u))
            st.apply_gate((t,), ut)
            seen.append(st.reset(t, v))
        return {"outcomes": seen, "state": st.buf}
    st.init_zero()
    if kind == "gates":
        state["circuit"].run_plain(st)
    else:
        state["plan"].run(st)
    probs, norm = st.probs()
    return {"state": st.buf, "probs": probs, "norm": norm}


# ----------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------------------
def _op_work(op, n, amp):
    """(bytes, flops) of one operation on a state of 2^n amplitudes of `amp` bytes: amplitudes it changes, read and
    written once; 8 flops per complex multiply-add."""
    full = float(2 * amp << n)
    if op.kind == "fswap":
        return full * (1 - 2.0 ** -op.s), 0.0
    if op.kind == "diag":
        share = float(np.mean(op.mat.reshape(-1) != 1.0))
        return full * share, 6.0 * (1 << n) * share
    share = 2.0 ** -len(op.controls)
    moves = np.count_nonzero(op.mat) == len(op.mat)
    return full * share, 0.0 if moves else 8.0 * len(op.mat) * (1 << n) * share


def _planned_flops(ops, n):
    """Flops of a circuit whose 1-qubit gates are all multiplied into wider ones (or, alone, into one another)."""
    two = sum(1 for o in ops if o.kind != "fswap" and len(o.targets) + len(o.controls) > 1)
    return 32.0 * (1 << n) * max(two, n / 2)


def work(case):
    kind, amp = case["kind"], 16 if case["dtype"] == "c128" else 8
    if kind == "batch":
        # states that fit a compute unit's memory never leave it; the others are kept in HBM by any form that runs
        # them, but each circuit's probabilities are all that has to be written
        sizes = _batch_sizes(case)
        return {"bytes": float(sum(8 << n for n, _ in sizes)),
                "flops": float(sum(32.0 * (1 << n) * ((n - 1) // 2) * depth for n, depth in sizes))}
    n = case["n"]
    size = float(amp << n)
    if kind == "sample":
        return {"bytes": size + 16.0 * case["shots"], "flops": 4.0 * (1 << n)}
    if kind == "measure":
        # per cycle: a dense gate, a controlled one, a dense gate; two measurements that read the state, then read the
        # half they keep and write the whole
        per = 2 * (2 * size) + size + 2 * (size + size / 2 + size)
        return {"bytes": per * case["layers"], "flops": case["layers"] * (1 << n) * (16.0 * 2 + 8.0 + 2 * 5.0)}
    ops = _circuit(case, 0)
    out = size + float(8 << n)  # the state and its probabilities, written
    if kind == "gates":
        w = [_op_work(o, n, amp) for o in ops]
        return {"bytes": out + size + sum(b for b, _ in w), "flops": sum(f for _, f in w) + 3.0 * (1 << n)}
    # planned: the state has to be written and read back at least once per pass, and a pass takes gates on at most
    # 13 qubits (6 as fused dense blocks): a lower bound of one pass per (qubits / width) of the layers
    width = 6 if kind == "fuse" else 13
    passes = max(1, math.ceil(n / width))
    return {"bytes": out + 2 * size * passes, "flops": _planned_flops(ops, n) + 3.0 * (1 << n)}


# ----------------------------------------------------------------------------------------------------------
# the same outputs from plain torch in complex128
# ----------------------------------------------------------------------------------------------------------
def _members(x, n, targets, controls):
    """The 2^k slices of x (a vector of 2^n) with the controls at 1 and targets[j] at bit j of the slice's number."""
    qs = sorted(targets + controls, reverse=True)
    shape, where, above = [], {}, n
    for q in qs:
        shape += [1 << (above - 1 - q), 2]
        where[q] = len(shape) - 1
        above = q
    v = x.view(shape + [1 << above])
    out = []
    for a in range(1 << len(targets)):
        at = [slice(None)] * v.dim()
        for c in controls:
            at[where[c]] = 1
        for j, t in enumerate(targets):
            at[where[t]] = (a >> j) & 1
        out.append(v[tuple(at)])
    return out


def _apply(x, n, op):
    if op.kind == "fswap":
        lo, hi, s = min(op.p, op.q), max(op.p, op.q), op.s
        v = x.view(1 << (n - hi - s), 1 << s, 1 << (hi - lo - s), 1 << s, 1 << lo)
        return v.transpose(1, 3).contiguous().view(-1)
    part = _members(x, n, op.targets, op.controls)
    if op.kind == "diag":
        for p, d in zip(part, op.mat.reshape(-1)):
            if d != 1:
                p *= complex(d)
        return x
    old = [p.clone() for p in part]
    for p, row in zip(part, op.mat):
        acc = None
        for u, o in zip(row, old):
            if u != 0:
                acc = o * complex(u) if acc is None else acc.add_(o, alpha=complex(u))
        p.copy_(acc)
    return x


def _seconds(ops, n):
    """About what _apply takes over `ops`."""
    t = 0.0
    for o in ops:
        m = 1 if o.kind in ("fswap", "diag") else 1 << len(o.targets)
        t += m * (80.0 * (1 << n) / 2.5e12) + m * m * 15e-6
    return t


def _zero_state(n):
    x = torch.zeros(1 << n, dtype=torch.complex128, device="cuda" if torch.cuda.is_available() else "cpu")
    x[0] = 1.0
    return x


def _square(x):
    return x.real.square() + x.imag.square()


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None  # whole numbers
    if kind == "batch":
        circuits = _batch_circuits(case, seed)
        if sum(_seconds(ops, n) for n, ops in circuits) > 12:
            return None
        out = []
        for n, ops in circuits:
            x = _zero_state(n)
            for op in ops:
                x = _apply(x, n, op)
            out.append(_square(x))
        return out
    n = case["n"]
    if kind == "measure":
        x = _random_vector(n, seed).to(_torch_dtype(case)).to(torch.complex128)
        seen = []

        def outcome(x, q, u):
            zero, one = _members(x, n, (q,), ())
            p0, p1 = float(_square(zero).sum()), float(_square(one).sum())
            bit = 1 if u * (p0 + p1) < p1 else 0
            keep, drop, p = (one, zero, p1) if bit else (zero, one, p0)
            keep /= math.sqrt(p)
            drop.zero_()
            return bit, p1 / (p0 + p1)

        for a, ua, t, ut, (u, v) in _ancilla(case, seed):
            x = _apply(x, n, Op("dense", (a,), ua))
            x = _apply(x, n, Op("ctrl", (t,), ut, (a,)))
            seen.append(outcome(x, a, u))
            x = _apply(x, n, Op("dense", (t,), ut))
            bit, _ = outcome(x, t, v)
            if bit:
                x = _apply(x, n, Op("dense", (t,), X))
            seen.append(bit)
        return {"outcomes": seen, "state": x}
    ops = _circuit(case, seed)
    if n > 28 or _seconds(ops, n) > 12:
        return None
    x = _zero_state(n)
    for op in ops:
        x = _apply(x, n, op)
    probs = _square(x)
    return {"state": x, "probs": probs, "norm": float(probs.sum())}
