"""A gate list's rounding (``sv.run``) beside that of the one-gate kernels
(``sv.apply``): how far each ends from the same matrices applied in 80 bits.

The list may be no further off.  Lists of 200 to 400 gates end 0.6e-15
(complex128) to 0.7e-6 (complex64) of the state's norm away, list by list with
a scatter of 5 to 10%; the root mean square over six lists scatters by 2 to 3%
(a model of both paths' roundings, 8 times 6 lists a family).  Hence 1.1."""
import math

import numpy as np
import pytest

from workloads import Gate, layered_u3_cz, random_mixed_circuit

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")

N, LISTS = 10, 6


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


def unitary(rng):
    return np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]


def matrices(seed):
    """Explicit one-target matrices on every qubit and a CZ brick."""
    rng = np.random.default_rng(seed)
    g = []
    for layer in range(20):
        g += [Gate("unitary", (q,), (), (), -1, unitary(rng)) for q in range(N)]
        g += [Gate("z", (q + 1,), (q,)) for q in range(layer % 2, N - 1, 2)]
    return g


def rotations(seed):
    """Runs of RX, RY, RZ on every qubit and a cyclic row of CNOTs."""
    rng = np.random.default_rng(seed)
    g = []
    for _ in range(10):
        g += [Gate(r, (q,), (), (float(rng.uniform(0, 2 * math.pi)),)) for q in range(N) for r in ("rx", "ry", "rz")]
        g += [Gate("x", (q,), ((q + 1) % N,)) for q in range(N)]
    return g


def phases(seed):
    """Phases that wait through X and Y gates and controlled ones."""
    rng = np.random.default_rng(seed)
    g = [Gate("h", (q,)) for q in range(N)]
    while len(g) < 300:
        a, b = (int(v) for v in rng.choice(N, 2, replace=False))
        th = (float(rng.uniform(0, 2 * math.pi)),)
        g += [[Gate("rz", (a,), (), th)], [Gate("p", (a,), (), th), Gate("x", (a,))], [Gate("t", (a,)), Gate("y", (a,))],
              [Gate("x", (a,), (b,))], [Gate("p", (a,), (b,), th)], [Gate("rzz", (a, b), (), th)],
              [Gate("h", (a,))]][int(rng.integers(7))]
    return g


FAMILIES = {"layered": lambda s: layered_u3_cz(N, 20, s), "matrices": matrices, "rotations": rotations, "phases": phases,
            "mixed": lambda s: random_mixed_circuit(N, 200, s, kmax=3, max_ctrl=2)}


def in_80_bits(gates):
    """The state after the gates' own matrices (as the library lowers them)."""
    ix = np.arange(1 << N)
    psi = np.zeros(1 << N, np.clongdouble)
    psi[0] = 1
    for g in gates:
        m = qvm.gate_matrix(g)
        base = ix[[all((i >> c) & 1 for c in g.controls) and not any((i >> t) & 1 for t in g.targets) for i in ix]]
        rows = [base | sum(((j >> r) & 1) << t for r, t in enumerate(g.targets)) for j in range(m.shape[0])]
        v = [psi[r] for r in rows]
        for i, r in enumerate(rows):
            psi[r] = sum(np.clongdouble(m[i, j]) * v[j] for j in range(m.shape[0]))
    return psi


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="no 80-bit type")
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("family", FAMILIES)
def test_no_further_off_than_gate_by_gate(family, dtype):
    run2 = one2 = 0.0
    for seed in range(LISTS):
        gates = FAMILIES[family](40 + seed)
        want = in_80_bits(gates)
        sv, one = qvm.StateVector(N, dtype), qvm.StateVector(N, dtype)
        sv.run(gates)
        for g in gates:
            one.apply(g)
        off = [float(np.sum(np.abs(s.amplitudes().astype(np.clongdouble) - want) ** 2)) for s in (sv, one)]
        run2 += off[0]
        one2 += off[1]
    run, each = math.sqrt(run2 / LISTS), math.sqrt(one2 / LISTS)
    print(f"{family} {dtype}: list {run:.3g}, gate by gate {each:.3g}, ratio {run / each:.3f}", flush=True)
    assert run <= 1.1 * each
