"""Gate lists whose one-target gates are split into rotations and phases that
wait on their bit (``sv.run``): phases that must be applied before, after or
through the gates around them, on slots, other tile bits and outer bits, and
factors of the whole state, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from tests.util import C128_TOL, c64_bound, gate_ks
from workloads import Gate

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


def waiting_phases(n, count, seed):
    """Rotations, phases, X and Y (through which a phase passes as its
    conjugate) and general unitaries, with diagonal, controlled and two-target
    gates in between; one bit with phases alone."""
    rng = np.random.default_rng(seed)
    last = n - 1
    g = [Gate("h", (q,)) for q in range(n)]
    while len(g) < count:
        a, b, c = (int(v) for v in rng.choice(last, 3, replace=False))
        th = tuple(float(v) for v in rng.uniform(-7, 7, 3))
        u = np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]
        anti = np.array([[0, np.exp(1j * th[0])], [np.exp(1j * th[1]), 0]])
        g += [[Gate("u3", (a,), (), th)], [Gate("rz", (a,), (), th[:1]), Gate("x", (a,))], [Gate("t", (a,)), Gate("y", (a,))],
              [Gate("rx", (a,), (), th[:1])], [Gate("ry", (a,), (), (0.0,)), Gate("ry", (b,), (), (np.pi,))],
              [Gate("unitary", (a,), (), (), -1, anti)], [Gate("unitary", (a,), (), (), -1, u)],
              [Gate("z", (a,), (b,)), Gate("z", (b,), (c,))], [Gate("p", (a,), (b,), th[:1])], [Gate("rzz", (a, b), (), th[:1])],
              [Gate("x", (a,), (b,))], [Gate("ry", (a,), (b, c), th[:1])], [Gate("swap", (a, b), (c,))],
              [Gate("rz", (last,), (), th[:1]), Gate("s", (last,)), Gate("z", (last,), (a,))]][int(rng.integers(14))]
    return g


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 8, 12, 13, 16, 21])
def test_waiting_phases(n, dtype):
    gates = waiting_phases(n, 150, 300 + n)
    sv = qvm.StateVector(n, dtype)
    sv.run(gates)
    want = oracle.simulate(n, gates)
    tol = C128_TOL if dtype == "c128" else c64_bound(gate_ks(gates))
    err = float(np.max(np.abs(sv.amplitudes() - want)))
    print(f"n={n} {dtype} gates={len(gates)} err={err:.2e} tol={tol:.2e}", flush=True)
    assert err <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_phases_alone_and_undone(dtype):
    """Lists of phases alone, a list that undoes itself, and many signs."""
    n = 14
    rng = np.random.default_rng(5)
    ang = [(float(v),) for v in rng.uniform(-7, 7, n)]
    signs = [Gate("z", (int(a),), (int(b),)) for a, b in (rng.choice(n, 2, replace=False) for _ in range(200))]
    spread = [Gate("h", (q,)) for q in range(n)]
    for gates in ([Gate("rz", (q,), (), ang[q]) for q in range(n)],
                  [Gate("s", (0,)), Gate("x", (1,), (0,)), Gate("z", (0,)), Gate("x", (1,), (0,)), Gate("s", (0,))],
                  signs, spread + signs + spread):
        sv = qvm.StateVector(n, dtype)
        sv.run(spread)
        sv.run(gates)
        want = oracle.simulate(n, spread + gates)
        tol = C128_TOL if dtype == "c128" else c64_bound(gate_ks(spread + gates))
        assert float(np.max(np.abs(sv.amplitudes() - want))) <= tol
