"""The adjoint sweeps' passes and groups against the FP64 oracle's adjoint: any
one-target gates with up to three controls, runs of rotations on one qubit,
matrices and shared parameters, on both sides of the tile widths and of the
slots a thread holds, and lists longer than a pass, a group and the record
table take."""
import numpy as np
import pytest

import oracle
from tests.util import c64_bound
from workloads import Gate

pytestmark = pytest.mark.gpu

adj = pytest.importorskip("paper_2212_14201_amd.adjoint")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


def any_gates(n, count, seed):
    rng = np.random.default_rng(seed)
    gates, P = [], 0
    while len(gates) < count:
        q = int(rng.integers(n))
        others = rng.permutation([x for x in range(n) if x != q])
        ctl = tuple(int(x) for x in others[:int(rng.choice([0, 0, 0, 1, 2, 3]))])
        kind = int(rng.integers(6))
        if kind < 2:                             # a run of rotations, some of them sharing a parameter
            for name in rng.permutation(["rx", "ry", "rz"])[:int(rng.integers(1, 4))]:
                share = P > 0 and rng.random() < 0.2
                gates.append(Gate(str(name), (q,), ctl if kind else (), (0.0,), int(rng.integers(P)) if share else P))
                P += not share
        elif kind == 2:
            m = np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]
            gates.append(Gate("unitary", (q,), ctl, (), -1, m))
        elif kind == 3:
            gates.append(Gate(str(rng.choice(["rx", "ry", "rz"])), (q,), ctl, (float(rng.uniform(0, 6)),)))
        else:
            gates.append(Gate(str(rng.choice(["h", "x", "y", "z", "s", "t"])), (q,), ctl))
    return gates, P


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,count,batch", [(1, 30, 2), (2, 60, 1), (3, 80, 3), (4, 80, 2), (5, 3000, 2), (10, 100, 1),
                                           (11, 100, 2), (12, 120, 2), (13, 120, 1), (15, 200, 3)])
def test_any_gates(n, count, batch, dtype):
    gates, P = any_gates(n, count, 100 + n)
    rng = np.random.default_rng(n)
    xs, zs = rng.integers(0, 1 << n, (2, 5)).astype(np.uint64)
    cs = rng.normal(size=5)
    theta = rng.uniform(-3, 3, (batch, P))
    f, g = adj.AdjointProblem(n, gates, P, xs, zs, cs, batch, dtype).run(theta)
    csum = float(np.sum(np.abs(cs)))
    # a rounding per gate forward, two in reverse; a shared parameter adds up its gates
    share = max([1] + [sum(x.pidx == p for x in gates) for p in range(P)])
    tol = (1e-12 * (1 + csum) if dtype == "c128" else 2 * c64_bound([1] * (3 * len(gates)) + [2] * 5) * csum) * share
    for b in range(batch):
        fo, go = oracle.adjoint(n, gates, theta[b], xs, zs, cs)
        err = max(abs(f[b] - fo), float(np.max(np.abs(g[b] - go))))
        print(f"n={n} {dtype} gates={len(gates)} b={b} err={err:.2e} tol={tol:.2e}", flush=True)
        assert err <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,count", [(2, 24), (5, 60), (9, 80), (12, 100), (14, 120)])
def test_matrices_that_are_not_unitary(n, count, dtype):
    """The sweep undoes a matrix by its adjoint.  For one that is not unitary
    the sums of gates on other qubits must then be taken in program order."""
    gates, P = any_gates(n, count, 700 + n)
    rng = np.random.default_rng(n)
    for at in sorted(rng.integers(0, len(gates), 3), reverse=True):
        m = np.array([[1.0, 0.3j], [-0.2, 0.8]]) + 0.1 * rng.normal(size=(2, 2))
        gates.insert(int(at), Gate("unitary", (int(rng.integers(n)),), (), (), -1, m / np.linalg.norm(m, 2)))
    gates += [Gate(r, (q,), (), (0.0,), P + 2 * q + i) for q in range(n) for i, r in enumerate(("rx", "ry"))]
    P += 2 * n
    gates.insert(len(gates) - n, Gate("unitary", (n - 1,), (0,) if n > 2 else (), (), -1, np.array([[0.5, 0.2], [0.1, 0.9]]) + 0j))
    xs, zs = rng.integers(0, 1 << n, (2, 5)).astype(np.uint64)
    cs = rng.normal(size=5)
    theta = rng.uniform(-3, 3, (2, P))
    f, g = adj.AdjointProblem(n, gates, P, xs, zs, cs, 2, dtype).run(theta)
    csum = float(np.sum(np.abs(cs)))
    share = max(sum(x.pidx == p for x in gates) for p in range(P))
    tol = (1e-12 * (1 + csum) if dtype == "c128" else 2 * c64_bound([1] * (3 * len(gates)) + [2] * 5) * csum) * share
    for b in range(2):
        fo, go = oracle.adjoint(n, gates, theta[b], xs, zs, cs)
        err = max(abs(f[b] - fo), float(np.max(np.abs(g[b] - go))))
        print(f"n={n} {dtype} gates={len(gates)} b={b} err={err:.2e} tol={tol:.2e}", flush=True)
        assert err <= tol
