"""Gate lists that share passes over the state (``sv.run``): every kind of
gate, on both sides of each size at which the tile width or the amplitudes a
thread holds change, against the FP64 oracle and the one-gate kernels
(``sv.apply``), in the identity and in a permuted layout, and captured."""
import numpy as np
import pytest

import oracle
from tests.util import C128_TOL, c64_bound, gate_ks
from workloads import Gate, layered_u3_cz, random_mixed_circuit

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


def every_kind(n, seed):
    """Mixed gates with up to two controls, then the forms with a rule of
    their own: swaps and two- and three-target matrices in both orders of
    their targets, parity and general diagonals across the lowest and the
    highest bits, matrices that are moves, and runs that merge or cancel."""
    rng = np.random.default_rng(seed)
    g = random_mixed_circuit(n, 90, seed, kmax=min(3, n), max_ctrl=min(2, max(0, n - 3)))
    perm = np.zeros((8, 8))
    perm[np.arange(8) ^ 5, np.arange(8)] = 1
    for a, b, c in ((0, n - 1, n // 2), (n - 1, 0, 1), (1, n // 2, n - 1)):
        th = float(rng.uniform(0, 6))
        g += [Gate("swap", (a, b)), Gate("swap", (b, a), (c,)), Gate("rzz", (b, a), (c,), (th,)),
              Gate("unitary", (a, c, b), (), (), -1, np.diag(np.exp(1j * rng.uniform(0, 6, 8)))),
              Gate("unitary", (b, a), (c,), (), -1, np.diag(np.exp(1j * rng.uniform(0, 6, 4)))),
              Gate("unitary", (c, b, a), (), (), -1, perm), Gate("x", (a,), (b, c)), Gate("y", (b,), (a,))]
        g += [Gate("h", (a,)), Gate("t", (a,)), Gate("rx", (a,), (), (th,)), Gate("x", (b,)), Gate("x", (b,)),
              Gate("s", (c,)), Gate("z", (c,)), Gate("rz", (c,), (a,), (th,))]
    return g


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 5, 9, 12, 13, 14, 17, 20, 21, 22])
def test_every_gate_kind(n, dtype):
    gates = every_kind(n, 70 + n)
    init = (1 << n) - 3
    sv = qvm.StateVector(n, dtype, init=init)
    sv.run(gates)
    got = sv.amplitudes()
    one = qvm.StateVector(n, dtype, init=init)
    for g in gates:
        one.apply(g)
    want = oracle.simulate(n, gates, init=init)
    tol = C128_TOL if dtype == "c128" else c64_bound(gate_ks(gates))
    err, err1 = np.max(np.abs(got - want)), np.max(np.abs(got - one.amplitudes()))
    print(f"n={n} {dtype} gates={len(gates)} err={err:.2e} against the one-gate kernels {err1:.2e}")
    assert err <= tol and err1 <= 2 * tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_permuted_layout(dtype):
    """A list run on the layout that a fused plan leaves behind."""
    n = 15
    first, then = layered_u3_cz(n, 6, 3), every_kind(n, 5)
    sv = qvm.StateVector(n, dtype)
    qvm.Plan(first, n, dtype, k_max=3, tile_qubits=8).run(sv)
    assert np.any(sv.layout() != np.arange(n))
    sv.run(then)
    want = oracle.simulate(n, first + then)
    tol = C128_TOL if dtype == "c128" else c64_bound(gate_ks(first + then))
    assert np.max(np.abs(sv.amplitudes() - want)) <= tol


def test_long_list_and_single_gates():
    """More gates than the scheduler takes at once, and lists of one gate."""
    n = 6
    gates = random_mixed_circuit(n, 5000, 8, kmax=3, max_ctrl=2)
    sv = qvm.StateVector(n, "c128")
    sv.run(gates)
    for g in gates[:40]:
        sv.run([g])
    sv.run([])
    want = oracle.simulate(n, gates + gates[:40])
    assert np.max(np.abs(sv.amplitudes() - want)) <= C128_TOL


def test_captured_list_replays():
    """A captured run holds its gate records: replays after other eager runs
    on the same workspace give the eager result."""
    import torch
    n = 13
    gates, other = every_kind(n, 3), every_kind(n, 4)
    ga = qvm.GateArray(gates)
    sv = qvm.StateVector(n, "c64")
    sv.run(ga)
    want = sv.amplitudes()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sv.sync_stream()
        sv.init_basis(0)
        sv.run(ga)
    sv.sync_stream()
    for _ in range(3):
        sv.run(other)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(sv.amplitudes(), want)
