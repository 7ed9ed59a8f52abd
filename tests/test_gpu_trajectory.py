"""Noisy runs in one call: groups of up to four qubits measured together,
against the FP64 oracle's trajectories, where the grouping can go wrong: states of fewer than four
qubits and of one tile, on both sides of the tile widths, gates passed over
between branchings, gates that are not unitary, noise on gates of more than
four qubits, controls named in any order, and a permuted layout."""
import functools

import numpy as np
import pytest

import oracle
from oracle import noise as onoise
from tests.util import C128_TOL, c64_bound, gate_ks
from workloads import Gate, layered_u3_cz, noisy_layers, random_mixed_circuit, uniform_stream

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")
noise = pytest.importorskip("paper_2212_14201_amd.noise")

MODEL = [("ry", "depolarizing", {"p": 0.08}), ("cnot", "damping", {"p": 0.2}), ("cnot", "dephasing", {"p": 0.1}),
         ("rz", "phase_damping", {"p": 0.15}), ("h", "bit_flip", {"p": 0.3}), ("toffoli", "bit_phase_flip", {"p": 0.2}),
         ("x+5c", "damping", {"p": 0.2}), ("rzz", "depolarizing", {"p": 0.1}), ("swap", "damping", {"p": 0.1})]


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


@functools.lru_cache(maxsize=None)
def oracle_run(n):
    """The oracle's trajectory with uniforms in the middle of the branch they
    draw, so that no decision lies near a boundary: (uniforms, branches,
    state, the smallest distance to a boundary)."""
    gates = circuits(n, 500 + n)
    model = noise.NoiseModel(MODEL)
    rng = np.random.default_rng(900 + n)
    psi = oracle.basis_state(n, 0)
    us, branches, gaps = [], [], []
    for g in gates:
        oracle.apply_matrix(psi, n, oracle.gate_matrix(g), g.targets, g.controls)
        for ops in model.channels_for(g):
            for q in tuple(g.targets) + tuple(g.controls):
                w = onoise.branch_weights(psi, n, q, ops)
                cum = np.concatenate([[0.0], np.cumsum(w / w.sum())])
                j = min(int(np.searchsorted(cum, rng.random(), side="right")) - 1, len(w) - 1)
                u = 0.5 * (cum[j] + cum[j + 1])
                psi, jj, _ = onoise.trajectory_step(psi, n, q, ops, u)
                assert jj == j
                us.append(u)
                branches.append(j)
                gaps.append(0.5 * (cum[j + 1] - cum[j]))
    return np.array(us), branches, psi, min(gaps)


def circuits(n, seed):
    g = noisy_layers(n, 2 if n < 20 else 1, seed)
    rng = np.random.default_rng(seed)
    if n >= 3:
        g += random_mixed_circuit(n, 30, seed, kmax=min(3, n), max_ctrl=min(2, n - 3))
        a, b, c = (int(q) for q in rng.permutation(n)[:3])
        g += [Gate("x", (a,), (c, b)), Gate("x", (b,), (a,)), Gate("x", (a,), (b,)),
              # not unitary: must not be passed over
              Gate("unitary", (c,), (), (), -1, np.array([[1.0, 0.2], [0.1, 0.7]]) + 0j), Gate("h", (a,)),
              Gate("swap", (c, a)), Gate("ry", (c,), (), (0.4,))]
    if n >= 8:
        g += [Gate("x", (2,), (7, 0, 5, 1, 6)), Gate("h", (3,)), Gate("rzz", (7, 0), (), (0.3,))]
    return g


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 8, 12, 13, 21])
def test_groups_match_the_oracle(n, dtype):
    gates = circuits(n, 500 + n)
    u, want_br, want, gap = oracle_run(n)
    assert gap > 1e-3
    sv = qvm.StateVector(n, dtype)
    br = noise.run_trajectory(sv, gates, noise.NoiseModel(MODEL), u)
    err = float(np.max(np.abs(sv.amplitudes() - want)))
    tol = C128_TOL if dtype == "c128" else 2 * c64_bound(gate_ks(gates) + [1] * len(want_br))
    print(f"n={n} {dtype} branchings={len(br)} smallest gap {gap:.1e} err {err:.1e} tol {tol:.1e}")
    assert br == want_br
    assert err <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_trajectory_on_a_permuted_layout(dtype):
    """The library call from a state that a fused plan left permuted, against
    the oracle's trajectory of the whole program."""
    n = 10
    first, then = layered_u3_cz(n, 4, 3), noisy_layers(n, 2, 8)
    model = [e for e in MODEL if e[0] in ("ry", "rz", "h")]
    m = noise.NoiseModel(model)
    u = uniform_stream(12, m.branchings(then))
    want, wbr, margins = onoise.noisy_run(n, first + then, model, u)
    sv = qvm.StateVector(n, dtype)
    qvm.Plan(first, n, dtype, k_max=3, tile_qubits=7).run(sv)
    assert np.any(sv.layout() != np.arange(n))
    rng_first, qubit, chan, chans = [0], [], [], [e[3] for e in m.entries]
    for g in then:
        for c, e in enumerate(m.entries):
            if e[0] == noise.gate_type(g):
                qubit.append(g.targets[0])
                chan.append(c)
        rng_first.append(len(qubit))
    assert min(margins) > 1e-4
    br = sv.run_trajectory(then, rng_first, qubit, chan, chans, u)
    assert br == wbr
    tol = C128_TOL if dtype == "c128" else 2 * c64_bound(gate_ks(first + then) + [1] * len(br))
    assert np.max(np.abs(sv.amplitudes() - want)) <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 9, 14, 21])
def test_lone_branchings(n, dtype):
    """One branching at a time: gates before it, on its qubits after it, on
    others meanwhile, and a group of two after it; from a permuted layout."""
    rng = np.random.default_rng(n)
    first = layered_u3_cz(n, 2, 7)
    a, b, c, d = (int(q) for q in rng.permutation(n)[:4])
    gates = [Gate("h", (a,)), Gate("rx", (a,), (), (0.4,)), Gate("x", (b,), (a,)), Gate("u3", (d,), (), (1.0, 2.0, 3.0)),
             Gate("z", (c,), (b,)), Gate("ry", (c,), (), (0.9,)), Gate("x", (d,), (c,)), Gate("h", (b,)), Gate("t", (b,)),
             Gate("swap", (a, d)), Gate("h", (c,)), Gate("x", (a,), (b,)), Gate("h", (d,))]
    at = {1: [a], 6: [c], 9: [a], 11: [b, a], 12: [d]}           # branchings after a gate
    ks = [noise.kraus_ops("damping", p=0.4), noise.kraus_ops("depolarizing", p=0.6)]
    psi = oracle.simulate(n, first)
    heads, qubit, chan, us, want = [0], [], [], [], []
    for i, g in enumerate(gates):
        oracle.apply_matrix(psi, n, oracle.gate_matrix(g), g.targets, g.controls)
        for q in at.get(i, []):
            k = len(us) % 2
            w = onoise.branch_weights(psi, n, q, ks[k])
            j = len(us) % len(w)
            us.append((np.sum(w[:j]) + 0.5 * w[j]) / w.sum())
            psi, jj, _ = onoise.trajectory_step(psi, n, q, ks[k], us[-1])
            qubit.append(q)
            chan.append(k)
            want.append(jj)
        heads.append(len(us))
    sv = qvm.StateVector(n, dtype)
    qvm.Plan(first, n, dtype, k_max=3, tile_qubits=min(n, 7)).run(sv)
    assert sv.run_trajectory(gates, heads, qubit, chan, ks, us) == want
    tol = C128_TOL if dtype == "c128" else 2 * c64_bound(gate_ks(first + gates) + [1] * len(us))
    assert np.max(np.abs(sv.amplitudes() - psi)) <= tol


@pytest.mark.parametrize("n,dtype", [(22, "c128"), (23, "c64")])
def test_measuring_workgroups_take_several_tiles(n, dtype):
    """1,024 tiles on 512 workgroups, a superposed state with coherences:
    several groups, the first one's rounds straight from memory."""
    rng = np.random.default_rng(n)
    gates = [Gate("ry", (q,), (), (float(rng.uniform(0, 6)),)) for q in range(n)]
    gates += [Gate("z", (q + 1,), (q,)) for q in range(0, n - 1, 2)] + [Gate("rx", (q,), (), (0.7 + q,)) for q in range(1, n, 3)]
    gates += [Gate("x", (0,), (n - 1,)), Gate("x", (n - 5,), (n - 1,)), Gate("h", (5,)), Gate("x", (n - 2,), (7,)),
              Gate("h", (n - 3,)), Gate("h", (1,))]
    model = noise.NoiseModel([("cnot", "depolarizing", {"p": 0.5}), ("h", "damping", {"p": 0.4})])
    psi, us, want = oracle.basis_state(n, 0), [], []
    for g in gates:
        oracle.apply_matrix(psi, n, oracle.gate_matrix(g), g.targets, g.controls)
        for ops in model.channels_for(g):
            for q in tuple(g.targets) + tuple(g.controls):
                w = onoise.branch_weights(psi, n, q, ops)
                j = len(us) % len(w)                         # (every branch is taken)
                us.append((np.sum(w[:j]) + 0.5 * w[j]) / w.sum())
                psi, jj, _ = onoise.trajectory_step(psi, n, q, ops, us[-1])
                want.append(jj)
    sv = qvm.StateVector(n, dtype)
    br = noise.run_trajectory(sv, gates, model, np.array(us))
    assert br == want
    tol = C128_TOL if dtype == "c128" else 2 * c64_bound(gate_ks(gates) + [1] * len(br))
    assert np.max(np.abs(sv.amplitudes() - psi)) <= tol


@pytest.mark.parametrize("n,dtype", [(4, "c128"), (4, "c64"), (6, "c128")])
def test_groups_longer_than_a_segment(n, dtype):
    """Thousands of noisy gates that never leave four qubits."""
    rng = np.random.default_rng(n)
    gates = []
    for _ in range(5000):
        a, b = (int(q) for q in rng.choice(4, 2, replace=False))
        gates.append([Gate("ry", (a,), (), (float(rng.uniform(0, 6)),)), Gate("x", (a,), (b,)), Gate("h", (n - 1,))]
                     [int(rng.choice(3, p=[0.3, 0.2, 0.5]))])
    model = noise.NoiseModel([("ry", "depolarizing", {"p": 0.05}), ("cnot", "damping", {"p": 0.1})])
    psi, us, want = oracle.basis_state(n, 0), [], []
    for g in gates:
        oracle.apply_matrix(psi, n, oracle.gate_matrix(g), g.targets, g.controls)
        for ops in model.channels_for(g):
            for q in tuple(g.targets) + tuple(g.controls):
                w = onoise.branch_weights(psi, n, q, ops)
                j = int(rng.choice(len(w), p=w / w.sum()))
                us.append((np.sum(w[:j]) + 0.5 * w[j]) / w.sum())
                psi, jj, _ = onoise.trajectory_step(psi, n, q, ops, us[-1])
                want.append(jj)
    sv = qvm.StateVector(n, dtype)
    br = noise.run_trajectory(sv, gates, model, np.array(us))
    assert br == want
    tol = C128_TOL if dtype == "c128" else 2 * c64_bound([1] * (len(gates) + len(us)))
    assert np.max(np.abs(sv.amplitudes() - psi)) <= tol


def test_group_beyond_the_plan_area():
    """Between two branchings, more dense gates on four qubits than the
    workspace holds records for at once (36,000 of 1,056 bytes; 32 MiB)."""
    n = 5
    rng = np.random.default_rng(1)
    ms = [np.linalg.qr(rng.normal(size=(8, 8)) + 1j * rng.normal(size=(8, 8)))[0] for _ in range(40)]
    gates = [Gate("h", (0,))]
    gates += [Gate("unitary", tuple(int(q) for q in rng.permutation(4)[:3]), (), (), -1, ms[int(rng.integers(40))])
              for _ in range(36000)]
    gates.append(Gate("h", (3,)))
    k = noise.kraus_ops("depolarizing", p=0.9)
    psi, us, want = oracle.basis_state(n, 0), [], []
    for i, g in enumerate(gates):
        oracle.apply_matrix(psi, n, oracle.gate_matrix(g), g.targets, g.controls)
        if i in (0, len(gates) - 1):
            w = onoise.branch_weights(psi, n, g.targets[0], k)
            us.append((w[0] + 0.5 * w[1]) / w.sum())
            psi, j, _ = onoise.trajectory_step(psi, n, g.targets[0], k, us[-1])
            want.append(j)
    first = [0] + [1] * (len(gates) - 1) + [2]
    sv = qvm.StateVector(n, "c128")
    assert sv.run_trajectory(gates, first, [0, 3], [0, 0], [k], us) == want == [1, 1]
    assert np.max(np.abs(sv.amplitudes() - psi)) <= C128_TOL


def test_argument_errors():
    sv = qvm.StateVector(5, "c128")
    g = [Gate("h", (0,))]
    k = noise.kraus_ops("damping", p=0.5)
    for q, c, ks, u in (([5], [0], [k], [0.5]), ([0], [1], [k], [0.5]), ([0], [0], [k], [1.0]),
                        ([0], [0], [np.zeros((17, 2, 2))], [0.5]), ([0], [0], [np.zeros((1, 2, 2))], [0.5])):
        with pytest.raises(qvm.QvmError):
            sv.run_trajectory(g, [0, 1], q, c, ks, u)
    assert sv.run_trajectory([], [0], [], [], [], []) == []
    assert abs(sv.norm() - 1) < 1e-12
