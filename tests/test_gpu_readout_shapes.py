"""Readouts at the sizes where their kernels change shape (states smaller
than a block's row of pieces, one to eight iterations, more blocks than
rows), on random states in a permuted layout, against the FP64 oracle: every
<Z_q>, Pauli strings of both kinds on low, high and mixed bits, marginals
with qubits inside and above a row, samples, the norm and its rescaling."""
import numpy as np
import pytest

import oracle
from tests.util import C128_TOL, c64_bound, cdf_eps, cdf_window, gate_ks
from workloads import Gate, layered_u3_cz

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


def paulis(n, rng):
    """Strings of any weight, several per x (more than 16 of one kind for
    x = 0), x on the lowest, the highest and mixed bits."""
    lim = 1 << n
    xs, zs = [], []
    for x in [0, 1, 1 << (n - 1), lim - 1] + [int(rng.integers(1, lim)) for _ in range(4)]:
        for z in {int(rng.integers(0, lim)) for _ in range(40 if x == 0 else 20)}:
            xs.append(x)
            zs.append(z)
    order = rng.permutation(len(xs))
    return np.array(xs, np.uint64)[order], np.array(zs, np.uint64)[order]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 6, 8, 9, 10, 12, 13, 19, 21, 23])
def test_readouts_match_the_oracle(n, dtype):
    rng = np.random.default_rng(n)
    gates = layered_u3_cz(n, 3, 40 + n)
    sv = qvm.StateVector(n, dtype)
    sv.run(gates)
    if n >= 8:
        # relabelled wires: a permuted layout, no data moved
        p = [int(q) for q in rng.permutation(n)]
        swaps = [Gate("swap", (p[2 * i], p[2 * i + 1])) for i in range(n // 2)]
        qvm.Plan(swaps, n, dtype, k_max=3, tile_qubits=8).run(sv)
        gates = gates + swaps
    psi = oracle.simulate(n, gates)
    tau = 1e-13 if dtype == "c128" else c64_bound(gate_ks(gates))
    ptol = 2 * tau + tau * tau
    assert np.max(np.abs(sv.expect_z_all() - oracle.expect_z_all(psi))) <= 2 * ptol
    xs, zs = paulis(n, rng)
    got, _ = sv.expect_pauli(xs, zs)
    want = np.array([oracle.expect_pauli(psi, int(x), int(z))[0] for x, z in zip(xs, zs)])
    assert np.max(np.abs(got - want)) <= 2 * ptol
    for m in {1, n // 2, min(n, 11), min(n, 18)} - {0}:
        qs = [int(q) for q in rng.permutation(n)[:m]]
        assert np.max(np.abs(sv.probabilities(qs) - oracle.marginal(psi, qs))) <= 2 * ptol
    u = rng.random(400)
    s = sv.sample(u).astype(np.int64)
    cdf = np.cumsum(oracle.probabilities(psi))
    ok, _ = cdf_window(s, cdf, u, cdf_eps(tau) if dtype == "c64" else 1e-12)
    assert ok.all()
    assert abs(sv.norm() - float(cdf[-1])) <= 2 * ptol
    before = sv.renormalize()
    assert abs(before - float(cdf[-1])) <= 2 * ptol
    assert np.max(np.abs(sv.amplitudes() - psi)) <= (C128_TOL if dtype == "c128" else 2 * tau)


def test_many_strings_take_several_launches():
    """More x masks than one launch's jobs."""
    n = 11
    gates = layered_u3_cz(n, 3, 4)
    sv = qvm.StateVector(n, "c128")
    sv.run(gates)
    psi = oracle.simulate(n, gates)
    rng = np.random.default_rng(0)
    xs = rng.permutation(1 << n)[:1300].astype(np.uint64)
    zs = rng.integers(0, 1 << n, 1300).astype(np.uint64)
    got, tot = sv.expect_pauli(xs, zs, np.ones(1300))
    pick = rng.integers(0, 1300, 60)
    want = np.array([oracle.expect_pauli(psi, int(xs[i]), int(zs[i]))[0] for i in pick])
    assert np.max(np.abs(got[pick] - want)) <= 1e-13
    assert abs(tot - float(np.sum(got))) <= 1e-12


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 3, 8, 9, 10, 11, 13, 16, 18, 20, 24])
def test_marginals_of_runs_of_qubits(n, dtype):
    """Marginal qubits in one run and in several, at the bottom, across and
    above a row, in ascending and in any other order: rows folded over every
    set of their bits, sums in one launch and in two, few rows a block."""
    import torch
    rng = np.random.default_rng(n)
    v = rng.normal(size=(1 << n, 2)) / np.sqrt(2.0 ** (n + 1))
    v = v.astype(np.float32 if dtype == "c64" else np.float64)
    sv = qvm.StateVector(n, dtype)
    sv.amps.copy_(torch.from_numpy(v).reshape(sv.amps.shape))
    p = np.sum(v.astype(np.longdouble) ** 2, axis=1)            # (numpy adds along an axis one by one: in 80 bits)
    sets = {tuple(range(m)) for m in (1, 4, 7, 9, 12)} | {tuple(range(n - m, n)) for m in (1, 4, 8, 12, 16)}
    sets |= {tuple(range(n - 1, max(n - 9, -1), -1)), tuple(range(0, n, 3)), tuple(range(5, min(n, 12))),
             (n - 1,) + tuple(range(0, n - 1, 4)), tuple(range(6, min(n, 10))) + tuple(range(12, n))}
    for qs in sets:
        qs = tuple(q for q in qs if 0 <= q < n)
        if not qs or len(set(qs)) < len(qs) or len(qs) > 18:
            continue
        axes = p.reshape((2,) * n).sum(axis=tuple(n - 1 - q for q in range(n) if q not in qs))
        kept = sorted(qs, reverse=True)
        want = axes.transpose([kept.index(q) for q in reversed(qs)]).reshape(-1)
        got = sv.probabilities(list(qs))
        # sums of at most 2^24 positive terms in a tree
        assert np.max(np.abs(got - want) / want) <= 64 * 2.0 ** -53, (qs, np.max(np.abs(got - want) / want))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 8, 9, 17, 19, 20, 21, 24])
def test_norm_at_every_row_count(n, dtype):
    """Fewer rows than blocks, one, and some each."""
    import torch
    rng = np.random.default_rng(n)
    v = rng.normal(size=2 << n).astype(np.float32 if dtype == "c64" else np.float64)
    sv = qvm.StateVector(n, dtype)
    sv.amps.copy_(torch.from_numpy(v).reshape(sv.amps.shape))
    want = float(np.sum(v.astype(np.float64) ** 2))
    assert abs(sv.norm() - want) <= 64 * 2.0 ** -53 * want
