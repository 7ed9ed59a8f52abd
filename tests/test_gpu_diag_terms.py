"""Short diagonal runs of tile passes, each term on every kind of index bit:
the lanes of a wave (0 to 5), the waves of a workgroup (6 to 8), a thread's
elements (from 9) and the bits outside the tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,tile", [(4, 0), (8, 0), (9, 0), (10, 0), (12, 0), (13, 0), (14, 10)])
def test_terms_on_each_kind_of_bit(n, tile, dtype):
    from workloads import Gate
    # a rounded entry and two rounded products and their sum for each
    # component of an amplitude below 1; a sign is exact
    unit = 2.0 ** -53 if dtype == "c128" else 2.0 ** -24
    prep = [Gate("rx", (q,), (), (0.3 + 0.2 * q,)) for q in range(n)]
    idx = np.arange(1 << n)
    qubits = [q for q in (0, 5, 6, 8, 9, 11, n - 1) if q < n]
    pairs = [(a, b) for a in qubits for b in qubits if a < b]
    for a, b in pairs:
        both = ((idx >> a) & (idx >> b) & 1).astype(bool)
        for gates, factor in (([Gate("z", (a,), (b,))], -1), ([Gate("p", (a,), (b,), (0.7,))], np.exp(0.7j)),
                              ([Gate("z", (a,), (b,)), Gate("p", (b,), (a,), (0.7,))], -np.exp(0.7j))):
            sv = qvm.StateVector(n, dtype)
            sv.run(prep)
            want = sv.amplitudes()
            want = np.where(both, want * factor, want)
            plan = qvm.Plan(gates, n, dtype, k_max=3, tile_qubits=tile)
            assert plan.stats()["diag_ops"] == len(gates) and plan.stats()["blocks"] == 0
            plan.run(sv)
            err = float(np.max(np.abs(sv.amplitudes() - want)))
            assert err <= (0 if factor == -1 else 8 * unit), (n, a, b, gates, err)
