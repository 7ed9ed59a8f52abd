"""The state brought back to the identity layout (``reset_layout``) from any
layout: on both sides of the smallest permuted state and of the tile widths,
few and many swaps away, with and without the lowest bits; amplitudes are
moved, never changed."""
import numpy as np
import pytest

from workloads import Gate

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")
profiling = pytest.importorskip("paper_2212_14201_amd.profiling")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 7, 8, 9, 11, 12, 13, 14, 16, 19, 22])
def test_reset_layout(n, dtype):
    import torch
    rng = np.random.default_rng(n)
    fixed = list(range(n))
    for perm in ([int(p) for p in rng.permutation(n)], fixed[1:] + fixed[:1], fixed[::-1],
                 [n - 1] + fixed[1:-1] + [0], fixed[:-2] + [n - 1, n - 2], fixed):
        sv = qvm.StateVector(n, dtype)
        swaps, at = [], list(fixed)
        for q in range(n):                       # at[q]: which qubit ends up as q
            p = at.index(perm[q])
            if p != q:
                swaps.append(Gate("swap", (q, p)))
                at[p], at[q] = at[q], at[p]
        if swaps:
            qvm.Plan(swaps, n, dtype, k_max=3, tile_qubits=min(n, 12)).run(sv)
        state = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
        state = state.astype(np.complex64 if dtype == "c64" else np.complex128)
        sv.amps.copy_(torch.view_as_real(torch.from_numpy(state)).reshape(sv.amps.shape))
        want = sv.amplitudes()
        moved = [int(b) for b in sv.layout()] != fixed
        sv.reset_layout()
        assert [int(b) for b in sv.layout()] == fixed
        assert np.array_equal(sv.amplitudes(), want)
        assert np.array_equal(sv.amps.cpu().numpy().reshape(-1).view(state.dtype), want)
        print(f"n={n} {dtype} moved={moved}", flush=True)


@pytest.mark.parametrize("dtype,bit", [("c64", 3), ("c128", 2)])
def test_one_swap_with_the_highest_bit_of_a_line(dtype, bit):
    """A layout one such swap away moves half of the state, not all of it."""
    n = 20
    sv = qvm.StateVector(n, dtype)
    sv.init_basis(5)
    qvm.Plan([Gate("swap", (bit, n - 1))], n, dtype, k_max=3, tile_qubits=12).run(sv)
    profiling.begin(sv)
    sv.reset_layout()
    stats = profiling.end(sv)
    assert stats["swappair"]["launches"] == 1
    assert stats["swappair"]["bytes"] == (1 << n) * (8 if dtype == "c64" else 16)
