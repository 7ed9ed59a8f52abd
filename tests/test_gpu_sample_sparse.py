"""Samples of states most of whose amplitudes are zero, drawn with uniforms at
and next to the steps of the distribution, where offsets that are sums of the
same numbers in another order differ in the last place: no index without
probability may come out, and none further than that from its place."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

qvm = pytest.importorskip("paper_2212_14201_amd.qvm")


@pytest.fixture(autouse=True)
def _gpu(require_gpu):
    pass


# one chunk; chunks of one group, several and many; chunks with one amplitude and with thousands
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,count", [(3, 3), (9, 40), (12, 700), (16, 9), (20, 120), (22, 700), (24, 1500), (24, 40000), (25, 5000)])
def test_only_indices_with_probability(n, count, dtype):
    import torch
    rng = np.random.default_rng(n + count)
    ix = np.sort(rng.choice(1 << n, count, replace=False))
    w = rng.uniform(0.1, 1.0, count) * 10.0 ** rng.uniform(-3, 0, count)
    real = np.float32 if dtype == "c64" else np.float64
    v = np.zeros((count, 2), real)
    v[:, 0] = np.sqrt(w / w.sum())
    sv = qvm.StateVector(n, dtype)
    a = sv.amps.view(-1, 2)
    a.zero_()
    a[torch.from_numpy(ix).to(a.device)] = torch.from_numpy(v).to(a.device)
    p = v[:, 0].astype(np.float64) ** 2
    cdf = np.cumsum(p.astype(np.longdouble))
    edge = (cdf / cdf[-1]).astype(np.float64)
    steps = [edge]
    for to in (0.0, 2.0):
        e = edge
        for _ in range(4):
            e = np.nextafter(e, to)
            steps.append(e)
    u = np.concatenate(steps + [rng.random(500), [0.0, np.nextafter(1.0, 0.0)]])
    u = u[(u >= 0.0) & (u < 1.0)]
    s = sv.sample(u).astype(np.int64)
    k = np.searchsorted(ix, s)
    assert np.all((k < count) & (ix[np.minimum(k, count - 1)] == s)), "an index without probability"
    # the sums of 2^n probabilities in any order: the relative error of one of
    # at most 64 roundings, doubled for the target
    t, eps = u * float(cdf[-1]), 128 * 2.0 ** -53
    hi, lo = cdf[k].astype(np.float64), np.concatenate([[0.0], cdf[:-1].astype(np.float64)])[k]
    assert np.all((t >= lo - eps) & (t <= hi + eps))


@pytest.mark.parametrize("n", [5, 12, 14, 23])
def test_states_without_probability(n):
    """All zeros draw the last index, as without amplitudes past the target."""
    sv = qvm.StateVector(n, "c64")
    sv.amps.zero_()
    assert np.all(sv.sample([0.0, 0.5, 0.999]) == (1 << n) - 1)
