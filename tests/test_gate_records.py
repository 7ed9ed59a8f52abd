"""GateArray's records against the field-by-field way of writing them: every
kind of gate, parameters by index, lists and arrays of any number type, and
what a record cannot hold."""
import ctypes

import numpy as np
import pytest

from paper_2212_14201_amd import qvm
from workloads import Gate, layered_u3_cz, random_mixed_circuit


def by_field(gates, params=None):
    arr = (qvm.QvmGate * max(1, len(gates)))()
    keep = []
    for rec, g in zip(arr, gates):
        ps = list(g.params)
        if params is not None and g.pidx is not None and g.pidx >= 0:
            ps = [float(params[g.pidx])]
        u = None
        if g.name == "unitary":
            u = np.ascontiguousarray(np.asarray(g.matrix, np.complex128)).view(np.float64).ravel().copy()
            keep.append(u)
        qvm.GateArray._record(rec, qvm.KIND[g.name], g.targets, g.controls, ps, u)
    return arr, keep


def fields(arr, n):
    return [(r.kind, r.k, list(r.targets), r.ctrl_mask, list(r.params),
             [r.u[i] for i in range(2 << (2 * r.k))] if r.u else None) for r in arr[:n]]


@pytest.mark.parametrize("gates", [
    random_mixed_circuit(9, 120, 3, kmax=3, max_ctrl=2), layered_u3_cz(6, 3, 4), [],
    [Gate("x", [np.int64(3)], (np.int32(1), 2)), Gate("rz", (0,), (), [np.float32(0.5)]), Gate("u3", (1.0,), (), (1, 2, 3)),
     Gate("p", (True,), (), (0.25, 7.0, 8.0, 9.0)), Gate("z", (2**31 + 5,), (70,)), Gate("h", (-1,)),
     Gate("x", np.array([1]), np.array([0])), Gate("rx", np.array([2]), np.array([1, 3]), np.array([0.0]))]],
    ids=["mixed", "layered", "empty", "odd"])
def test_records(gates):
    ga = qvm.GateArray(gates)
    arr, keep = by_field(gates)
    assert ga.n == len(gates) and fields(ga.arr, ga.n) == fields(arr, ga.n)
    assert ctypes.sizeof(ga.arr) == 72 * max(1, len(gates))


@pytest.mark.parametrize("params", [np.arange(4) * 0.3, np.arange(4, dtype=np.float32), [0.1, 2, np.float64(3), 4.5],
                                    np.arange(4)])
def test_parameters_by_index(params):
    gates = [Gate("ry", (q,), (), (9.0,), p) for q, p in enumerate((2, -1, 0, 3))]
    arr, _ = by_field(gates, params)
    assert fields(qvm.GateArray(gates, params).arr, 4) == fields(arr, 4)


def test_refused():
    for bad, err in ((Gate("no", (0,)), KeyError), (Gate("x", tuple(range(9))), IndexError), (Gate("x", (0,), (-1,)), ValueError),
                     (Gate("rz", (0,), (), ("a",)), ValueError), (Gate("x", (None,)), TypeError)):
        with pytest.raises(err):
            qvm.GateArray([bad])
    with pytest.raises(IndexError):
        qvm.GateArray([Gate("rz", (0,), (), (0.0,), 5)], np.zeros(2))


@pytest.mark.parametrize("again", [
    lambda v: map(float, v), lambda v: (x for x in v), lambda v: reversed(v[::-1]), iter,
    lambda v: dict.fromkeys(v).keys()], ids=["map", "generator", "reversed", "iterator", "keys"])
def test_iterators(again):
    """Parameters and controls that can be read once only; a fourth parameter
    (not held by a record) sends the record the other way."""
    ps, cs = [0.1, 0.2, 0.3], [3, 1, 2]
    make = lambda f: [Gate("u3", (0,), (), f(ps)), Gate("rx", (0,), f(cs), f(ps[1:2])),  # noqa: E731
                      Gate("u3", (4.0,), f(cs), f(ps)), Gate("p", (0,), (), f(ps + [7.0]))]
    arr, _ = by_field(make(list))
    assert fields(qvm.GateArray(make(again)).arr, 4) == fields(arr, 4)


def test_indexed_parameter_of_a_gate_without_parameters():
    with pytest.raises(TypeError):               # (a gate's own parameters have to be a sequence all the same)
        qvm.GateArray([Gate("ry", (2,), (), None, 0)], [0.7])
