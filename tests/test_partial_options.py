"""Options that name only a part of the tile shape: every entry point completes
them from one default, so all take or refuse the same ones."""
import itertools

import pytest

from paper_1804_04797_amd import qsv, workloads


def _status(call, *a):
    try:
        call(*a)
        return 0
    except qsv.QsvError as e:
        return e.status


@pytest.mark.parametrize("n", list(range(11, 18)) + [23, 24])
def test_same_answer_everywhere(n):
    rows, cols, pres = workloads.lattice_for_qubits(n)
    c = qsv.circuit_create(rows, cols, pres, 4, n)
    for r, t, low in itertools.product((0, 3, 4, 5, 6), (0, 6, 7, 8, 9), (0, 4, 9)):
        if (r and t) or not (r or t or low):
            continue
        o = dict(reg_qubits=r, thread_qubits=t, low_qubits=low)
        assert _status(qsv.sv_plan_info, c, 1, -1, o) == _status(qsv.sv_workspace_bytes, c, 1, -1, o), o


@pytest.mark.parametrize("n,part,ok", [
    (12, dict(reg_qubits=5), True), (12, dict(reg_qubits=4), True), (12, dict(thread_qubits=7), True),
    (12, dict(thread_qubits=8), False), (12, dict(thread_qubits=6), False), (13, dict(thread_qubits=9), False),
    (14, dict(thread_qubits=9), True), (16, dict(thread_qubits=6), False), (16, dict(low_qubits=9), True),
    (12, dict(low_qubits=9), False)])
def test_completed_from_the_largest_tile(n, part, ok):
    rows, cols, pres = workloads.lattice_for_qubits(n)
    c = qsv.circuit_create(rows, cols, pres, 4, n)
    assert (_status(qsv.sv_plan_info, c, 1, -1, part) == 0) == ok
