"""The generic kernel's lowered programs at their stated bound: scaled error
max|delta| 2^{n/2} <= 2^-24 * gates * norm, norm that of the reference (projections
shorten the state, and its rounding errors with it).  Branches whose projections
leave nothing are passed over."""
import numpy as np
import pytest

from oracle import sim
from paper_1804_04797_amd import qsv
from test_generic_programs import CASES, _explicit, _gates


@pytest.mark.parametrize("n,count,shape,br", CASES)
def test_emulated_programs_at_the_stated_bound(n, count, shape, br):
    c = _explicit(n, count, n * 1000 + count, br)
    o = dict(reg_qubits=shape[0], thread_qubits=shape[1], low_qubits=shape[2], jit=-1)
    start = np.zeros(1 << n, np.complex128)
    start[3] = 1
    done = 0
    for branch in range(32 if br else 1):
        gates = _gates(c, branch)
        ref = sim.run(start.copy(), n, gates)
        norm = np.linalg.norm(ref)
        if norm <= 0.01:  # this branch's projections leave nothing
            continue
        psi = start.astype(np.complex64)
        qsv.sv_debug_emulate(psi, c, branch=branch, opts=o)
        assert np.max(np.abs(psi - ref)) * 2.0 ** (n / 2) <= 2.0 ** -24 * len(gates) * norm
        done += 1
        if done == 2:
            break
    assert done
