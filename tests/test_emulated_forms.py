"""sv_debug_emulate over the generic kernel's programs returns the state for
starts whose amplitudes grow, for any finite or non-finite start, and with the
default tiles of both lowered forms."""
import numpy as np
import pytest

from oracle import sim
from paper_1804_04797_amd import qsv, workloads

INVERSE = {"H": "H", "T": "TDG", "TDG": "T", "SX": "SXDG", "SXDG": "SX", "SY": "SYDG", "SYDG": "SY", "CZ": "CZ", "Z": "Z"}


def _circuit(n, names):
    a = np.zeros(len(names), qsv.GATE_DTYPE)
    for i, (k, q0, q1) in enumerate(names):
        a[i] = (qsv.KIND[k], q0, q1 if k == "CZ" else 0, 0, i, 0)
    gates = [(k, q0, q1 if k == "CZ" else -1, i) for i, (k, q0, q1) in enumerate(names)]
    return qsv.circuit_create(1, n, None, gates=a), gates


def _err(psi, ref):
    # one rounding of 2^-24 per gate; the length of the state is 1 throughout
    return np.linalg.norm(psi.astype(np.complex128) - ref)


@pytest.mark.parametrize("n", [12, 14, 16, 18])
def test_uniform_start_to_one_amplitude(n):
    rng = np.random.default_rng(n)
    there = []
    for _ in range(150):
        q0 = int(rng.integers(n))
        there.append((list(INVERSE)[rng.integers(len(INVERSE))], q0, (q0 + 1 + int(rng.integers(n - 1))) % n))
    back = [(INVERSE[k], q0, q1) for k, q0, q1 in reversed(there)]
    c, gates = _circuit(n, there + back + [("H", q, 0) for q in range(n)])
    psi = np.full(1 << n, 2.0 ** (-n / 2), np.complex64)
    qsv.sv_debug_emulate(psi, c)
    ref = np.zeros(1 << n, np.complex128)
    ref[0] = 1
    assert _err(psi, ref) <= 2.0 ** -24 * len(gates)


@pytest.mark.parametrize("n,depth", [(12, 24), (13, 20), (16, 16), (20, 12)])
@pytest.mark.parametrize("plus", [False, True])
def test_default_tiles(n, depth, plus):
    rows, cols, pres = workloads.lattice_for_qubits(n)
    c = qsv.circuit_create(rows, cols, pres, depth, 3 * n)
    gates = [(qsv.KIND_NAME[int(g["kind"])], int(g["q0"]), int(g["q1"]) if int(g["kind"]) == qsv.KIND["CZ"] else -1,
              int(g["layer"])) for g in c.gates()]
    start = np.zeros(1 << n, np.complex128)
    start[0] = 1
    if plus:
        start[:] = 2.0 ** (-n / 2)
    psi = start.astype(np.complex64)
    qsv.sv_debug_emulate(psi, c)
    assert _err(psi, sim.run(start, n, gates)) <= 2.0 ** -24 * len(gates)


@pytest.mark.parametrize("value", [np.inf, np.nan, 1e30, 1e-42, 0.0])
def test_any_start_is_taken(value):
    c, _ = _circuit(12, [("H", q % 12, 0) for q in range(24)] + [("T", q, 0) for q in range(12)])
    psi = np.zeros(1 << 12, np.complex64)
    psi[5] = value
    qsv.sv_debug_emulate(psi, c)
    if value in (1e30, 0.0):  # H twice: back to the start up to the phases of T
        want = np.zeros(1 << 12)
        want[5] = value
        assert np.max(np.abs(np.abs(psi) - want)) <= 2.0 ** -24 * 36 * value
