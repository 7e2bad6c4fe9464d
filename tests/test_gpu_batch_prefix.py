"""Batches whose entries share a circuit and differ in their branches: the part
of the circuit before the branches differ runs once for the entries it is the
same for.  Every entry against its own sv_simulate from |+>^n.

Tolerance: either side takes one rounding (2^-24 relative) per gate on an
amplitude; rounding errors of the two add up over amplitudes of size 2^{-n/2}:
scaled difference max|delta| 2^{n/2} <= 2 * 2^-24 * gates."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

pytestmark = pytest.mark.gpu
KINDS = ("H", "T", "SX", "SY", "CZ", "TDG", "Z")


def _circuit(n, depth, marks, seed):
    """Random layers; marks: layer -> branch bits that PB and ZB gates take there."""
    rng = np.random.default_rng(seed)
    gates = [(qsv.KIND["H"], q, 0, 0, 0, 0) for q in range(n)]
    for layer in range(1, depth + 1):
        for q in rng.permutation(n)[: n - n // 4]:
            k = KINDS[rng.integers(len(KINDS))]
            q1 = (int(q) + 1 + int(rng.integers(n - 1))) % n
            gates.append((qsv.KIND[k], int(q), q1 if k == "CZ" else 0, 0, layer, 0))
        for bit in marks.get(layer, ()):
            gates.append((qsv.KIND["ZB" if bit % 3 else "PB"], int(rng.integers(n)), 0, bit, layer, 0))
    g = np.zeros(len(gates), qsv.GATE_DTYPE)
    for i, x in enumerate(gates):
        g[i] = x
    return qsv.circuit_create(1, n, None, gates=g), len(gates)


CASES = [  # qubits, entries, branch bits by layer, distinct branches
    (15, 256, {1: (0, 1, 2), 5: (3, 4, 5, 6, 7)}, 256),     # whole states in one tile, scratch
    (15, 255, {1: (0, 1, 2), 5: (3, 4, 5, 6, 7)}, 200),     # tiles of 2^13, some entries equal
    (15, 300, {4: (0, 1)}, 4),                              # many equal entries
    (15, 256, {1: tuple(range(8))}, 256),                   # nothing to share
    (13, 600, {2: (0,), 4: (1, 2, 3), 6: (4, 5, 6, 7, 8, 9)}, 600),
    (17, 40, {2: (0, 1), 5: (2, 3, 4, 5)}, 40),
    (20, 70, {2: (0, 1, 2, 3, 4), 5: (5, 6)}, 70),          # the shared states are above the scratch limit
    (14, 20, {2: (0, 1), 5: (2, 3, 4)}, 20),                # few tiles: no sharing
]


@pytest.mark.parametrize("n,count,marks,distinct", CASES)
@pytest.mark.parametrize("init_plus", [True, False])
def test_entries_equal_their_own_run(n, count, marks, distinct, init_plus):
    c, gates = _circuit(n, 6, marks, 100 * n + count)
    rng = np.random.default_rng(count)
    ids = [int(x) for x in rng.permutation(np.arange(count) % distinct)]
    states = torch.empty(count, 1 << n, dtype=torch.complex64, device="cuda")
    where = [states.data_ptr() + 8 * i * states.stride(0) for i in range(count)]
    batch = qsv.sv_batch_create([c] * count, ids)
    one = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
    for _ in range(2):  # the second run replays the graph over the first one's results
        if not init_plus:
            states.zero_()
            states[:, 5] = 1
        qsv.sv_batch_run(batch, where, init_plus=init_plus)
    torch.cuda.synchronize()
    bound = 2 * 2.0 ** -24 * gates
    for i in range(0, count, max(1, count // 64)):
        if init_plus:
            qsv.sv_simulate(one, c, branch=ids[i], init_kind=qsv.INIT_PLUS, layer_begin=1)
        else:
            qsv.sv_simulate(one, c, branch=ids[i], init_kind=qsv.INIT_BASIS, basis=5)
        assert float((states[i] - one).abs().max()) * 2.0 ** (n / 2) <= bound, i
