"""Device memory that a batch holds for states its entries share: bounded over
all its plans, and the entries are right where it has run out."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

pytestmark = pytest.mark.gpu


def test_bounded_over_the_plans():
    """Ten circuits of 16 qubits, 128 entries each; 2^6 states are shared up to the
    second mark, 32 MiB a plan: four plans' worth fits 128 MiB."""
    n, plans, count = 16, 10, 128
    circuits = []
    for k in range(plans):
        rng = np.random.default_rng(k)
        g = [("H", q, 0, 0, 0) for q in range(n)]
        for layer in range(1, 13):
            g += [(("T", "SX", "SY")[rng.integers(3)], int(q), 0, 0, layer) for q in rng.permutation(n)[:8]]
            g += [("CZ", int(q), int(q + 1) % n, 0, layer) for q in rng.permutation(n)[:4]]
            if layer == 1:
                g += [("ZB", int(rng.integers(n)), 0, b, layer) for b in range(6)]
            if layer == 11:
                g += [("PB", int(rng.integers(n)), 0, 6, layer)]
        a = np.zeros(len(g), qsv.GATE_DTYPE)
        for i, (name, q0, q1, arg, layer) in enumerate(g):
            a[i] = (qsv.KIND[name], q0, q1, arg, layer, 0)
        circuits.append(qsv.circuit_create(1, n, None, gates=a))
    states = torch.empty(plans * count, 1 << n, dtype=torch.complex64, device="cuda:0")
    where = [states.data_ptr() + 8 * i * states.stride(0) for i in range(plans * count)]
    ids = list(range(count)) * plans
    batch = qsv.sv_batch_create([c for c in circuits for _ in range(count)], ids)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    qsv.sv_batch_run(batch, where, init_plus=True)
    torch.cuda.synchronize()
    held = free - torch.cuda.mem_get_info()[0]
    # tables, code and the graph take a few MiB each
    assert held <= (128 + 48) << 20, held >> 20
    one = torch.empty(1 << n, dtype=torch.complex64, device="cuda:0")
    for p, c in enumerate(circuits):
        bound = 2 * 2.0 ** -24 * qsv.circuit_info(c)[2]  # one rounding per gate, on either side
        for i in range(0, count, 9):
            qsv.sv_simulate(one, c, branch=i, init_kind=qsv.INIT_PLUS, layer_begin=1)
            assert float((states[p * count + i] - one).abs().max()) * 2.0 ** (n / 2) <= bound, (p, i)
