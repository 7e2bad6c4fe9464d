"""sv_batch_create's low_qubits reaches the compiled plans that entries share."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv, workloads

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count", [(16, 8), (18, 9)])
def test_low_qubits(n, count, tmp_path, monkeypatch):
    rows, cols, pres = workloads.lattice_for_qubits(n)
    states, sources, masks = [], [], []
    for low in (2, 9):
        c = qsv.circuit_create(rows, cols, pres, 12, 7)
        masks.append(qsv.sv_plan_info(c, 1, -1, dict(reg_qubits=5, thread_qubits=8, low_qubits=low))["resident"])
        dump = tmp_path / f"{low}.hip"
        monkeypatch.setenv("QSV_JIT_DUMP", str(dump))
        a = torch.empty(count, 1 << n, dtype=torch.complex64, device="cuda:0")
        b = qsv.sv_batch_create([c] * count, opts=dict(low_qubits=low))
        qsv.sv_batch_run(b, list(a), init_plus=True)
        torch.cuda.synchronize()
        del b
        states.append(a.cpu().numpy().astype(np.complex128))
        sources.append(dump.read_text())
    assert list(masks[0]) != list(masks[1]) and sources[0] != sources[1]
    gates = qsv.circuit_info(c)[2]
    # one rounding of 2^-24 per gate on an amplitude of size 2^{-n/2}, on each side
    assert np.max(np.abs(states[0] - states[1])) * 2.0 ** (n / 2) <= 2 * 2.0 ** -24 * gates


def test_run_after_a_run_that_could_not_be_planned():
    """Tables are built per start of the run: a start whose tuned tile does not fit
    is refused, the other one still runs."""
    n = 21
    c = qsv.circuit_create(*workloads.lattice_for_qubits(n), 6, 3)
    qsv.sv_tune_set(c, dict(reg_qubits=5, thread_qubits=8, low_qubits=30, jit=1), layer_begin=0)
    a = torch.empty(1 << n, dtype=torch.complex64, device="cuda:0")
    batch = qsv.sv_batch_create([c])
    qsv.sv_batch_run(batch, [a], init_plus=True)
    torch.cuda.synchronize()
    want = a.clone()
    with pytest.raises(qsv.QsvError):
        qsv.sv_batch_run(batch, [a], init_plus=False)
    a.zero_()
    qsv.sv_batch_run(batch, [a], init_plus=True)
    torch.cuda.synchronize()
    assert torch.equal(a, want)
