"""Tiles and passes of a batch's compiled plans, read from the generated source."""
import re

import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

pytestmark = pytest.mark.gpu


def _source(lattice, count, seed, tmp_path, monkeypatch):
    """Source of the right half's plan, its qubits and its passes without sharing."""
    rows, cols, after, depth = lattice
    c = qsv.circuit_create(rows, cols, None, depth, seed)
    _, half, cuts, _ = qsv.circuit_split(c, sum(1 << (r * cols + x) for r in range(rows) for x in range(after + 1)))
    n = qsv.circuit_info(half)[0]
    dump = tmp_path / "passes.hip"
    monkeypatch.setenv("QSV_JIT_DUMP", str(dump))
    a = torch.empty(count, 1 << n, dtype=torch.complex64, device="cuda:0")
    batch = qsv.sv_batch_create([half] * count, [k % (1 << cuts) for k in range(count)])
    qsv.sv_batch_run(batch, [a.data_ptr() + 8 * k * a.stride(0) for k in range(count)], init_plus=True)
    torch.cuda.synchronize()
    return dump.read_text(), n, half


@pytest.mark.parametrize("count", [255, 256, 300, 512, 1024])
def test_15_qubit_states_on_the_2_13_tile(count, tmp_path, monkeypatch):
    """One workgroup of 1024 threads for a whole state lost against it between 256 and 512 states."""
    src, n, _ = _source((5, 6, 2, 12), count, 900 + count, tmp_path, monkeypatch)
    assert n == 15
    assert set(re.findall(r"__launch_bounds__\((\d+)", src)) == {"256"}


@pytest.mark.parametrize("lattice,count,shared", [
    ((4, 6, 2, 14), 1024, False), ((7, 4, 1, 14), 2048, False),      # one tile holds a state of 12 or 14 qubits
    ((6, 6, 2, 14), 20, False), ((6, 6, 2, 14), 64, True),           # 18 qubits
    ((5, 6, 2, 14), 30, False), ((5, 6, 2, 14), 300, True), ((4, 7, 2, 14), 255, True)])
def test_prefixes_shared_where_it_pays(lattice, count, shared, tmp_path, monkeypatch):
    """A plan cut for sharing has more passes than the circuit's own plan, or other ones."""
    src, n, half = _source(lattice, count, 70 + count, tmp_path, monkeypatch)
    tile = {12: (5, 7, 5), 14: (5, 9, 5)}.get(n, (5, 8, 5))
    own = qsv.sv_plan_info(half, 1, -1, dict(reg_qubits=tile[0], thread_qubits=tile[1], low_qubits=tile[2]))
    passes = len(re.findall(r"extern \"C\" __global__", src))
    assert (passes > own["n_passes"]) == shared, (passes, own["n_passes"])
