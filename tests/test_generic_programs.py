"""The generic kernel's lowered programs: folded diagonals, paired Hadamards,
programs split at their op limit, projections and branch signs on every kind
of slot, against the oracle.

Tolerances: an amplitude takes one rounding (2^-24 relative) per gate on it,
at most `gates` of them, and rounding errors of a unitary circuit add up like
a random walk over amplitudes of size 2^{-n/2}: scaled error
max|delta| 2^{n/2} <= 2^-24 * gates (a bound far above the walk's)."""
import numpy as np
import pytest

from oracle import sim
from paper_1804_04797_amd import qsv, workloads

KINDS = ("H", "T", "SX", "SY", "CZ", "TDG", "SXDG", "SYDG", "Z")


def _gates(c, branch=0):
    out = []
    for g in c.gates():
        name, l = qsv.KIND_NAME[int(g["kind"])], (branch >> int(g["arg"])) & 1
        if name == "PB":
            name = "P1" if l else "P0"
        if name == "ZB":
            if not l:
                continue
            name = "Z"
        out.append((name, int(g["q0"]), int(g["q1"]) if name == "CZ" else -1, int(g["layer"])))
    return out


def _explicit(n, count, seed, branch_gates=False):
    rng = np.random.default_rng(seed)
    g = np.zeros(count, qsv.GATE_DTYPE)
    for i in range(count):
        k = KINDS[rng.integers(len(KINDS))]
        if branch_gates and i % 37 == 5:
            k = "ZB"
        if branch_gates and i % 151 == 60:
            k = "PB"
        q0 = int(rng.integers(n))
        q1 = (q0 + 1 + int(rng.integers(n - 1))) % n
        g[i] = (qsv.KIND[k], q0, q1 if k == "CZ" else 0, i % 5, i // 4, 0)
    return qsv.circuit_create(1, n, None, gates=g)


def _check(got, ref, gates):
    norm = np.sqrt(np.vdot(ref, ref).real)
    err = np.max(np.abs(got - ref)) * np.sqrt(ref.size)
    assert err <= 2.0 ** -24 * len(gates) * max(norm, 1e-3) * 4, err


CASES = [  # (qubits, gates, shape, branch gates): split programs, every tile, n = tile and larger
    (5, 60, (2, 3, 2), True), (7, 200, (3, 4, 3), True), (9, 300, (3, 6, 4), False), (11, 600, (4, 6, 4), True),
    (11, 300, (4, 7, 4), False), (12, 900, (4, 8, 4), True), (13, 400, (4, 8, 5), True), (13, 300, (4, 9, 4), False),
    (14, 500, (5, 7, 4), True), (13, 600, (5, 8, 5), False), (14, 300, (5, 9, 4), True), (15, 300, (6, 7, 5), True),
    (14, 400, (6, 8, 5), True),
]


@pytest.mark.parametrize("n,count,shape,br", CASES)
def test_emulated_programs(n, count, shape, br):
    c = _explicit(n, count, n * 1000 + count, br)
    o = dict(reg_qubits=shape[0], thread_qubits=shape[1], low_qubits=shape[2], jit=-1)
    for branch in (0, 0b10110) if br else (0,):
        psi = np.zeros(1 << n, np.complex64)
        psi[3] = 1
        qsv.sv_debug_emulate(psi, c, branch=branch, opts=o)
        start = np.zeros(1 << n, np.complex128)
        start[3] = 1
        gates = _gates(c, branch)
        _check(psi.astype(np.complex128), sim.run(start, n, gates), gates)


@pytest.mark.gpu
@pytest.mark.parametrize("n,count,shape,br", CASES)
def test_programs_on_device(n, count, shape, br):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = _explicit(n, count, n * 1000 + count, br)
    o = dict(reg_qubits=shape[0], thread_qubits=shape[1], low_qubits=shape[2], jit=-1)
    for branch in (0, 0b10110) if br else (0,):
        start = np.zeros(1 << n, np.complex128)
        start[3] = 1
        gates = _gates(c, branch)
        ref = sim.run(start, n, gates)
        src = torch.empty(1 << n, dtype=torch.complex64, device="cuda:0")
        qsv.sv_init(src, n, qsv.INIT_BASIS, 3)
        before = src.clone()
        dst, sim_out = torch.full_like(src, float("nan")), torch.full_like(src, float("nan"))
        norm = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        qsv.sv_apply_fused_from(src, dst, c, branch=branch, opts=o)
        qsv.sv_simulate(sim_out, c, branch=branch, init_kind=qsv.INIT_BASIS, basis=3, opts=o, norm_out=norm)
        assert torch.equal(src, before)
        qsv.sv_apply_fused(src, c, branch=branch, opts=o)
        assert torch.equal(src, dst)
        _check(dst.cpu().numpy().astype(np.complex128), ref, gates)
        got = sim_out.cpu().numpy().astype(np.complex128)
        _check(got, ref, gates)
        want = np.vdot(got, got).real
        assert abs(norm.item() - want) <= 1e-12 * max(want, 1e-30)


@pytest.mark.gpu
@pytest.mark.parametrize("n,depth", [(12, 24), (15, 30), (19, 16), (23, 8)])
def test_default_shapes_on_device(n, depth):
    """sv_simulate and sv_apply_fused take different default tiles; both agree with the oracle."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rows, cols, pres = workloads.lattice_for_qubits(n)
    c = qsv.circuit_create(rows, cols, pres, depth, 77 + n)
    gates = _gates(c)
    ref = sim.simulate(gates, n)
    a = torch.empty(1 << n, dtype=torch.complex64, device="cuda:0")
    b = torch.empty_like(a)
    qsv.sv_simulate(a, c)
    qsv.sv_init(b, n, qsv.INIT_ZERO)
    qsv.sv_apply_fused(b, c)
    for x in (a, b):
        _check(x.cpu().numpy().astype(np.complex128), ref, gates)


@pytest.mark.gpu
@pytest.mark.parametrize("n,shape,m", [
    (7, (3, 4, 3), 1), (9, (3, 4, 3), 5), (11, (4, 7, 4), 100), (12, (4, 7, 4), 0), (13, (4, 8, 4), 1),
    (14, (4, 6, 4), 7), (14, (5, 8, 5), 1024), (16, (4, 7, 4), 1025), (15, (5, 9, 4), 3), (17, (4, 8, 4), 64)])
def test_norm_from_the_last_program(n, shape, m):
    """One tile, tiles up to the reduction's own block count (n >= 14) and more
    of them.  A sum of nonnegative FP64 terms with at most 2^8 additions on any
    path to the result: relative error <= 2^8 * 2^-53 each."""
    import torch
    c = _explicit(n, 120, 90 + n)
    o = {"reg_qubits": shape[0], "thread_qubits": shape[1], "low_qubits": shape[2], "jit": -1}
    a = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
    norm = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(n)
    bits = torch.from_numpy(rng.integers(0, 1 << n, max(m, 1)).astype(np.int64)).cuda()
    out = torch.zeros(max(m, 1), dtype=torch.complex64, device="cuda")
    for _ in range(2):
        qsv.sv_simulate(a, c, init_kind=qsv.INIT_PLUS, opts=o, norm_out=norm, bitstrings=bits if m else None,
                        amps_out=out if m else None)
    s = a.cpu().numpy().astype(np.complex128)
    want = float(np.sum(s.real ** 2 + s.imag ** 2))
    assert abs(float(norm[0]) - want) <= 2 * 2.0 ** 8 * 2.0 ** -53 * want
    if m:
        assert torch.equal(out, a[bits])
