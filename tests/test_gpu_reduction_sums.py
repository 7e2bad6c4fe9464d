"""Norm and inner product in FP64: short sums on the way to the result.

For a state whose amplitudes all equal one 24-bit real x the products x^2 have 48
bits, so a sum of 2^k of them in pairs is exact and one of up to 32 equal partial
sums in a row is too (53 bits): every sum along the way is exact up to 29 qubits,
unless more are added in a row."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("n", [14, 15, 20, 24, 27, 28, 29])
def test_equal_amplitudes_sum_exactly(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    for mant in (0xffffff, 0xaaaaab, 0xc9539d):
        x = float(np.float32(mant * 2.0 ** -24))
        assert x * 2 ** 24 == mant
        a = torch.full((1 << n,), complex(x, 0.0), dtype=torch.complex64, device="cuda")
        want = float(mant * mant) * 2.0 ** (n - 48)
        qsv.sv_norm_fp64(a, n, out[:1])
        assert out[0].item() == want
        qsv.sv_inner_product(a, a, n, out)
        assert out.tolist() == [want, 0.0]
        del a


@pytest.mark.gpu
@pytest.mark.parametrize("n", [14, 20, 24])
def test_random_states(n):
    """Depth of the sums: 3 additions in a load, 2 over a round, 16 in a row at
    most, then trees over 256 threads, 8 sums and 1024 threads: fewer than 48
    roundings of 2^-53 on any path, relative to the sum of the magnitudes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    s = [(rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)).astype(np.complex64) for _ in range(2)]
    a, b = (x.astype(np.clongdouble) for x in s)
    dot, size = np.sum(a.conj() * b), float(np.sum(np.abs(a) * np.abs(b)))
    norm = float(np.sum((a * a.conj()).real))
    ta, tb = (torch.from_numpy(x).cuda() for x in s)
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    qsv.sv_norm_fp64(ta, n, out[:1])
    assert abs(out[0].item() - norm) <= 48 * 2.0 ** -53 * norm
    qsv.sv_inner_product(ta, tb, n, out)
    assert abs(complex(*out.tolist()) - complex(dot)) <= 2 * 48 * 2.0 ** -53 * size
