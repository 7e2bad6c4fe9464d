"""sv_branch_combine at the edges of its work split (columns per workgroup,
branch groups, remainders) against numpy in complex128.  Each product of FP32
values takes at most two FP64 roundings and a sum of nb terms nb - 1 more:
|error| <= (nb + 4) 2^-53 sum_b |a_b| |b_b| per component (times sqrt 2)."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("nb,m", [(1, 1), (3, 1), (5000, 1), (1, 63), (2, 64), (17, 65), (64, 3), (63, 255),
                                  (1025, 256), (2048, 1024), (300, 1021), (257, 4097), (9, 16384), (40, 20001)])
def test_branch_combine_shapes(nb, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(nb * 100003 + m)
    a, b = ((rng.standard_normal((nb, m)) + 1j * rng.standard_normal((nb, m))).astype(np.complex64) for _ in range(2))
    sign = rng.integers(0, 2, m).astype(np.int8) * 2 - 1
    ta, tb, ts = (torch.from_numpy(x).cuda() for x in (a, b, sign))
    a, b = a.astype(np.complex128), b.astype(np.complex128)
    ref = (a * b).sum(0)
    tol = (nb + 4) * 2.0 ** -53 * np.sqrt(2) * (np.abs(a) * np.abs(b)).sum(0)
    for s, want in ((ts, ref * sign), (None, ref)):
        out = torch.full((m,), float("nan"), dtype=torch.complex128, device="cuda")
        qsv.sv_branch_combine(ta, tb, nb, m, s, out)
        again = torch.empty_like(out)
        qsv.sv_branch_combine(ta, tb, nb, m, s, again)
        assert torch.equal(out, again)  # fixed order
        assert np.all(np.abs(out.cpu().numpy() - want) <= tol)
