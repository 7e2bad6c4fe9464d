"""sv_branch_combine_full keeps the accuracy of each component: products of the
FP32 inputs are exact in FP64, so the real part is off by the roundings of its own
sum of 2 nb terms (Ar Br, -Ai Bi) and the imaginary part by those of Ar Bi, Ai Br,
however much smaller it is: |error| <= 2 nb 2^-53 times the sum of its terms'
magnitudes; the complex64 form rounds once more (2^-24)."""
import numpy as np
import pytest

from paper_1804_04797_amd import qsv

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _combine(a, b, na, nb, flags, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = torch.zeros(1 << (na + nb), dtype=dtype, device="cuda")
    qsv.sv_branch_combine_full(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), len(a), na, nb, (1 << na) - 1,
                               [], [], out, flags=flags)
    return out.cpu().numpy().reshape(1 << nb, 1 << na).T


@pytest.mark.parametrize("na,nb,branches", [(7, 7, 1), (8, 7, 64), (9, 8, 33), (11, 11, 17)])
@pytest.mark.parametrize("ratio", [1.0, 1e-4, 1e-10])
def test_parts_of_unequal_size(na, nb, branches, ratio):
    rng = np.random.default_rng(na + branches)
    a, b = ((rng.standard_normal((branches, 1 << k)) + 1j * ratio * rng.standard_normal((branches, 1 << k))).astype(
        np.complex64) for k in (na, nb))
    ar, ai, br, bi = (x.astype(np.float64) for x in (a.real, a.imag, b.real, b.imag))
    ld = np.longdouble
    rows = slice(0, 1 << na, max(1, (1 << na) >> 5))  # reference sums in extended precision on some rows
    re = sum((ar[k, rows, None] * br[k]).astype(ld) - ai[k, rows, None] * bi[k] for k in range(branches))
    im = sum((ar[k, rows, None] * bi[k]).astype(ld) + ai[k, rows, None] * br[k] for k in range(branches))
    size = {"re": np.abs(ar[:, rows]).T @ np.abs(br) + np.abs(ai[:, rows]).T @ np.abs(bi),
            "im": np.abs(ar[:, rows]).T @ np.abs(bi) + np.abs(ai[:, rows]).T @ np.abs(br)}
    for flags, dtype, last in ((qsv.COMBINE_OUT_C128, torch.complex128, 0.0), (0, torch.complex64, 2.0 ** -24)):
        got = _combine(a, b, na, nb, flags, dtype)[rows]
        for part, ref, x in (("re", re, got.real), ("im", im, got.imag)):
            tol = 2 * branches * 2.0 ** -53 * size[part] + last * np.abs(ref) * (1 + 2.0 ** -20)
            assert np.all(np.abs(x.astype(ld) - ref) <= tol), (part, flags)


def test_infinite_input():
    """inf (1 + i) has two infinite components and nothing else is touched."""
    a, b = (np.ones((1, 1 << 7), np.complex64) for _ in range(2))
    a[0, 3] = complex(np.inf, 0.0)
    b[0] = 1 + 1j
    for flags, dtype in ((0, torch.complex64), (qsv.COMBINE_OUT_C128, torch.complex128)):
        got = _combine(a, b, 7, 7, flags, dtype)
        assert np.all(np.isposinf(got[3].real)) and np.all(np.isposinf(got[3].imag))
        assert np.array_equal(np.delete(got, 3, axis=0), np.full((127, 128), 1 + 1j))
