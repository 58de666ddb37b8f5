"""complex64 products of operands at the top of the fp32 range: finite numbers that round to an infinite bf16 number,
and infinities, give what the fp32 matrix cores give (sizes whose products run on the bf16 tiles)."""
import numpy as np
import pytest

from tests.sigma_cases import make_case

pytestmark = pytest.mark.gpu


def _context(lr, case):
    c = lr.Context(0)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    return c


@pytest.mark.parametrize("nk,o,v,naux,nrhs", [(1, 6, 40, 30, 48), (2, 8, 33, 20, 6)])
def test_large_finite_operands(nk, o, v, naux, nrhs):
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, naux, nrhs, 17)
    x2 = np.zeros_like(case['x2'])
    # one antisymmetric pair of elements of the last right-hand side, between the largest bf16 and the largest fp32
    # number as the products hold it; its products with the blocks, below 1 in magnitude, stay finite
    sign = {(2, 1): 1, (1, 2): -1}
    for (i, j), s in sign.items():
        for (a, b), u in sign.items():
            x2[-1, 0, 0, 0, i, j, a, b] = s * u * 3.4e38
    x1 = np.zeros_like(case['x1'])
    x1[:, 0, 0, 0] = 1.0
    c = _context(lr, case)
    scale = 2.0 ** -20
    for fn, norm in ((c.apply_sigma, nk), (c.apply_sigma_adjoint, 1 / nk)):     # (held as x2 / nk, z2 nk)
        y = fn(x1, x2 * norm, None, lr.FP32)
        z = fn(x1 * scale, x2 * norm * scale, None, lr.FP32)
        for a, b in zip(y, z):
            # the same operations a factor of 2^20 apart, but for the sums that overflow in one of them
            ok = np.abs(b) < 3e38 * scale
            assert np.isfinite(a[ok]).all(), (fn.__name__, int((~np.isfinite(a[ok])).sum()))
            e = np.abs(a[ok] * scale - b[ok]).max() / np.abs(b[ok]).max()
            print(f"nk={nk} o={o} v={v} {fn.__name__}: {e:.1e}", flush=True)
            assert e < 1e-6
    c.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_operands_that_are_not_finite(value):
    """What an element that is not finite reaches, and nothing else, is not finite: as in complex128."""
    import paper_2508_01266_amd as lr
    case = make_case(2, 8, 33, 20, 6, 18)
    x2 = case['x2'].copy()
    x2[3, 0, 1, 1, 2, 5, 7, 11] = value
    c = _context(lr, case)
    for fn in (c.apply_sigma, c.apply_sigma_adjoint):
        for a, b in zip(fn(case['x1'], x2, case['omega'], lr.FP32), fn(case['x1'], x2, case['omega'], lr.FP64)):
            bad = ~np.isfinite(b)
            print(f"{value} {fn.__name__}: {int(bad.sum())} of {b.size} not finite", flush=True)
            assert bad.any() and not bad.all()
            assert np.array_equal(~np.isfinite(a), bad)
    c.close()
