"""Input and output kernels where many short rows go to one wave each, against the same vectors applied few at a
time (a workgroup per row), at the edges of a wave's 64 lanes and of the rule's 512 elements."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v,nrhs", [(4, 2, 77), (4, 8, 76), (4, 9, 80), (4, 16, 76), (4, 22, 76)])
def test_many_right_hand_sides_match_few(o, v, nrhs):
    import paper_2508_01266_amd as lr
    nk, few = 3, 7
    assert nk ** 3 * o * o * nrhs >= 32768 > nk ** 3 * o * o * few
    case = make_case(nk, o, v, 6, 1, 50 + v, noncanonical=0.2)
    rng = synth.rng_for(9400 + v, nk, o, v)
    x1, x2 = synth.random_vectors(nrhs, nk, o, v, rng, 0.1, 0.1)
    x2 *= nk
    omega = np.linspace(-0.1, 0.1, nrhs)
    c = lr.Context(0)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    # rounding of sums of at most some ten thousand products: complex128 and complex64
    for prec, tol in ((lr.FP64, 1e-12), (lr.FP32, 2e-6)):
        for fn in (c.apply_sigma, c.apply_sigma_adjoint):
            y1, y2 = fn(x1, x2, omega, prec)
            for r0 in range(0, nrhs, few):
                s = slice(r0, r0 + few)
                a1, a2 = fn(x1[s], x2[s], omega[s], prec)
                e = max(np.abs(y1[s] - a1).max() / np.abs(a1).max(), np.abs(y2[s] - a2).max() / np.abs(a2).max())
                assert e < tol, (prec, fn.__name__, r0, e)
        print(f"o={o} v={v} precision {prec}: ok", flush=True)
    c.close()
