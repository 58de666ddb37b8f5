"""Krylov steps of the device GMRES at the edges of its kernels: around the 8 basis vectors of one inner-product
workgroup, the longest restart length, vectors shorter and longer than a workgroup's part, one and several
right-hand sides.  The residual is formed from the product itself, in complex128."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,o,v,naux,nrhs", [(1, 2, 3, 5, 1), (1, 4, 12, 48, 7), (3, 3, 6, 8, 2)])
@pytest.mark.parametrize("krylov", [1, 7, 8, 9, 17, 60])
@pytest.mark.parametrize("prec", [0, 1])
def test_solutions_meet_their_residual(nk, o, v, naux, nrhs, krylov, prec):
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, naux, nrhs, 31)
    rng = synth.rng_for(8100, nk, o, v)
    b1, b2 = synth.random_vectors(nrhs, nk, o, v, rng, 0.1, 0.1)
    b2 = b2 * nk
    c = lr.Context(0)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    tol = 1e-3 if krylov == 1 else 1e-10          # a restart length of 1 converges slowly
    x1, x2, rep = c.solve_response(b1, b2, case['omega'], tol=tol, precision=prec, krylov=krylov)
    y1, y2 = c.apply_sigma(x1, x2, case['omega'], lr.FP64)
    worst = 0.0
    for r in range(nrhs):
        # the solver's norm: singles + doubles / 4
        num = np.sum(np.abs(b1[r] - y1[r]) ** 2) + 0.25 * np.sum(np.abs(b2[r] - y2[r]) ** 2)
        den = np.sum(np.abs(b1[r]) ** 2) + 0.25 * np.sum(np.abs(b2[r]) ** 2)
        worst = max(worst, float(np.sqrt(num / den)))
    print(f"nk={nk} o={o} v={v} nrhs={nrhs} krylov={krylov} precision {prec}: residual {worst:.1e} {rep}", flush=True)
    assert rep['converged'] == 1
    assert worst <= 2 * tol                      # the estimate of the last step against the residual itself
    c.close()
