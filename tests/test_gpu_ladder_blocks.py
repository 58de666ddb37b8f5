"""Ladder over integral blocks whose tiles without unique pairs are left out, against the kernel that rebuilds the
integrals itself, at virtual counts around the edges of the tiles (16, 32, 64 and 128 rows of (e, a))."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,o,v,naux,nrhs", [(1, 2, 2, 4, 1), (1, 3, 3, 5, 2), (1, 2, 8, 7, 1), (1, 3, 16, 9, 3),
                                              (1, 2, 17, 30, 2), (1, 2, 33, 20, 1), (1, 2, 65, 24, 1), (2, 2, 5, 6, 2),
                                              (2, 3, 13, 26, 5), (4, 2, 9, 8, 1)])
@pytest.mark.parametrize("mode", [2, 3])
def test_block_ladder_matches_rebuilt_integrals(nk, o, v, naux, nrhs, mode):
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, naux, nrhs, 60 + v)
    rng = synth.rng_for(9600 + v, nk, o, v)
    z1, z2 = synth.random_vectors(nrhs, nk, o, v, rng, 0.1, 0.1)
    z2 = z2 * nk
    out = {}
    for m in (1, mode):
        c = lr.Context(0)
        c.set_ladder_mode(m)
        c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
        c.set_amplitudes(case['t1'], case['t2'])
        out[m] = [y for prec in (lr.FP64, lr.FP32) for y in
                  c.apply_sigma(case['x1'], case['x2'], case['omega'], prec) +
                  c.apply_sigma_adjoint(z1, z2, case['omega'], prec)]
        c.close()
    for q, (a, b) in enumerate(zip(out[mode], out[1])):
        e = float(np.abs(a - b).max() / np.abs(b).max())
        # rounding of sums of some thousand products, in complex128 (first four) and complex64
        assert e < (1e-12 if q < 4 else 5e-6), (q, e)
    print(f"nk={nk} o={o} v={v} mode {mode}: ok", flush=True)
