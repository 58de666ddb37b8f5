"""Grouped launches of the sigma and transpose programs (independent products of one dependency level
side by side, contributions to one tensor in separate arrays) against the oracle at the edges of their
tiles (16, 32 and 64 rows or columns, 16-deep reduction steps), with empty pair sets (one occupied or one
virtual orbital), split reductions and repeated applications on other inputs."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import FP32_REL, make_case, oracle_sigma, oracle_sigma_adjoint

pytestmark = pytest.mark.gpu

# (nk, o, v, naux, nrhs, mesh)
SIZES = [(1, 1, 1, 3, 1, None), (1, 1, 9, 5, 4, None), (1, 4, 1, 5, 2, None), (1, 4, 16, 17, 1, None),
         (1, 4, 17, 16, 2, None), (1, 3, 33, 20, 7, None), (2, 4, 8, 15, 16, None), (2, 5, 13, 9, 3, None),
         (3, 2, 7, 6, 33, None), (4, 2, 5, 4, 5, (2, 2))]


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


@pytest.mark.parametrize("nk,o,v,naux,nrhs,mesh", SIZES)
def test_grouped_products_match_oracle(nk, o, v, naux, nrhs, mesh):
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, naux, nrhs, 70 + v, mesh=mesh)
    rng = synth.rng_for(7200 + v, nk, o, v)
    z1, z2 = synth.random_vectors(nrhs, nk if mesh is None else mesh, o, v, rng, 0.1, 0.1)
    z2 = z2 * nk
    ref, adj = oracle_sigma(case), oracle_sigma_adjoint(case, z1, z2)
    c = lr.Context(0)
    if mesh is not None:
        c.set_kmesh(*mesh)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    for prec, tol in ((lr.FP64, 1e-11), (lr.FP32, FP32_REL)):
        c.apply_sigma(z1, z2, case['omega'], prec)          # other inputs first: nothing of them may stay
        y = c.apply_sigma(case['x1'], case['x2'], case['omega'], prec)
        c.apply_sigma_adjoint(case['x1'], case['x2'], case['omega'], prec)
        g = c.apply_sigma_adjoint(z1, z2, case['omega'], prec)
        pairs = nk * o > 1 and nk * v > 1
        if not pairs:      # no unique pair: the doubles vanish up to the rounding of the inputs' antisymmetry
            assert max(np.abs(a).max() for a in (y[1], g[1])) <= 10 * max(np.abs(a).max() for a in (case['x2'], z2))
        e = [_rel(a, b) for a, b in zip(y + g, ref + adj) if pairs or a.ndim == 4]
        print(f"nk={nk} o={o} v={v} nrhs={nrhs} precision {prec}: rel err {max(e):.1e}", flush=True)
        assert max(e) < tol
    c.close()
