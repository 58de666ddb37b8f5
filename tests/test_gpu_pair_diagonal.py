"""One-body terms of x2 by W-bar and the output step: orbitals that do not diagonalise the Fock matrix, at the edges
of the output's tiles (32 x 32) and over several of them, against the oracle; and the transpose, which acts on
the antisymmetric part of z2."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import FP32_REL, make_case, oracle_sigma, oracle_sigma_adjoint

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def _context(case, mesh):
    import paper_2508_01266_amd as lr
    c = lr.Context(0)
    if mesh is not None:
        c.set_kmesh(*mesh)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    return lr, c


@pytest.mark.parametrize("nk,o,v,naux,nrhs,mesh", [(1, 2, 2, 5, 3, None), (1, 3, 32, 9, 2, None), (1, 2, 33, 9, 1, None),
                                                   (1, 2, 45, 6, 1, None), (3, 2, 9, 7, 3, None), (4, 3, 5, 6, 2, (2, 2))])
def test_noncanonical_products_match_oracle(nk, o, v, naux, nrhs, mesh):
    case = make_case(nk, o, v, naux, nrhs, 90 + v, mesh=mesh, noncanonical=0.3)
    rng = synth.rng_for(9200 + v, nk, o, v)
    z1, z2 = synth.random_vectors(nrhs, nk if mesh is None else mesh, o, v, rng, 0.1, 0.1)
    z2 = z2 * nk
    ref, adj = oracle_sigma(case), oracle_sigma_adjoint(case, z1, z2)
    lr, c = _context(case, mesh)
    for prec, tol in ((lr.FP64, 1e-11), (lr.FP32, FP32_REL)):
        y = c.apply_sigma(case['x1'], case['x2'], case['omega'], prec)
        g = c.apply_sigma_adjoint(z1, z2, case['omega'], prec)
        e = [_rel(a, b) for a, b in zip(y + g, ref + adj)]
        print(f"nk={nk} o={o} v={v} nrhs={nrhs} precision {prec}: rel err {max(e):.1e}", flush=True)
        assert max(e) < tol
    c.close()


@pytest.mark.parametrize("nk,o,v", [(1, 3, 5), (3, 2, 4)])
def test_transpose_acts_on_the_antisymmetric_part(nk, o, v):
    """A^T z of an arbitrary z2 is that of its antisymmetric part."""
    nrhs = 2
    case = make_case(nk, o, v, 7, nrhs, 95, noncanonical=0.3)
    rng = synth.rng_for(9300, nk, o, v)
    z1 = rng.standard_normal((nrhs, nk, o, v)) + 1j * rng.standard_normal((nrhs, nk, o, v))
    shape = (nrhs, nk, nk, nk, o, o, v, v)
    z2 = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    p2 = np.stack([synth._antisym_blocks(z, nk) for z in z2]) / 2
    lr, c = _context(case, None)
    zero = np.zeros(nrhs)
    a = c.apply_sigma_adjoint(z1, z2, zero, lr.FP64)
    b = c.apply_sigma_adjoint(z1, p2, zero, lr.FP64)
    assert max(_rel(x, y) for x, y in zip(a, b)) < 1e-12
    c.close()
