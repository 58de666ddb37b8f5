"""Forward product of doubles of any symmetry: the one-body terms of x2 from the difference of two Fock matrices, at the edges of the output's tiles (32 x 32), on chains and a mesh; and products
written over their operands."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import FP32_REL, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,o,v,nrhs,mesh", [(1, 1, 1, 1, None), (1, 3, 5, 2, None), (1, 2, 33, 1, None),
                                              (3, 2, 5, 3, None), (4, 2, 4, 2, (2, 2))])
def test_one_body_terms_of_any_doubles(nk, o, v, nrhs, mesh):
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, 6, nrhs, 40 + v, mesh=mesh, noncanonical=0.3)
    rng = synth.rng_for(9700 + v, nk, o, v)
    x2 = rng.standard_normal(case['x2'].shape) + 1j * rng.standard_normal(case['x2'].shape)
    d = rng.standard_normal((nk, o + v, o + v)) + 1j * rng.standard_normal((nk, o + v, o + v))
    d[:, :o, o:] = d[:, o:, :o] = 0
    d += d.conj().transpose(0, 2, 1)
    fock = case['H']['fock']
    shifted = fock + d
    upper = np.triu(np.ones((v, v)), 1)
    h = np.empty_like(x2)
    for ki in range(nk):
        for kj in range(nk):
            for ka in range(nk):
                kb = synth.kb_of(ki, kj, ka, nk if mesh is None else mesh)
                x, w = x2[:, ki, kj, ka], 1 if ka < kb else upper if ka == kb else 0
                h[:, ki, kj, ka] = 0.5 * np.einsum('rijae,be->rijab', x, d[kb, o:, o:]) \
                    - np.einsum('rimab,mj->rijab', w * x, d[kj, :o, :o])
    ref = np.stack([2 * synth._antisym_blocks(a, nk, mesh) for a in h])
    y = {}
    c = lr.Context(0)
    if mesh is not None:
        c.set_kmesh(*mesh)
    for name, f in (("plain", fock), ("shifted", shifted)):
        c.set_hamiltonian(case['o'], f, case['H']['chol'], case['H']['dip'])
        c.set_amplitudes(case['t1'], case['t2'])
        for prec in (lr.FP64, lr.FP32):
            y[name, prec] = c.apply_sigma(case['x1'], x2, np.zeros(nrhs), prec)[1]
    # the rounding of the two products, sums of some hundred terms
    for prec, tol in ((lr.FP64, 1e-13), (lr.FP32, FP32_REL)):
        e = np.abs(y["shifted", prec] - y["plain", prec] - ref).max() / np.abs(y["shifted", prec]).max() \
            if nk * o > 1 and nk * v > 1 else np.abs(y["shifted", prec]).max()
        a = np.stack([synth._antisym_blocks(b, nk, mesh) / 2 for b in y["shifted", prec]])
        s = np.abs(y["shifted", prec] - a).max() / max(np.abs(a).max(), 1.0)
        print(f"nk={nk} o={o} v={v} nrhs={nrhs} precision {prec}: {e:.1e}, symmetric part {s:.1e}", flush=True)
        assert e < tol and s < 1e-15 * 8
    c.close()


@pytest.mark.parametrize("nk,o,v,nrhs", [(1, 3, 31, 2), (1, 3, 33, 2), (1, 2, 65, 1), (3, 2, 34, 1)])
def test_products_in_place(nk, o, v, nrhs):
    import torch
    import paper_2508_01266_amd as lr
    case = make_case(nk, o, v, 6, nrhs, 41 + v, noncanonical=0.3)
    c = lr.Context(0)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_amplitudes(case['t1'], case['t2'])
    dev = torch.device("cuda:0")
    om = torch.from_numpy(case['omega']).to(dev)
    for prec in (lr.FP64, lr.FP32):
        for adjoint in (False, True):
            x1, x2 = torch.from_numpy(case['x1']).to(dev), torch.from_numpy(case['x2']).to(dev)
            y1, y2 = torch.empty_like(x1), torch.empty_like(x2)
            c.apply_sigma_dev(x1, x2, y1, y2, om, prec, adjoint=adjoint)
            c.apply_sigma_dev(x1, x2, x1, x2, om, prec, adjoint=adjoint)
            torch.cuda.synchronize()
            assert torch.equal(x1, y1) and torch.equal(x2, y2), (prec, adjoint)     # the same operations
    print(f"nk={nk} o={o} v={v} nrhs={nrhs}: in place ok", flush=True)
    c.close()
