"""Which programs run grouped, and through which launches: the plan dump of the products on the device, and the grouped
form against the same program op by op where it uses the bf16 tiles, launches of their own and arrays cleared in
every run (doubles of more than 64 MB)."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import FP32_REL, make_case
from tests.test_gpu_grouped import SIZES

pytestmark = pytest.mark.gpu


def _context(lr, case, mesh=None, mode=0):
    c = lr.Context(0)
    if mesh is not None:
        c.set_kmesh(*mesh)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_ladder_mode(mode)
    c.set_amplitudes(case['t1'], case['t2'])
    return c


def _grouped(text):
    """Launch names of the grouped forms in a plan dump, one list each."""
    out = []
    for ln in text.splitlines():
        if ln.startswith("grouped: "):
            out.append([])
        elif ln.startswith("  ") and out:
            out[-1].append(ln.strip())
    return out


@pytest.mark.parametrize("nk,o,v,naux,nrhs,mesh", SIZES)
def test_products_run_grouped(monkeypatch, capfd, nk, o, v, naux, nrhs, mesh):
    import paper_2508_01266_amd as lr
    monkeypatch.setenv("LRCC_PLAN_DUMP", "1")
    case = make_case(nk, o, v, naux, nrhs, 70 + v, mesh=mesh)
    c = _context(lr, case, mesh)
    assert len(_grouped(capfd.readouterr().err)) == 1            # the amplitude-dependent blocks
    for prec in (lr.FP64, lr.FP32):
        for fn in (c.apply_sigma, c.apply_sigma_adjoint):
            fn(case['x1'], case['x2'], case['omega'], prec)
            forms = _grouped(capfd.readouterr().err)
            if nk * o == 1 or nk * v == 1:     # no unique pair: arrays that are cleared and never written
                assert len(forms) <= 1
                continue
            assert len(forms) == 1 and forms[0][-1] == "output", (prec, fn.__name__)
    c.close()


# complex64: some hundred bf16 tiles a level; complex128: doubles of 116 MB (adjoint: parts of arrays cleared in
# every run) and products that fill the device alone
@pytest.mark.parametrize("nk,o,v,naux,nrhs,kinds", [(2, 8, 33, 20, 13, ("bf16 tiles", "clear", "gemm"))])
def test_grouped_form_matches_op_by_op(tmp_path, monkeypatch, capfd, nk, o, v, naux, nrhs, kinds):
    import paper_2508_01266_amd as lr
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LRCC_TUNE_CACHE", str(cache))
    monkeypatch.setenv("LRCC_PLAN_DUMP", "1")
    case = make_case(nk, o, v, naux, nrhs, 46)
    rng = synth.rng_for(9900, nk, o, v)
    z1, z2 = synth.random_vectors(nrhs, nk, o, v, rng, 0.1, 0.1)
    args = ((case['x1'], case['x2']), (z1, z2 * nk))

    def products(c):
        return [y for prec in (lr.FP64, lr.FP32) for fn, x in zip((c.apply_sigma, c.apply_sigma_adjoint), args)
                for y in fn(*x, case['omega'], prec)]

    cache.write_text("")
    c = _context(lr, case, mode=2)
    c.set_autotune(True)
    products(c)
    c.close()
    names = [n for form in _grouped(capfd.readouterr().err) for n in form]
    print(sorted({" ".join(n.split()[-2:]) if n.startswith("level") else n.split()[0] for n in names}), flush=True)
    for k in kinds:
        assert any(k in n for n in names), k
    lines = [ln.split() for ln in cache.read_text().splitlines()]
    assert len(lines) == 4
    out = []
    for form in ("0", "1"):                       # the default launches, grouped and op by op
        text = "".join(" ".join([ln[0]] + ["0"] * (len(ln) - 2) + [form]) + "\n" for ln in lines)
        cache.write_text(text)
        c = _context(lr, case, mode=2)
        c.set_autotune(True)
        out.append(products(c))
        c.close()
        assert cache.read_text() == text
    for q, (a, b) in enumerate(zip(*out)):
        e = np.abs(a - b).max() / np.abs(b).max()
        print(f"output {q}: {e:.1e}", flush=True)
        assert e < (1e-12 if q < 4 else FP32_REL)
