"""complex64 products formed from bf16 products of split operands (128x64 tiles, 32-deep steps): forced for
every product that can take them, on sizes with ragged rows, columns and reductions (inside one step, one
element past a step, triangle splits, runs that are not multiples of eight), against the oracle; and no
further from it than the products on the fp32 matrix cores."""
import numpy as np
import pytest

import synth
from tests.sigma_cases import FP32_REL, make_case, oracle_sigma, oracle_sigma_adjoint

pytestmark = pytest.mark.gpu

SIZES = [(1, 4, 8, 33, 8, 90), (1, 5, 17, 32, 5, 91), (2, 3, 11, 24, 15, 92), (3, 2, 6, 31, 33, 93)]


def _norm(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("nk,o,v,naux,nrhs,seed", SIZES)
def test_split_products_match_oracle(tmp_path, monkeypatch, nk, o, v, naux, nrhs, seed):
    import paper_2508_01266_amd as lr
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LRCC_TUNE_CACHE", str(cache))
    case = make_case(nk, o, v, naux, nrhs, seed)
    rng = synth.rng_for(7300 + seed, nk, o, v)
    z1, z2 = synth.random_vectors(nrhs, nk, o, v, rng, 0.1, 0.1)
    z2 = z2 * nk
    ref = oracle_sigma(case) + oracle_sigma_adjoint(case, z1, z2)

    def run():
        c = lr.Context(0)
        c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
        c.set_amplitudes(case['t1'], case['t2'])
        c.set_autotune(True)
        out = c.apply_sigma(case['x1'], case['x2'], case['omega'], lr.FP32) + \
            c.apply_sigma_adjoint(z1, z2, case['omega'], lr.FP32)
        c.close()
        return out

    cache.write_text("")
    run()
    lines = [ln.split() for ln in cache.read_text().splitlines() if "f32" in ln]
    assert len(lines) == 2
    err = {}
    # the candidates of a product start with the default one: index 1 is the bf16 tile where the default is
    # another, index 0 where it is the bf16 tile (the last entry, 1, runs the program op by op)
    for name, index in (("default", 0), ("other", 1)):
        cache.write_text("".join(" ".join([ln[0]] + [str(index)] * (len(ln) - 2) + ["1"]) + "\n" for ln in lines))
        y = run()
        assert max(np.abs(a - b).max() / np.abs(b).max() for a, b in zip(y, ref)) < FP32_REL
        err[name] = [_norm(a, b) for a, b in zip(y, ref)]
    print(f"nk={nk} o={o} v={v} nrhs={nrhs}: default tiles {err['default']}, others {err['other']}", flush=True)
    # both carry the rounding of the complex64 inputs and sums, 2^-24 per operation
    assert max(err["default"] + err["other"]) < 1e-6
