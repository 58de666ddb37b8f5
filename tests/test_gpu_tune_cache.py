"""Cached tuning choices are taken only for a program with as many launches."""
import pytest

from tests.sigma_cases import make_case, oracle_sigma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cut", [-1, -3, 2])
def test_lines_of_another_length_are_not_used(tmp_path, monkeypatch, cut):
    import numpy as np
    import paper_2508_01266_amd as lr
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LRCC_TUNE_CACHE", str(cache))
    case = make_case(1, 3, 9, 8, 5, 44)
    ref = oracle_sigma(case)

    def run():
        c = lr.Context(0)
        c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
        c.set_amplitudes(case['t1'], case['t2'])
        c.set_autotune(True)
        y = c.apply_sigma(case['x1'], case['x2'], case['omega'], lr.FP64)
        c.close()
        assert max(np.abs(a - b).max() / np.abs(b).max() for a, b in zip(y, ref)) < 1e-11
        return [ln.split() for ln in cache.read_text().splitlines()]

    cache.write_text("")
    line = next(ln for ln in run() if "forward" in ln[0])
    other = line[:cut] if cut < 0 else line + ["0"] * cut
    cache.write_text(" ".join(other) + "\n")
    lines = run()
    assert [len(ln) for ln in lines if ln[0] == line[0]] == [len(other), len(line)], "tuned again and appended"
    assert run() == lines, "then found"
    print(f"{len(line) - 1} choices, line of {len(other) - 1}: ok", flush=True)
