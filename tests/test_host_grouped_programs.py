"""Layout of the grouped form of small recorded programs (dry run, no device)."""
import pytest

from tests.grouped_cases import run


def test_array_stored_in_part_is_not_the_tensors_buffer(tmp_path):
    """The op-by-op form leaves the whole sum in the tensor's buffer, which a grouped run of the same program
    would add again wherever the array there is not stored."""
    rc, out = run(tmp_path, "partial")
    assert rc == 0 and "arrays 3" in out, out


def test_sum_of_constant_arrays_is_formed(tmp_path):
    """A tensor of copies of arrays that no op writes, read as an operand."""
    rc, out = run(tmp_path, "constants")
    assert rc == 0, out


def test_tensor_that_is_only_cleared(tmp_path):
    """A tensor with a clear and no other writer, read by other programs."""
    rc, out = run(tmp_path, "cleared")
    assert rc == 0, out


@pytest.mark.parametrize("nk,o,v,naux,nrhs", [(1, 1, 1, 1, 1), (1, 3, 5, 4, 2), (3, 5, 7, 9, 2)])
def test_tensors_fit_their_arrays(nk, o, v, naux, nrhs):
    """The dry run compares the extent that each op of a grouped program declares with the array it stores to
    (the real diagonals of the preconditioner are half as large as complex ones)."""
    from paper_2508_01266_amd import plan_check
    plan_check(nk, o, v, naux, nrhs)


def test_extra_arrays_leave_free_memory(tmp_path):
    rc, out = run(tmp_path, "budget")
    assert rc == 0, out


@pytest.mark.parametrize("nk,o,v,naux,nrhs", [(1, 4, 12, 48, 9), (3, 4, 20, 72, 12), ((2, 2, 2), 1, 3, 4, 2)])
def test_recorded_programs_run_grouped(monkeypatch, capfd, nk, o, v, naux, nrhs):
    """The programs of the plan check: the blocks of the amplitudes, products and transposes in both precisions, lean
    and perturbation forms."""
    from paper_2508_01266_amd import plan_check
    monkeypatch.setenv("LRCC_PLAN_DUMP", "1")
    plan_check(nk, o, v, naux, nrhs)
    forms = [ln for ln in capfd.readouterr().err.splitlines() if ln.startswith("grouped: ")]
    assert len(forms) == 20, forms
