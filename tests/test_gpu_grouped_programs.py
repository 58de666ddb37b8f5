"""Small recorded programs run grouped, op by op and grouped again on the same buffers; rounding of long complex64
reductions."""
import pytest

from tests.grouped_cases import run

pytestmark = pytest.mark.gpu


def test_grouped_after_op_by_op(tmp_path):
    rc, out = run(tmp_path, "partial", "run")
    print(out, flush=True)
    assert rc == 0 and out.count("ok") == 4, out


def test_rounding_of_long_complex64_reductions(tmp_path):
    """One product on the bf16 tiles in one piece.  A sum of n = K / 32 steps is rounded once a step, each time by
    0.42 2^-24 of it (root mean square over the mantissas), and the sums of a random reduction grow like a random
    walk: 0.42 2^-24 sqrt(n / 2) of the result in all; with the rounding of a step's own sum, and a margin,
    2^-24 (0.5 sqrt(n / 2) + 1.5)."""
    rc, out = run(tmp_path, "reduction", "run")
    print(out, flush=True)
    assert rc == 0, out
    lines = [ln.split() for ln in out.splitlines() if ln[:1].isdigit()]
    assert len(lines) == 5
    for k, fp32, bf16 in ((int(a), float(b), float(c)) for a, b, c in lines):
        assert bf16 < 2.0 ** -24 * (0.5 * (k / 64) ** 0.5 + 1.5), (k, bf16)
        # 128 elements, 32 instructions a sum, 32 roundings of the 128 in a second sum
        assert fp32 < 2.0 ** -24 * (0.5 * (k / 256) ** 0.5 + 6), (k, fp32)
