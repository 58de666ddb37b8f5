"""Small recorded programs run grouped, op by op and grouped again on the same buffers."""
import pytest

from tests.grouped_cases import run

pytestmark = pytest.mark.gpu


def test_grouped_after_op_by_op(tmp_path):
    rc, out = run(tmp_path, "partial", "run")
    print(out, flush=True)
    assert rc == 0 and out.count("ok") == 4, out
