"""Matrix-core flops of the complex64 ladder against the tiles that its products run on: six bf16 products per real
one on the bf16 tiles, one on the others, grouped and op by op."""
import pytest

from tests.sigma_cases import make_case

pytestmark = pytest.mark.gpu


# unique rows, outputs and reductions: 180 x 66 x 66 (4 bf16 tiles: fp32 tiles in a grouped launch) and
# 1344 x 1770 x 1770 (308, which fill the device: bf16)
@pytest.mark.parametrize("o,v,naux,nrhs,factor", [(4, 12, 20, 30, 1), (8, 60, 20, 48, 6)])
def test_grouped_ladder_counts_its_tiles(o, v, naux, nrhs, factor):
    import paper_2508_01266_amd as lr
    case = make_case(1, o, v, naux, nrhs, 45)
    c = lr.Context(0)
    c.set_hamiltonian(case['o'], case['H']['fock'], case['H']['chol'], case['H']['dip'])
    c.set_ladder_mode(2)
    c.set_amplitudes(case['t1'], case['t2'])
    ratio = c.ladder_mfma_flops(nrhs, lr.FP32) / c.ladder_flops(nrhs, lr.FP32)
    print(f"o={o} v={v} nrhs={nrhs}: {ratio}", flush=True)
    assert ratio == factor
    assert c.ladder_mfma_flops(nrhs, lr.FP64) == c.ladder_flops(nrhs, lr.FP64)
    c.close()
