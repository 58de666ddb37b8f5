"""The fp64 matrix cores run at half the fp32 rate, and so do the library's measured peaks."""
import pytest

pytestmark = pytest.mark.gpu


def test_measured_fp64_rate_is_half_of_fp32():
    import paper_2508_01266_amd as lr
    p = lr.measure_peaks(0)
    ratio = p["mfma_f64_tflops"] / p["mfma_f32_tflops"]
    print(f"measured: {p}, ratio {ratio:.3f}", flush=True)
    assert 0.45 < ratio < 0.55           # 78.6 / 157.3, and the clock of two streams of some milliseconds
