"""The matrix-core ceilings are those of kernels that do nothing but independent
matrix-core steps: within 15% of the published dense FP64 and FP32 peaks (the clock under
load), so no kernel of the library can appear faster than its ceiling."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,peak", [("DFJK_F64", 78.6), ("DFJK_F32", 157.3)])
def test_rate(dtype, peak):
    import paper_2506_06661_amd as pkg
    r = pkg.dfjk_probe_mfma(getattr(pkg, dtype))
    print(f"{dtype}: {r:.1f} TFLOP/s", flush=True)
    assert 0.85 * peak < r < 1.05 * peak
