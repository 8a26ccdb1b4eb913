"""The autotuner reports panels of 8 columns at 1024 and 2048 points, where 16 selects no kernel of its own."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1024, 2048])
def test_autotuner_reports_the_panels_that_run(gpu, N):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: autotuned panels at {N} rows", flush=True)
    rng = np.random.default_rng(N)
    S = np.fft.fftshift(np.fft.fft2(rng.standard_normal((3, N, 64))), axes=(1, 2))
    with ShearletSystem.from_spectra(S) as s:
        assert s.autotune(2)[:2] == (8, 8)
