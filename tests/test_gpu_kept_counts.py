"""Kept counts of the denoising row kernel at the block shapes of its counting: blocks of less than a
wavefront (16 and 32 columns), one wavefront, and several (up to 512 threads), against the counts taken
from the forward transform's own coefficients, which the fused kernel recomputes bit for bit; and the
images with and without counts are the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,K,B", [(16, 16, 3, 2), (32, 32, 5, 3), (64, 64, 2, 1), (16, 256, 4, 5), (128, 512, 3, 2),
                                     (32, 1024, 2, 3), (64, 2048, 2, 1)])
def test_kept_counts_by_block_shape(gpu, N, M, K, B):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: kept counts {N}x{M} K={K} B={B}", flush=True)
    rng = np.random.default_rng(N + M + K)
    ker = rng.standard_normal((K, N, M))
    ker = ker + ker[:, (-np.arange(N)) % N][:, :, (-np.arange(M)) % M]
    with ShearletSystem.from_spectra(np.fft.fftshift(np.fft.fft2(ker), axes=(1, 2))) as s:
        x = torch.from_numpy(rng.standard_normal((B, N, M)).astype(np.float32)).to(gpu)
        c = s.forward(x).abs()
        thr = c.flatten(2).median(dim=2).values * torch.linspace(0.2, 1.8, K, device=gpu)
        thr[0, 0] = 0.0
        thr[-1, -1] = float("inf")
        want = (c >= thr[:, :, None, None]).sum(dim=(2, 3))
        y, kept = s.denoise(x, thr, kept=True)
        again = s.denoise(x, thr)
        torch.cuda.synchronize()
        assert torch.equal(kept, want)
        assert torch.equal(y, again)
