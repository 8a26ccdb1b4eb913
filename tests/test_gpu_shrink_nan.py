"""Non-finite coefficients of the low-pass plane in the learned shrinkage with the thresholds as an output: shrunk = c
where |z| >= tau, and tau is 0 there, so infinities are kept and a NaN, which is not >= 0, gives 0, for an image
alone (blocks of one tile) and in a batch (the persistent kernel), and whether the low-pass plane shares a group of
16 planes or is alone in its group. An image whose noise level is NaN keeps nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [2, 16, 17, 18, 33, 49, 64])
def test_low_pass_nan_does_not_depend_on_the_batch(gpu, K):
    from oracle import shrink as OS
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: low-pass NaN K={K}", flush=True)
    N, B = 128, 16  # 512 tiles: the persistent kernel at 17, 33 and 49 planes (two tiles per CU, 256 CUs)
    rng = np.random.default_rng(K)
    S = np.fft.fft2(rng.standard_normal((K, N, N)))
    rms = np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))
    c = (rng.standard_normal((B, K, N, N)) * 30.0 * rms[None, :, None, None]).astype(np.float32)
    c[:, -1, 5, 7] = np.nan
    c[:, -1, 64, 100] = np.inf
    c[:, -1, 127, 127] = -np.inf
    want = np.where(np.isnan(c[:, -1]), np.float32(0.0), c[:, -1])
    want[-1] = 0.0
    p = OS.init_params(K, seed=7, tau0=2.0)
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {n: getattr(p, n) for n in ShrinkNet.NAMES})
        ct = torch.from_numpy(c).to(gpu)
        sigma = torch.full((B,), 20.0, device=gpu)
        sigma[-1] = float("nan")
        out, tau = net.apply(ct, sigma, tau=True)
        for b in (0, B - 1):
            one, tau1 = net.apply(ct[b:b + 1].contiguous(), sigma[b:b + 1].contiguous(), tau=True)
            torch.cuda.synchronize()
            assert np.array_equal(one[0, -1].cpu().numpy(), want[b]), "image alone"
            assert np.array_equal(out[b, -1].cpu().numpy(), want[b]), "in a batch"
            assert float(tau1[:, -1].abs().max()) == 0.0
        assert float(tau[:, -1].abs().max()) == 0.0
