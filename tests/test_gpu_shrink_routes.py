"""The shrink layer without thresholds: one-tile blocks up to 16 planes and, with two or four groups of 16 planes, below
512 or 256 tiles of 8 x 64 (256 CUs), the persistent kernel elsewhere. Both take the same sums and decisions: an
image alone and in batches on either side of the line gives the same bits; the low-pass plane is kept whole, a NaN
included."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 16, 17, 18, 32, 33, 34, 49, 50, 64])
def test_shrunk_bits_across_the_line(gpu, K):
    from oracle import shrink as OS
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: shrink routes K={K}", flush=True)
    N = 128  # 32 tiles an image: 7 and 8 images are below and at 256 tiles, 15 and 16 at 512
    rng = np.random.default_rng(K)
    S = np.fft.fft2(rng.standard_normal((K, N, N)))
    rms = torch.from_numpy(np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))).float().to(gpu)
    gen = torch.Generator(device=gpu)
    gen.manual_seed(K)
    c = torch.randn((16, K, N, N), generator=gen, device=gpu) * 30.0 * rms[None, :, None, None]
    c[0, -1, 3, 5] = float("nan")
    p = OS.init_params(K, seed=7, tau0=2.0)
    params = {"W1": p.W1, "b1": p.b1 + 0.1, "W2": p.W2, "b2": p.b2 - 0.05, "W3": 10.0 * p.W3, "b3": p.b3}
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, params)
        sigma = torch.linspace(15.0, 40.0, 16, device=gpu)
        res = {b: net.apply(c[:b], sigma[:b]) for b in (1, 7, 8, 15, 16)}
        torch.cuda.synchronize()
        bits = res[16].view(torch.int32)
        for b in (1, 7, 8, 15):
            assert torch.equal(res[b].view(torch.int32), bits[:b]), b
        assert torch.equal(bits[:, -1], c[:, -1].view(torch.int32))
        if K > 1:
            assert 0.0 < float((res[16][:, :-1] == 0).float().mean()) < 1.0
