"""The last network layer with the thresholds as an output: the persistent kernel from 512 tiles of 8 x 64 on where the
low-pass plane is alone in its group of 16 (17, 33, 49 planes), from 1536 with four groups, on 256 CUs; one-tile blocks
below and at the other counts. Both take the same sums in the same order: the same bits for an image in a batch
on either side of the line and alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,sizes", [(17, (15, 16)), (33, (15, 16)), (49, (15, 16)), (48, (16, 48)), (50, (47, 48)), (64, (47, 48))])
def test_tau_bits_across_the_line(gpu, K, sizes):
    from oracle import shrink as OS
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: tau across the line K={K} {sizes}", flush=True)
    N = 128  # 32 tiles an image
    rng = np.random.default_rng(K)
    S = np.fft.fft2(rng.standard_normal((K, N, N)))
    rms = torch.from_numpy(np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))).float().to(gpu)
    gen = torch.Generator(device=gpu)
    gen.manual_seed(K)
    c = torch.randn((sizes[1], K, N, N), generator=gen, device=gpu) * 30.0 * rms[None, :, None, None]
    p = OS.init_params(K, seed=7, tau0=2.0)
    params = {"W1": p.W1, "b1": p.b1 + 0.1, "W2": p.W2, "b2": p.b2 - 0.05, "W3": 10.0 * p.W3, "b3": p.b3}
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, params)
        sigma = torch.linspace(15.0, 40.0, sizes[1], device=gpu)
        res = [net.apply(c[:b], sigma[:b], tau=True) for b in (*sizes, 1)]
        torch.cuda.synchronize()
        for v in range(2):
            assert torch.equal(res[0][v], res[1][v][:sizes[0]])
            assert torch.equal(res[2][v], res[1][v][:1])
        assert float(res[1][1][:, -1].abs().max()) == 0.0 and torch.equal(res[1][0][:, -1], c[:, -1])
        assert 0.0 < float((res[1][0] == 0).float().mean()) < 1.0
