"""Training kernels that walk several tiles per block (the first layer's ring of staged rows with the scales of the
next image, the z it writes, the masked backward data, weight-gradient units of 16 rows to the whole height): a
batch against its parts of few images, where a block has at most one tile and units have 8 rows, the shapes that
the other training tests compare with the oracle. Batches are powers of two, so that the loss scale and with it
every bfloat16 gradient of the batch is the part's times a power of two, exactly: the whole is the mean of
the parts but for the order of FP32 sums of at most 320 additions an accumulator (about 1e-6; bar 2e-5, where one
wrong tile of 2048 is 5e-4 or more), the loss but for the rounding of each part's (bar 1e-6)."""
import numpy as np
import pytest

from oracle import shrink as OS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


# rows, columns, filters, images, images per part. 512 images of 16 x 128: 2048 tiles of the first layer and as many
# of the backward data, 8 to a block of 256, two images each. 128 x 256: units of 16, 32, 64 and 128 rows.
@pytest.mark.parametrize("N,M,K,B,part", [(16, 128, 17, 512, 32), (16, 128, 40, 512, 32), (16, 128, 64, 512, 32),
                                          (128, 256, 5, 16, 4), (128, 256, 33, 32, 4), (128, 256, 5, 64, 4),
                                          (128, 256, 16, 128, 4)])
def test_batch_is_the_mean_of_its_parts(gpu, N, M, K, B, part):
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: training tiles {N}x{M} K={K} B={B} in parts of {part}", flush=True)
    rng = np.random.default_rng(N + K + B)
    S = np.fft.fft2(rng.standard_normal((K, N, M)))
    rms = torch.from_numpy(np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))).float().to(gpu)[None, :, None, None]
    gen = torch.Generator(device=gpu)
    gen.manual_seed(K)
    sig = torch.rand(B, generator=gen, device=gpu) * 30.0 + 10.0
    cc = torch.randn((B, K, N, M), generator=gen, device=gpu) * 20.0 * rms
    cn = cc + torch.randn((B, K, N, M), generator=gen, device=gpu) * sig[:, None, None, None] * rms
    p = OS.init_params(K, seed=60 + K, tau0=2.5)
    p = OS.ShrinkParams(p.W1, p.b1 + 0.05 * rng.standard_normal(32), p.W2, p.b2 + 0.05 * rng.standard_normal(32),
                        p.W3 * 10.0, p.b3)
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {n: getattr(p, n) for n in ShrinkNet.NAMES})
        loss = net.train_step(cn, cc, sig, lr=0.0).double()
        whole = {n: net.grad(n).double().clone() for n in ShrinkNet.NAMES}
        mean = {n: torch.zeros_like(whole[n]) for n in ShrinkNet.NAMES}
        ml = 0.0
        for b in range(0, B, part):
            pl = net.train_step(cn[b:b + part], cc[b:b + part], sig[b:b + part], lr=0.0)
            ml = ml + pl.double() * (part / B)
            for n in ShrinkNet.NAMES:
                mean[n] += net.grad(n).double() * (part / B)
        torch.cuda.synchronize()
        assert abs(float(loss) - float(ml)) <= 1e-6 * float(ml)
        for n in ShrinkNet.NAMES:
            e = _rel(whole[n], mean[n])
            print(f"grad {n}: rel L2 {e:.2e}")
            assert e <= 2e-5, n
