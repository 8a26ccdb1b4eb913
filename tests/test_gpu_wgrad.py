"""The weight-gradient kernels of the shrinkage network at the edges of their tiling, through
shear_shrink_train_step against the oracle's analytic gradients: images of a few rows (units of 8
rows, fewer units than blocks, rows that wrap), one to four groups of 16 output channels, odd batches,
and a batch large enough for units of more than 8 rows. The bars are the training step's (rounding
flips of the bfloat16 operands, not the sums, set them): 3e-3 relative L2 per tensor, the loss 1e-3."""
import numpy as np
import pytest

from oracle import shrink as OS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("K,N,M,B", [(16, 16, 128, 1), (5, 32, 128, 3), (33, 16, 256, 3), (48, 64, 128, 5), (17, 128, 256, 9),
                                     (64, 16, 128, 2)])
def test_weight_gradients_at_tile_edges(gpu, K, N, M, B):
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: weight gradients {N}x{M} K={K} B={B}", flush=True)
    rng = np.random.default_rng(1000 + K * 7 + N + B)
    S = np.fft.fft2(rng.standard_normal((K, N, M)))
    rms = np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))
    sig = rng.uniform(10.0, 40.0, B)
    cc = (rng.standard_normal((B, K, N, M)) * 20.0 * rms[None, :, None, None]).astype(np.float32)
    cn = (cc + rng.standard_normal(cc.shape) * sig[:, None, None, None] * rms[None, :, None, None]).astype(np.float32)
    p = OS.init_params(K, seed=60 + K, tau0=2.5)
    p = OS.ShrinkParams(p.W1, p.b1 + 0.05 * rng.standard_normal(32), p.W2, p.b2 + 0.05 * rng.standard_normal(32),
                        p.W3 * 10.0, p.b3)
    T = 0.5
    scale = 1.0 / (B * (K - 1) * N * M)
    L, want = 0.0, {n: 0.0 for n in ShrinkNet.NAMES}
    for b in range(B):
        Lb, gb = OS.train_loss(cn[b], cc[b], sig[b], rms, p, T, scale, rounded=True)
        L += Lb
        for n in want:
            want[n] = want[n] + gb[n]
    to = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(gpu)  # noqa: E731
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {n: getattr(p, n) for n in ShrinkNet.NAMES})
        loss = net.train_step(to(cn), to(cc), to(sig), lr=0.0, temperature=T)
        first = net.grads.clone()
        again = net.train_step(to(cn), to(cc), to(sig), lr=0.0, temperature=T)
        torch.cuda.synchronize()
        assert torch.equal(first, net.grads)  # the sums are taken in a fixed order
        assert abs(float(loss) - L) <= 1e-3 * L and abs(float(again) - L) <= 1e-3 * L
        for n in want:
            e = _rel(net.grad(n).cpu().numpy(), want[n])
            print(f"grad {n}: rel L2 {e:.2e}")
            assert e <= 3e-3, n
