"""The last network layer with the thresholds as an output has two routes: blocks of one tile for few tiles, the
persistent kernel for many. Both take the same sums in the same order, so an image alone (32 tiles) and in a
batch of 12 (384 tiles: from half a tile per CU on, 256 CUs) gives the same bits. Plane counts around the
groups of 16 channels: the low-pass plane inside its group, alone (copied) and last of four."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [2, 16, 17, 18, 32, 33, 48, 49, 50, 64])
def test_tau_routes_agree_bitwise(gpu, K):
    from oracle import shrink as OS
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: tau routes K={K}", flush=True)
    N, B = 128, 12
    rng = np.random.default_rng(K)
    S = np.fft.fft2(rng.standard_normal((K, N, N)))
    rms = np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))
    c = (rng.standard_normal((B, K, N, N)) * 30.0 * rms[None, :, None, None]).astype(np.float32)
    p = OS.init_params(K, seed=7, tau0=2.0)
    params = {"W1": p.W1, "b1": p.b1 + 0.1, "W2": p.W2, "b2": p.b2 - 0.05, "W3": 10.0 * p.W3, "b3": p.b3}
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {k: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(gpu) for k, v in params.items()})
        ct = torch.from_numpy(c).to(gpu)
        sigma = torch.linspace(15.0, 40.0, B, device=gpu)
        out, tau = net.apply(ct, sigma, tau=True)
        for b in (0, 5, B - 1):
            one, tau1 = net.apply(ct[b:b + 1].contiguous(), sigma[b:b + 1].contiguous(), tau=True)
            torch.cuda.synchronize()
            assert torch.equal(one[0], out[b]) and torch.equal(tau1[0], tau[b])
        assert float(tau[:, -1].abs().max()) == 0.0 and torch.equal(out[:, -1], ct[:, -1])
        assert 0.0 < float((out == 0).float().mean()) < 1.0
