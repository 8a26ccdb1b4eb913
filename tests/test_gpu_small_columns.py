"""Column passes of 16 to 64 points, whose splits follow the batch by their own rules: batches on both sides of each
line on 256 compute units (forward groups 1, 2 and more; inverse 4, 8 and 16 columns per block), real and complex
banks, 8 packed columns and more, against the FP64 oracle (relative L2 <= 1e-5)."""
import numpy as np
import pytest

from oracle import transform as OT

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _bank(rng, K, N, M, real):
    ker = rng.standard_normal((K, N, M))
    if real:
        ker = ker + ker[:, (-np.arange(N)) % N][:, :, (-np.arange(M)) % M]
    return np.fft.fft2(ker)


@pytest.mark.parametrize("N,M,K,B", [(16, 16, 5, 1), (16, 16, 5, 600), (16, 16, 5, 1100), (16, 16, 5, 2100), (16, 64, 7, 200),
                                     (16, 64, 7, 520), (16, 64, 7, 1030), (32, 32, 9, 3), (32, 32, 9, 515), (32, 32, 9, 1025),
                                     (64, 64, 9, 130), (64, 64, 9, 257), (64, 64, 9, 513), (64, 32, 17, 1)])
@pytest.mark.parametrize("real", [True, False])
def test_small_columns_against_oracle(gpu, N, M, K, B, real):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: small columns {N}x{M} K={K} B={B} real={real}", flush=True)
    rng = np.random.default_rng(N + M + K + B)
    S = _bank(rng, K, N, M, real)
    W = np.sum(np.abs(S) ** 2, 0)
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        x = torch.from_numpy(rng.standard_normal((B, N, M)).astype(np.float32)).to(gpu)
        ct = s.forward(x)
        y, a = s.inverse(ct), s.adjoint(ct)
        torch.cuda.synchronize()
        for b in sorted({0, B // 2, B - 1}):
            c64 = ct[b].double().cpu().numpy()
            assert _rel(c64, OT.forward_plain(x[b].double().cpu().numpy(), S)) <= TOL, b
            assert _rel(y[b].cpu().numpy(), OT.inverse_plain(c64, S, W)) <= TOL, b
            assert _rel(a[b].cpu().numpy(), OT.adjoint_plain(c64, S)) <= TOL, b
