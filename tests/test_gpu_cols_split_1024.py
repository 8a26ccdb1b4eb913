"""The splits of the inverse column pass at 1024 points: 1, 2 and 4 columns per block (8, 4 and 2 groups of filters)
follow from the call's columns on a device of 256 compute units, here 256, 512 and 2048; inverse and adjoint
against the FP64 oracle (relative L2 <= 1e-5), real and complex banks, and with the workspace cut into chunks
bit for bit."""
import numpy as np
import pytest

from oracle import transform as OT

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("B", [1, 2, 8])
@pytest.mark.parametrize("real", [True, False])
def test_split_inverse_1024_against_oracle(gpu, B, real):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: split inverse 1024x512 K=3 real={real} B={B}", flush=True)
    N, M, K = 1024, 512, 3
    rng = np.random.default_rng(B + 10 * real)
    ker = rng.standard_normal((K, N, M))
    if real:
        ker = ker + ker[:, (-np.arange(N)) % N][:, :, (-np.arange(M)) % M]
    S = np.fft.fft2(ker)
    W = np.sum(np.abs(S) ** 2, 0)
    Sc = np.fft.fftshift(S, axes=(1, 2))
    ch = rng.standard_normal((B, K, N, M)).astype(np.float32)
    c = torch.from_numpy(ch).to(gpu)
    plane = N * (M // 2) * 8
    with ShearletSystem.from_spectra(Sc) as s, \
            ShearletSystem.from_spectra(Sc, max_workspace_bytes=(B + 2 * K) * plane + 16) as small:
        y, a, yc = s.inverse(c), s.adjoint(c), small.inverse(c)
        torch.cuda.synchronize()
        assert torch.equal(y, yc)
        for b in sorted({0, B // 2, B - 1}):
            c64 = ch[b].astype(np.float64)
            assert _rel(y[b].cpu().numpy(), OT.inverse_plain(c64, S, W)) <= TOL, b
            assert _rel(a[b].cpu().numpy(), OT.adjoint_plain(c64, S)) <= TOL, b
