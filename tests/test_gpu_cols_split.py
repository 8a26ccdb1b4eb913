"""The inverse column pass's split of the filters over the thread groups of a block, and the forward's
groups by batch: sizes and batches that take each split (1, 2, 4 and 8 columns per block), fewer filters
than groups, a lone packed column of a block, complex and real banks, against the FP64 oracle (relative L2
<= 1e-5); a workspace cap that forces chunks leaves every bit as it is, as the split follows the batch of
the call."""
import numpy as np
import pytest

from oracle import transform as OT

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _bank(rng, K, N, M, real):
    ker = rng.standard_normal((K, N, M))
    if real:
        ker = ker + ker[:, (-np.arange(N)) % N][:, :, (-np.arange(M)) % M]
    return np.fft.fft2(ker)


@pytest.mark.parametrize("N,M,K,real,B", [(256, 16, 3, False, 1), (256, 64, 9, True, 40), (512, 64, 17, True, 1),
                                          (512, 128, 5, False, 7), (512, 64, 2, True, 70), (128, 64, 17, True, 3),
                                          (128, 128, 4, False, 70), (64, 32, 33, True, 9), (16, 64, 7, True, 5),
                                          (1024, 32, 9, False, 1), (1024, 64, 3, True, 9), (2048, 16, 5, True, 2)])
def test_split_inverse_against_oracle(gpu, N, M, K, real, B):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: split inverse N={N} M={M} K={K} real={real} B={B}", flush=True)
    rng = np.random.default_rng(N + 3 * M + K + B)
    S = _bank(rng, K, N, M, real)
    W = np.sum(np.abs(S) ** 2, 0)
    x = torch.from_numpy(rng.standard_normal((B, N, M)).astype(np.float32)).to(gpu)
    ch = rng.standard_normal((B, K, N, M)).astype(np.float32)
    c = torch.from_numpy(ch).to(gpu)
    Sc = np.fft.fftshift(S, axes=(1, 2))
    with ShearletSystem.from_spectra(Sc) as s:
        fwd = s.forward(x)
        for pw in (16, 8) if M >= 32 else (8,):
            s.set_schedule(0, pw)
            y, a = s.inverse(c), s.adjoint(c)
            again = s.inverse(c)
            torch.cuda.synchronize()
            assert torch.equal(y, again)
            for b in sorted({0, B // 2, B - 1}):
                c64 = ch[b].astype(np.float64)
                assert _rel(y[b].cpu().numpy(), OT.inverse_plain(c64, S, W)) <= TOL, (pw, b)
                assert _rel(a[b].cpu().numpy(), OT.adjoint_plain(c64, S)) <= TOL, (pw, b)
                assert _rel(fwd[b].cpu().numpy(), OT.forward_plain(x[b].double().cpu().numpy(), S)) <= TOL, b
        plane = N * (M // 2) * 8
        last = s.inverse(c)
        with ShearletSystem.from_spectra(Sc, max_workspace_bytes=(B + 2 * K) * plane + 16) as small:
            small.set_schedule(0, 16 if M >= 32 else 8)
            s.set_schedule(0, 16 if M >= 32 else 8)
            whole, chunks, fchunks = s.inverse(c), small.inverse(c), small.forward(x)
            torch.cuda.synchronize()
            assert torch.equal(whole, chunks) and torch.equal(fwd, fchunks)
        assert _rel(last.cpu().numpy(), whole.cpu().numpy()) <= 1e-6
