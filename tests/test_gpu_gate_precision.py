"""Relative precision of the training loss's gate at small thresholds: with W3 = 0 the network's output is its bias, so
every band has the threshold tau = softplus(o) exactly, and a temperature of tau / 4 puts the gate's slope there.
The loss follows from |z| - tau: an error of tau relative to tau changes it by a few times as much. Bars: softplus from
the hardware's exponential and logarithm within 2e-6 gives a loss within 5e-5 relative; log(1 + u) without the
correction for the rounding of 1 + u is off by 6e-8 / (2 tau) (7e-4 at o = -10; all of tau at o = -17.5). The
gradient of b3 is a sum of gradients rounded to bfloat16 on both sides: 3e-3, as in the other training tests."""
import numpy as np
import pytest

from oracle import shrink as OS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o", [-17.5, -10.0, -6.0, 2.0])
def test_small_thresholds_keep_their_precision(gpu, o):
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: gate precision o={o}", flush=True)
    K, N, M, B = 4, 16, 128, 2
    rng = np.random.default_rng(77)
    S = np.fft.fft2(rng.standard_normal((K, N, M)))
    rms = np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))
    tau = float(OS.softplus(o))
    sig = np.array([1.0, 3.0])
    z = rng.uniform(0.0, 3.0, (B, K, N, M)) * rng.choice([-1.0, 1.0], (B, K, N, M)) * tau
    cn = (z * (sig[:, None] * rms[None])[:, :, None, None]).astype(np.float32)
    cc = (0.5 * cn * rng.uniform(0.0, 2.0, cn.shape)).astype(np.float32)
    p = OS.init_params(K, seed=5)
    p = OS.ShrinkParams(p.W1, p.b1, p.W2, p.b2, 0.0 * p.W3, np.full(K, o))
    T = float(np.float32(tau / 4.0))
    scale = 1.0 / (B * (K - 1) * N * M)
    L, db3 = 0.0, np.zeros(K)
    for b in range(B):
        Lb, g = OS.train_loss(cn[b], cc[b], sig[b], rms, p, T, scale, rounded=True)
        L += Lb
        db3 += g["b3"]
    to = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(gpu)  # noqa: E731
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {n: getattr(p, n) for n in ShrinkNet.NAMES})
        loss = float(net.train_step(to(cn), to(cc), to(sig), lr=0.0, temperature=T))
        torch.cuda.synchronize()
        got = net.grad("b3").cpu().numpy().astype(np.float64)
    eg = float(np.linalg.norm(got - db3) / np.linalg.norm(db3))
    print(f"loss rel {abs(loss - L) / L:.2e}, grad b3 rel L2 {eg:.2e}")
    assert abs(loss - L) <= 5e-5 * L
    assert eg <= 3e-3


@pytest.mark.parametrize("b3,T,zscale,nan", [(200.0, 0.5, 1.0, False), (-200.0, 0.5, 1.0, False), (1.0, 1e-38, 20.0, False),
                                             (1.0, 3e38, 1.0, False), (float("nan"), 0.5, 1.0, True),
                                             (1.0, 0.5, float("nan"), True)])
def test_gate_at_the_ends_of_its_range(gpu, b3, T, zscale, nan):
    """Outputs whose exponential underflows, temperatures whose quotient overflows or vanishes, and NaN, which the
    loss keeps. At 1e-38 the gate is a step (|z| far from tau), at 3e38 it is 1/2 everywhere, with outputs of
    200 it is closed and with -200 half open at z = 0 only: the loss from FP64 within 5e-5 in each case."""
    from paper_2006_04591_amd import ShearletSystem, ShrinkNet

    print(f"case: gate range b3={b3} T={T} zscale={zscale}", flush=True)
    K, N, M = 3, 16, 128
    rng = np.random.default_rng(7)
    S = np.fft.fft2(rng.standard_normal((K, N, M)))
    rms = np.sqrt(np.mean(np.abs(S) ** 2, axis=(1, 2)))
    z = rng.choice([-1.0, 1.0], (1, K, N, M)) * rng.uniform(2.0, 4.0, (1, K, N, M)) * zscale
    cn = (z * rms[None, :, None, None]).astype(np.float32)
    cc = np.nan_to_num(0.5 * cn, nan=1.0).astype(np.float32)
    p = OS.init_params(K, seed=5)
    p = OS.ShrinkParams(p.W1, p.b1, p.W2, p.b2, 0.0 * p.W3, np.full(K, b3))
    to = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(gpu)  # noqa: E731
    with ShearletSystem.from_spectra(np.fft.fftshift(S, axes=(1, 2))) as s:
        net = ShrinkNet(s, {n: getattr(p, n) for n in ShrinkNet.NAMES})
        loss = float(net.train_step(to(cn), to(cc), torch.ones(1, device=gpu), lr=0.0, temperature=T))
        torch.cuda.synchronize()
        gb3 = net.grad("b3")
    if nan:
        assert np.isnan(loss)
        return
    sc = (1.0 / rms)[None, :, None, None]
    z64, zc64, tau = cn * sc, cc * sc, OS.softplus(b3)
    x = np.clip((np.abs(z64) - tau) / T, -1e4, 1e4)
    want = float(np.mean(((z64 / (1.0 + np.exp(np.clip(-x, -700, 700))) - zc64) ** 2)[:, :-1]))
    assert abs(loss - want) <= 5e-5 * want
    assert bool(torch.isfinite(gb3).all())
