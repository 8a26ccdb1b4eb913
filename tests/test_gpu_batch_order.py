"""The inverse's summation order over the filters and the batch: as built it follows the batch (an image alone and in a
batch agree to rounding, 1e-6 relative L2 as between schedules), with kg_inv above 1 it does not (bit for bit)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("N,J,B,pw", [(256, 3, 24, 16), (256, 3, 24, 8), (512, 4, 8, 16), (1024, 2, 4, 8)])
def test_order_with_partial_sums_does_not_follow_the_batch(gpu, N, J, B, pw):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: batch order {N}x{N} J={J} B={B} pw={pw}", flush=True)
    with ShearletSystem.build(N, N, J) as s:
        x = torch.from_numpy(synth.cartoon_batch(B, N, N, config=3, sigma=20.0)).to(gpu)
        c = s.forward(x)
        thr = torch.from_numpy(np.tile(s.paper_thresholds(20.0), (B, 1))).to(gpu)

        def results(b0, b1):
            return s.inverse(c[b0:b1]), s.adjoint(c[b0:b1]), s.denoise(x[b0:b1], thr[b0:b1])

        for kg in (1, 3):
            s.set_schedule(0, pw, 0, kg)
            whole = results(0, B)
            for b in (0, B - 1):
                for one, all_ in zip(results(b, b + 1), whole):
                    torch.cuda.synchronize()
                    assert _rel(one[0], all_[b]) <= 1e-6
                    if kg > 1:
                        assert torch.equal(one[0], all_[b])
