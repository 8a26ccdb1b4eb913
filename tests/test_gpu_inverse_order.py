"""The inverse sums its filters in groups within a block at small batches. The low-pass plane, the last filter, holds
most of an image's energy: a sum that takes it first rounds every later addition at its size. The error of the
grouped sum against the FP64 inverse of the same coefficients may not exceed that of one filter after the other
(which kg_inv = K gives: partial sums of one filter each, added in order) by more than 3 % (root mean square over
at least 65536 pixels, which repeats to well under 1 %)."""
import numpy as np
import pytest

import synth
from oracle import filters as OF
from oracle import transform as OT

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,J,B", [(512, 4, 1), (512, 4, 4), (256, 3, 1), (256, 3, 8)])
def test_grouped_sum_is_as_accurate_as_one_after_the_other(gpu, N, J, B):
    from paper_2006_04591_amd import ShearletSystem

    print(f"case: summation order {N}x{N} J={J} B={B}", flush=True)
    ref = OF.build_system(N, N, J)
    x = torch.from_numpy(synth.cartoon_batch(B, N, N, config=3, sigma=20.0)).to(gpu)
    with ShearletSystem.build(N, N, J) as s:
        c = s.forward(x)
        grouped = s.inverse(c)
        s.set_schedule(0, 0, 0, s.K)
        ordered = s.inverse(c)
        torch.cuda.synchronize()
        c, grouped, ordered = (v.double().cpu().numpy() for v in (c, grouped, ordered))
    want = np.stack([OT.inverse_plain(c[b], ref.spectra, ref.W) for b in range(B)])
    eg, eo = (float(np.linalg.norm(v - want) / np.linalg.norm(want)) for v in (grouped, ordered))
    print(f"grouped {eg:.3e}, one after the other {eo:.3e}")
    assert eg <= 1.03 * eo
