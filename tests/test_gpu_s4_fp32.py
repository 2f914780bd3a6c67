"""The FP32 S4 kernels (frame sums on the FP32 matrix cores) at the edges of
their tiles and frame batches, against the FP64 oracle.

Tolerance: a frame sum of m <= 24 terms carries at most (m + 2) 2^-24 = 1.6e-6
of the sum of its terms' magnitudes and the coefficients 1.4e-7 each; the
combination adds nothing in FP64.  1e-5 of the spectrum's maximum, the bar of
the parity tests, bounds both with room for the estimator's cancellation."""
import numpy as np
import pytest

import oracle as O
from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5


# grids around the 64-point tile (one channel) and the 32-point tile (channel
# pairs), chunks around the 10-frame batch and odd frame counts
@pytest.mark.parametrize("C,Nf,m", [(1, 1, 4), (1, 63, 5), (1, 64, 10), (1, 65, 11), (1, 128, 9), (1, 100, 20),
                                    (1, 40, 23), (2, 1, 4), (2, 31, 5), (2, 33, 10), (2, 64, 11), (2, 47, 21)])
def test_fp32_s4_edges(C, Nf, m):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] fp32 s4", C, Nf, m, flush=True)
    N = 256
    if C == 1:
        z = synth.ar2_chi2(N * m * 3 + 11, seed=100 + Nf + m)
    else:
        z = synth.mixed_channels(N * m * 3 + 11, seed=100 + Nf + m, n_channels=C)[0].astype(np.float32)
    with Plan(frame_len=N, n_freq=Nf, m=m, orders=(2, 4), n_channels=C, precision="fp32") as p:
        out = p.execute(torch.from_numpy(z).to("cuda:0"))
        torch.cuda.synchronize()
        ref = O.polyspectra(z, N, Nf, m, window_kind="acg", orders=(2, 4), combos2=p.combos2, combos4=p.combos4)
    got = torch.view_as_complex(out.s4).cpu().numpy()
    err = out.s4_err.cpu().numpy()
    assert np.max(np.abs(got - ref["s4"])) <= TOL * np.max(np.abs(ref["s4"]))
    assert np.max(np.abs(err - ref["s4_err"])) <= TOL * np.max(np.abs(ref["s4_err"]))
