"""The two forms of the two-stage direct transform at the edges of their rule
and of their blocks, against the FP64 FFT.

Tolerance: the windowed samples and the first stage's sums are rounded to FP32
(2^-24 each), the result as well, everything else is FP64: three roundings of
6e-8, 2e-7 of the largest coefficient."""
import numpy as np
import pytest

import oracle as O
from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# rows in a block (frames x N1): 15 x 4 and 16 x 2 frames, one frame of 64 and of
# 90 rows, 24 rows (8 x 127 in three frames), 17 rows (17 x 307, one frame), and
# the other form's 8 (8 x 251), 11 (11 x 727) and 13 (13 x 331); frame counts
# around the frames of a block
@pytest.mark.parametrize("N", [285, 272, 300, 6144, 8190, 1016, 5219, 2008, 7997, 4303])
@pytest.mark.parametrize("n_frames", [1, 4, 9])
def test_two_stage_transform(N, n_frames):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] two-stage transform", N, n_frames, flush=True)
    z = synth.ar2_chi2(N * n_frames, seed=N + n_frames).astype(np.float32)
    with Plan(frame_len=N, n_freq=N // 4 + 1, m=1 if n_frames == 1 else n_frames, orders=(1,)) as p:
        got = p.coefficients(torch.from_numpy(z).to("cuda:0"))
        torch.cuda.synchronize()
        got, K = got.cpu().numpy()[0], p.n_coef
    frames = z.reshape(n_frames, N).astype(np.float64) * O.window("acg", N)
    ref = (N * np.fft.ifft(frames, axis=-1))[:, :K]
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) <= 2e-7 * np.max(np.abs(ref))
