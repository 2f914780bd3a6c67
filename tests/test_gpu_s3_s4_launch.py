"""S3 and the single-channel S4 in one launch: the numbers of the two separate
launches, which stage timing keeps."""
import numpy as np
import pytest

from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# Every precision, grids of one partial tile, one tile and several, frame counts
# at both ends of the small batch and one that keeps the two launches (m = 11);
# one record in pieces and 600 in whole tiles, per chunk and interlaced.  The
# blocks run the same code on the same work: equal bit for bit.
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "fp16x2s"])
@pytest.mark.parametrize("Nf,m,n_chunks", [(1, 4, 3), (63, 5, 9), (64, 10, 40), (130, 10, 7), (200, 11, 5)])
@pytest.mark.parametrize("interlaced", [False, True])
def test_one_launch_and_two(precision, Nf, m, n_chunks, interlaced):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] S3 and S4 launches", precision, Nf, m, n_chunks, interlaced, flush=True)
    if precision == "fp16x2s" and m > 10:
        pytest.skip("scaled FP16 x 2 takes at most ten frames")
    N = 1024
    x = torch.from_numpy(synth.ar2_chi2(N * m * n_chunks, seed=Nf).astype(np.float32)).to("cuda:0")
    with Plan(frame_len=N, n_freq=Nf, m=m, precision=precision, interlaced=interlaced) as p:
        runs = []
        for timed in (False, True):
            p.profile(timed)
            alone, many, seq = p.execute(x), p.execute([x] * 600), p.sequential(x)
            runs.append((alone, many[0], many[599], seq))
        p.profile(False)
        torch.cuda.synchronize()
        for a, b in zip(*runs):
            for k in ("s2", "s3", "s4"):
                assert torch.isfinite(getattr(a, k)).all(), k
                assert torch.equal(getattr(a, k), getattr(b, k)), k
