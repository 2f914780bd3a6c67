"""The error bars of S3 and S4 in one launch and in two: they come from sums and
stores of their own (the squares), so equal spectra do not show them equal."""
import numpy as np
import pytest

from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one record in pieces, 600 in whole tiles (of one chunk: no error bar); the blocks
# run the same code on the same work: equal bit for bit, NaN for NaN
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "fp16x2s"])
@pytest.mark.parametrize("Nf,m,n_chunks", [(1, 4, 3), (63, 5, 9), (64, 10, 40), (130, 10, 7), (70, 6, 1)])
@pytest.mark.parametrize("interlaced", [False, True])
def test_error_bars_of_one_launch_and_two(precision, Nf, m, n_chunks, interlaced):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] error bars of S3 and S4", precision, Nf, m, n_chunks, interlaced, flush=True)
    N = 1024
    x = torch.from_numpy(synth.ar2_chi2(N * m * n_chunks + N // 2, seed=Nf).astype(np.float32)).to("cuda:0")
    with Plan(frame_len=N, n_freq=Nf, m=m, precision=precision, interlaced=interlaced) as p:
        runs = []
        for timed in (False, True):     # stage timing keeps two launches
            p.profile(timed)
            alone, many = p.execute(x), p.execute([x] * 600)
            runs.append((alone, many[0], many[599]))
        p.profile(False)
        torch.cuda.synchronize()
        for a, b in zip(*runs):
            for k in ("s2", "s3", "s4", "s2_err", "s3_err", "s4_err"):
                u, v = getattr(a, k), getattr(b, k)
                assert torch.equal(torch.isnan(u), torch.isnan(v)), k
                assert torch.isnan(u).any() == (n_chunks == 1 and k.endswith("_err")), k
                assert torch.equal(torch.nan_to_num(u), torch.nan_to_num(v)), k
