"""The finalize in one launch and, from 32768 blocks of an order on, in one
launch per order: the same numbers either way."""
import numpy as np
import pytest

from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 2048 chunks of one tile are 32768 blocks of S3 (and of S4): the first count
# below and at the limit; a chunk's estimate does not depend on its neighbours,
# so pieces of 300 chunks (one launch) have to agree bit for bit
@pytest.mark.parametrize("n_chunks", [2047, 2048, 2100])
@pytest.mark.parametrize("orders", [(1, 2, 3, 4), (3,)])
def test_sequential_across_the_launch_limit(n_chunks, orders):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] finalize launches", n_chunks, orders, flush=True)
    N, m = 256, 4
    x = torch.from_numpy(synth.ar2_chi2(N * m * n_chunks, seed=n_chunks).astype(np.float32)).to("cuda:0")
    with Plan(frame_len=N, n_freq=40, m=m, orders=orders) as p:
        whole = p.sequential(x)
        for lo in (0, 900, n_chunks - 300):
            piece = p.sequential(x, chunk_lo=lo, n_chunks=300)
            for o in orders:
                a, b = getattr(whole, f"s{o}")[lo:lo + 300], getattr(piece, f"s{o}")
                assert torch.isfinite(b).all() and torch.equal(a, b), (o, lo)
                assert torch.isnan(getattr(whole, f"s{o}_err")[..., 0]).all()
        torch.cuda.synchronize()
