"""The finalize in one launch and, from 32768 blocks of an order on, in one
launch per order, and the tiles that the moment kernels finalize themselves: the
same numbers each way."""
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
# (interlaced windows take every tile through the finalize)
@pytest.mark.parametrize("interlaced", [False, True])
def test_sequential_across_the_launch_limit(n_chunks, orders, interlaced):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] finalize launches", n_chunks, orders, interlaced, flush=True)
    N, m = 256, 4
    x = torch.from_numpy(synth.ar2_chi2(N * m * n_chunks, seed=n_chunks).astype(np.float32)).to("cuda:0")
    with Plan(frame_len=N, n_freq=40, m=m, orders=orders, interlaced=interlaced) as p:
        whole = p.sequential(x)
        for lo in (0, 900, n_chunks - 300):
            piece = p.sequential(x, chunk_lo=lo, n_chunks=300)
            for o in orders:
                a, b = getattr(whole, f"s{o}")[lo:lo + 300], getattr(piece, f"s{o}")
                assert torch.isfinite(b).all() and torch.equal(a, b), (o, lo)
                assert torch.isnan(getattr(whole, f"s{o}_err")[..., 0]).all()
        torch.cuda.synchronize()


# Tiles taken whole by one block against the same tiles cut into pieces: many
# records make whole tiles, a record alone is cut.  Grids around the 64-point
# tile, one channel and two, every precision, one chunk (no error bar) to nine.
# The FP64 sums of nine chunks may be added in another order: 1e-13.
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "fp16x2s"])
@pytest.mark.parametrize("C,Nf,n_chunks", [(1, 1, 2), (1, 64, 9), (1, 65, 3), (1, 100, 1), (2, 33, 9), (2, 65, 2)])
def test_whole_tiles(precision, C, Nf, n_chunks):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] whole tiles", precision, C, Nf, n_chunks, flush=True)
    N, m = 512, 5
    z = synth.mixed_channels(N * m * n_chunks, seed=Nf, n_channels=C)[0].astype(np.float32)
    x = torch.from_numpy(np.ascontiguousarray(z[0] if C == 1 else z)).to("cuda:0")
    with Plan(frame_len=N, n_freq=Nf, m=m, n_channels=C, precision=precision) as p:
        alone = p.execute(x)
        many = p.execute([x] * 600)
        torch.cuda.synchronize()
        for k in ("s2", "s3", "s4", "s2_err", "s3_err", "s4_err"):
            a = getattr(alone, k)
            for b in (getattr(many[0], k), getattr(many[599], k)):
                if n_chunks == 1 and k.endswith("_err"):
                    assert torch.isnan(a[..., 0]).all() and torch.isnan(b[..., 0]).all()
                    continue
                assert torch.isfinite(b).all(), k
                assert (a - b).abs().max() <= 1e-13 * a.abs().max(), k
                if k.startswith("s3") or (k.startswith("s4") and C == 1):       # S3 of (a, a, .), S4 of one channel
                    i = 0
                    assert torch.equal(b[i], b[i].transpose(0, 1)), k
