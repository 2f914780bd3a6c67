"""Calls whose launches have more blocks than a dispatch counts threads for
(2^32): every output against calls of fewer chunks."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# S2's finalize has 16 blocks a chunk and S1's one: 10^6 chunks are 1.7e7 blocks
# together, 16e6 for S2 alone; 1.06e6 are more than 2^24 for S2 alone
@pytest.mark.parametrize("n_chunks", [1000000, 1060000])
def test_sequential_of_a_million_chunks(n_chunks):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] finalize of", n_chunks, "chunks", flush=True)
    N, m = 256, 2
    x = (torch.arange(N * m * n_chunks, device="cuda:0", dtype=torch.int32) % 1009).to(torch.int16)
    with Plan(frame_len=N, n_freq=1, m=m, orders=(1, 2)) as p:
        whole = p.sequential(x)
        for lo in (0, 222700, n_chunks // 2, n_chunks - 1000):
            piece = p.sequential(x, chunk_lo=lo, n_chunks=1000)
            for k in ("s1", "s2"):
                a, b = getattr(whole, k)[lo:lo + 1000], getattr(piece, k)
                assert torch.isfinite(b).all() and (b != 0).any(), (k, lo)
                assert torch.equal(a, b), (k, lo)
        torch.cuda.synchronize()


# A chunk repeated 2^24 + 4096 times: one block each in the centring pass (and in
# k_power, S1 and S2 alone).  Every chunk's estimate is the same: n equal FP64
# terms in any order are off by n 2^-53 = 2e-9 at most, and the variance of the
# mean by as much of the mean squared, over n: sigma below 2e-8 of the mean.
@pytest.mark.parametrize("orders,m", [((1, 2), 2), ((1, 2, 3), 3)])
def test_record_of_more_chunks_than_a_launch_has_blocks(orders, m):
    from paper_2505_01231_amd import Plan
    n = (1 << 24) + 4096
    print("[gpu-case] record of", n, "chunks", orders, flush=True)
    g = torch.Generator().manual_seed(m)
    c = (torch.randn(256 * m, generator=g) * 1000 + 50).to(torch.int16).to("cuda:0")
    with Plan(frame_len=256, n_freq=1, m=m, orders=orders) as p:
        one, many = p.execute(c), p.execute(c.repeat(n))
        torch.cuda.synchronize()
        assert many.n_chunks == n
        for o in orders:
            a, b, e = getattr(one, f"s{o}"), getattr(many, f"s{o}"), getattr(many, f"s{o}_err")
            assert torch.isfinite(a).all() and a.abs().max() > 0, o
            assert (a - b).abs().max() <= 1e-8 * a.abs().max(), o
            assert e.abs().max() <= 1e-7 * a.abs().max(), o
