"""Cross-channel S4 on the matrix cores (BF16 x 3): the forms that share Grams
between coinciding channels, and between (a, b, c, d) and (a, b, d, c), against
the form that shares none.

The forms add the same FP32 values in the same order, so only the order of the
FP64 chunk sums (the work split) may differ: 16 sums of relative rounding 2^-53
and the subtraction in the error bar, whose square cancels by less than 10^4
here, stay below 1e-10 of the largest value."""
import numpy as np
import pytest

from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10


def _s4(z, N, Nf, m, combos, **kw):
    from paper_2505_01231_amd import Plan
    with Plan(frame_len=N, n_freq=Nf, m=m, orders=(4,), n_channels=4, precision="bf16x3", combos4=combos, **kw) as p:
        out = p.execute(torch.from_numpy(z).to("cuda:0"))
        torch.cuda.synchronize()
        return out.s4.cpu().numpy(), out.s4_err.cpu().numpy()


def _close(a, b, what):
    for x, y, name in zip(a, b, ("s4", "err")):
        assert np.all(np.isfinite(x)) and np.all(np.isfinite(y)), (what, name)
        assert np.max(np.abs(x - y)) <= TOL * np.max(np.abs(y)), (what, name)


# grids around the 32-point tile, chunks around the 10-frame batch; ten chunks
# so that blocks take several
@pytest.mark.parametrize("Nf,m", [(1, 4), (31, 5), (32, 10), (33, 11), (64, 13), (47, 21)])
@pytest.mark.parametrize("schedule", ["batched", "per_chunk"])
def test_s4_cross_forms(Nf, m, schedule):
    print("[gpu-case] s4 cross forms", Nf, m, schedule, flush=True)
    N = 256
    z = synth.mixed_channels(N * m * 10 + 5, seed=7 * Nf + m, n_channels=4)[0].astype(np.float32)
    args = dict(schedule=schedule)
    # a pair, its combinations listed twice, against each combination alone
    both = [(0, 1, 2, 3), (0, 1, 3, 2), (0, 1, 3, 2), (0, 1, 2, 3), (2, 0, 0, 1)]
    got = _s4(z, N, Nf, m, both, **args)
    for i, c in enumerate(both):
        _close([x[i] for x in got], [x[0] for x in _s4(z, N, Nf, m, [c], **args)], c)
    # channels that hold the same samples under two numbers go the general way
    z[1], z[3] = z[0], z[2]
    general = _s4(z, N, Nf, m, [(0, 1, 2, 3)], **args)
    for c in ((0, 0, 2, 3), (0, 1, 2, 2), (0, 0, 2, 2)):
        _close(_s4(z, N, Nf, m, [c], **args), general, c)
