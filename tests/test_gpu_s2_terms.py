"""S1 and S2 from the chunk terms that the centring pass forms: S1 and S2 alone
(no centred coefficients), with higher orders, finalized directly or through
partial sums, against each other and the FP64 oracle.

The paths form the same FP32 chunk terms; their FP64 sums may differ in order
only: 1e-12 of the largest value bounds that for a few hundred chunks.  The
oracle comparison has the bar of the parity tests, 1e-5."""
import numpy as np
import pytest

import oracle as O
from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 256


def _run(x, orders, m, C, **kw):
    from paper_2505_01231_amd import Plan
    with Plan(frame_len=N, n_freq=41, m=m, orders=orders, n_channels=C, **kw) as p:
        out = p.execute(x)
        torch.cuda.synchronize()
        return {k: getattr(out, k).cpu().numpy() for k in ("s1", "s1_err", "s2", "s2_err")}, p.combos2


def _same(a, b, what, tol=1e-12):
    for k in a:
        assert np.all(np.isfinite(a[k])) and np.all(np.isfinite(b[k])), (what, k)
        assert np.max(np.abs(a[k] - b[k])) <= tol * np.max(np.abs(b[k])), (what, k)


# m around the 16 and 32 frames held in registers, channel counts around what
# fits with them (4 x 16, 2 x 32); 513 chunks go through partial sums
@pytest.mark.parametrize("C,m,n_chunks", [(1, 4, 1), (1, 16, 512), (1, 17, 513), (1, 32, 40), (1, 33, 40), (2, 10, 513),
                                          (2, 16, 5), (2, 20, 40), (3, 16, 40), (3, 17, 40), (4, 10, 7), (4, 16, 40)])
@pytest.mark.parametrize("kw", [{}, {"interlaced": True}, {"schedule": "per_chunk"}],
                         ids=["batched", "interlaced", "per_chunk"])
def test_s2_terms(C, m, n_chunks, kw):
    print("[gpu-case] s2 terms", C, m, n_chunks, kw, flush=True)
    if kw.get("schedule") == "per_chunk":
        n_chunks = min(n_chunks, 40)
    n_chunks = max(n_chunks, 3)
    z = synth.mixed_channels(N * m * n_chunks + N, seed=C * 100 + m, n_channels=C)[0].astype(np.float32)
    z = z[0] if C == 1 else z
    x = torch.from_numpy(np.ascontiguousarray(z)).to("cuda:0")
    alone, combos = _run(x, (1, 2), m, C, **kw)
    four = {} if m <= 32 else {"precision": "fp32"}
    with_s4, _ = _run(x, (1, 2, 4), m, C, combos4=[(0, 0, 0, 0)], **kw, **four)
    _same(alone, with_s4, "with S4")
    if kw:
        return
    ref = O.polyspectra(z, N, 41, m, window_kind="acg", orders=(1, 2), combos2=combos)
    got = alone["s2"][..., 0] + 1j * alone["s2"][..., 1]
    assert np.max(np.abs(got - ref["s2"])) <= 1e-5 * np.max(np.abs(ref["s2"]))
    assert np.max(np.abs(alone["s2_err"] - ref["s2_err"])) <= 1e-5 * np.max(np.abs(ref["s2_err"]))


def test_s2_terms_pairs_and_running_sum():
    """Pairs in any order and twice, and a running accumulation (partial sums)."""
    from paper_2505_01231_amd import Accumulator, Plan
    m, n_chunks = 10, 30
    z = synth.mixed_channels(N * m * n_chunks, seed=5, n_channels=3)[0].astype(np.float32)
    x = torch.from_numpy(z).to("cuda:0")
    pairs = [(1, 0), (0, 1), (2, 2), (0, 1), (2, 0)]
    got, _ = _run(x, (1, 2), m, 3, combos2=pairs)
    for i, c in enumerate(pairs):
        one, _ = _run(x, (1, 2, 4), m, 3, combos2=[c], combos4=[(0, 0, 0, 0)])
        _same({k: got[k][[i]] for k in ("s2", "s2_err")}, {k: one[k] for k in ("s2", "s2_err")}, c)
    with Plan(frame_len=N, n_freq=41, m=m, orders=(1, 2), n_channels=3, combos2=pairs) as p:
        acc = Accumulator(p, N * m * 7, dtype=torch.float32)
        for at in range(0, z.shape[1], N * m * 7):
            acc.push(x[:, at:at + N * m * 7].contiguous())
        out = acc.end()
        torch.cuda.synchronize()
        _same({k: getattr(out, k).cpu().numpy() for k in got}, got, "running")
