"""The workspace holds no partial-sum slots for records of one chunk, which the
moment kernels finalize."""
import numpy as np
import pytest

from paper_2505_01231_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _record(N, m, n_chunks, C, seed):
    z = synth.mixed_channels(N * m * n_chunks, seed=seed, n_channels=C)[0].astype(np.float32)
    return torch.from_numpy(np.ascontiguousarray(z[0] if C == 1 else z)).to("cuda:0")


# Coefficients, S2's chunk terms, S1's means and (scaled FP16 x 2) S4's operand
# records, and a table of at most eight segments of 256 bytes per combination and
# chunk; the slots of every tile would be 192 KB a tile more.
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "fp16x2s"])
def test_sequential_workspace_has_no_slots(precision):
    from paper_2505_01231_amd import Plan
    N, Nf, m, n = 1024, 200, 4, 120
    print("[gpu-case] sequential workspace", precision, flush=True)
    x = _record(N, m, n, 1, 3)
    with Plan(frame_len=N, n_freq=Nf, m=m, orders=(1, 2, 3, 4), precision=precision) as p:
        p.sequential(x)
        torch.cuda.synchronize()
        coefficients, terms, s1 = 8 * n * m * p.n_coef, 8 * n * Nf, 8 * n
        operands = n * 256 * (3 * 16 * 4 + 16) if precision == "fp16x2s" else 0
        tables = n * 4 * 8 * 256 + 65536
        assert p._last_workspace.numel() <= coefficients + terms + s1 + operands + tables


# One chunk: every tile is whole and has no slot.  The per-chunk schedule forms
# the same sums and takes every tile through a slot and the finalize; mean and
# scale are then two roundings on either side: 4 * 2^-53 of the value.  Two
# channels in BF16 x 3 are the combinations formed in pairs.
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "fp16x2s"])
@pytest.mark.parametrize("C,Nf", [(1, 1), (1, 64), (1, 100), (2, 33), (2, 65)])
def test_one_chunk_without_slots(precision, C, Nf):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] one chunk without slots", precision, C, Nf, flush=True)
    N, m, n = 512, 5, 9
    x = _record(N, m, n, C, Nf)
    kw = dict(frame_len=N, n_freq=Nf, m=m, n_channels=C, orders=(1, 2, 3, 4), precision=precision)
    with Plan(**kw) as p, Plan(schedule="per_chunk", **kw) as q:
        seq = p.sequential(x)
        chunks = [x[..., i * N * m:(i + 1) * N * m].contiguous() for i in range(n)]
        many, ref = p.execute(chunks), q.execute(chunks)
        torch.cuda.synchronize()
        for i in range(n):
            for k in ("s1", "s2", "s3", "s4"):
                r = getattr(ref[i], k)
                assert torch.isfinite(r).all(), k
                for a in (getattr(seq, k)[i], getattr(many[i], k)):
                    assert (a - r).abs().max() <= 4 * 2.0 ** -53 * r.abs().max(), (k, i)
                e, f = getattr(ref[i], k + "_err"), getattr(many[i], k + "_err")
                assert torch.isnan(e[..., 0]).all() and torch.equal(torch.isnan(e), torch.isnan(f)), (k, i)
