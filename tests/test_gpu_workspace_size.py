"""What the workspace holds: no partial-sum slots for records of one chunk, which
the moment kernels finalize, and S2's chunk terms only where they are bounded and
fit.

Without the terms S2's sums come from the same FP32 chunk terms, formed from the
coefficients, in another FP64 order: 1e-12 of the largest value, as in the tests
of the terms."""
import ctypes as C

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


def _workspace_size(p, n_samples, C_):
    """ps_workspace_size of a record that is not there (nothing reads it)."""
    from paper_2505_01231_amd import _lib as L
    r = L.ps_record()
    r.d_data, r.n_samples, r.channel_stride, r.dtype = 1 << 20, n_samples, n_samples, L.PS_F32
    n = C.c_size_t()
    L.check(p._lib.ps_workspace_size(p._handle, C.byref(r), 1, C.byref(n)), "ps_workspace_size")
    return n.value


# Pairs of four channels at two frames a chunk: more bytes of terms than of
# coefficients.  Beyond their 8 GiB the workspace is the coefficients', S1's and
# the slots'.
@pytest.mark.parametrize("log2n", [20, 28, 33])
def test_chunk_terms_are_bounded(log2n):
    from paper_2505_01231_amd import Plan
    print("[gpu-case] bounded chunk terms", log2n, flush=True)
    N, m, n = 1024, 2, 1 << log2n
    with Plan(frame_len=N, n_freq=257, m=m, n_channels=4, orders=(1, 2)) as p:
        n_chunks = n // (N * m)
        coefficients, s1, slots = 4 * n_chunks * m * p.n_coef * 8, 4 * n_chunks * 8, 64 << 20
        assert _workspace_size(p, n, 4) <= coefficients + s1 + slots + (8 << 30)
        if log2n == 33:
            assert _workspace_size(p, n, 4) <= coefficients + s1 + slots


def _equal(a, b, tol=1e-12):
    for k in ("s1", "s1_err", "s2", "s2_err", "s3", "s3_err"):
        x, y = getattr(a, k), getattr(b, k)
        if x is None:
            continue
        assert torch.isfinite(y).all(), k
        assert (x - y).abs().max() <= tol * y.abs().max(), k


# A workspace that lacks half of the chunk terms: the call runs without them, as
# a graph too; one that lacks the coefficients is refused.
@pytest.mark.parametrize("orders,C_,m,n_chunks", [((1, 2), 4, 2, 2048), ((1, 2), 1, 20, 700), ((1, 2, 3), 2, 4, 1024)])
def test_workspace_without_room_for_the_terms(orders, C_, m, n_chunks):
    from paper_2505_01231_amd import Plan
    from paper_2505_01231_amd import _lib as L
    print("[gpu-case] no room for the terms", orders, C_, m, n_chunks, flush=True)
    N = 512
    x = _record(N, m, n_chunks, C_, 7)
    with Plan(frame_len=N, n_freq=65, m=m, n_channels=C_, orders=orders) as p:
        want = p.execute(x)
        full = p.workspace_bytes([x])
        pairs = len(p.combos2) if 3 not in orders else C_
        terms = pairs * n_chunks * 65 * 8
        coefficients = C_ * n_chunks * m * p.n_coef * 8
        ws = torch.full((full - terms // 2,), 0xFF, dtype=torch.uint8, device="cuda:0")
        st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        rec = (L.ps_record * 1)(p.record(x))
        out = p.allocate_outputs(x.device)
        o = (L.ps_output * 1)(out.c_struct())
        L.check(p._lib.ps_execute(p._handle, rec, 1, ws.data_ptr(), ws.numel(), o, st), "ps_execute")
        torch.cuda.synchronize()
        _equal(out, want)
        g, out = C.c_void_p(), p.allocate_outputs(x.device)
        o = (L.ps_output * 1)(out.c_struct())
        L.check(p._lib.ps_graph_create(p._handle, rec, 1, ws.data_ptr(), ws.numel(), o, C.byref(g)), "ps_graph_create")
        for _ in range(3):
            ws.fill_(0xFF)
            L.check(p._lib.ps_graph_launch(g, st), "ps_graph_launch")
            torch.cuda.synchronize()
            _equal(out, want)
        p._lib.ps_graph_destroy(g)
        assert p._lib.ps_execute(p._handle, rec, 1, ws.data_ptr(), coefficients, o, st) == L.PS_E_WORKSPACE


# The static scratch (256 MiB) holds a record's layout without the terms but not
# with them: S1 and S2 alone (centred coefficients written instead of held), and
# S2 beside S3.  The first length above the scratch is searched for, so that the
# branch is the one taken.
@pytest.mark.parametrize("orders,C_,m", [((1, 2), 4, 2), ((1, 2), 1, 4), ((1, 2, 3), 1, 4), ((2, 4), 1, 4)])
def test_static_scratch_without_the_terms(orders, C_, m):
    from paper_2505_01231_amd import Plan
    from paper_2505_01231_amd import _lib as L
    print("[gpu-case] static scratch without the terms", orders, C_, m, flush=True)
    N, Nf = 512, 65
    with Plan(frame_len=N, n_freq=Nf, m=m, n_channels=C_, orders=orders) as p:
        per_chunk = N * m
        lo, hi = 1, 1 << 21                       # chunks: fits, does not
        assert _workspace_size(p, hi * per_chunk, C_) > L.PS_STATIC_SCRATCH_BYTES
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if _workspace_size(p, mid * per_chunk, C_) <= L.PS_STATIC_SCRATCH_BYTES else (lo, mid)
        g = torch.Generator(device="cuda:0").manual_seed(m)
        x = torch.randn((C_, hi * per_chunk), generator=g, device="cuda:0") + 0.3
        x = x[0] if C_ == 1 else x
        assert p.workspace_bytes([x]) > L.PS_STATIC_SCRATCH_BYTES
        want, out = p.execute(x), p.allocate_outputs(x.device)
        rec, o = p.record(x), out.c_struct()
        st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        for _ in range(2):
            L.check(p._lib.ps_execute_static(p._handle, C.byref(rec), 1, C.byref(o), st), "ps_execute_static")
            torch.cuda.synchronize()
            _equal(out, want)
        if 4 in orders:
            assert torch.equal(out.s4, want.s4) and torch.equal(out.s4_err, want.s4_err)
