"""The power-of-two transform over its sample types, alignments and numbers of
columns: whole numbers below 2^15 are the same samples in int16, float32 and
float64, so every form gives the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# Columns around a quarter of the frame (the batch of eight per thread), all of
# them (the last column is one thread's) and a few; frames that end inside a block
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096, 8192])
def test_types_alignments_and_columns(N):
    from paper_2505_01231_amd import Plan
    m, n_chunks = 5, 7
    rng = np.random.default_rng(N)
    z = rng.integers(-30000, 30000, N * m * n_chunks + 1).astype(np.int16)
    z[0] = 12345                    # (the shifted views start after it)
    spectra = {}
    for nf in (3, N // 4 - 1, N // 4, N // 4 + 1, N // 2, N // 2 + 1):
        with Plan(frame_len=N, n_freq=nf, m=m, orders=(1, 2)) as p:
            for dtype in (np.int16, np.float32, np.float64):
                for aligned in (True, False):
                    print("[gpu-case] transform", N, nf, dtype.__name__, aligned, flush=True)
                    x = torch.from_numpy((z[1:] if aligned else z).astype(dtype)).to("cuda:0")
                    s2 = p.execute(x if aligned else x[1:]).s2
                    torch.cuda.synchronize()
                    spectra[nf, dtype, aligned] = s2.cpu().numpy().reshape(-1, 2)
    full = spectra[N // 2 + 1, np.float32, True]
    assert full.shape[0] == N // 2 + 1 and (full[1:-1, 0] > 0).all()
    for (nf, _, _), s in spectra.items():
        assert s.shape[0] == nf and np.array_equal(s, full[:nf]), nf
