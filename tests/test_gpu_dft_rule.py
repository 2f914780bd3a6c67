"""The two forms of the two-stage direct transform on both sides of the lines of
their rule (rows in a block, bank conflicts of the few-rows form, long second
stages), against the FP64 FFT with the tolerance of test_gpu_dft_two_stage."""
import pytest

from tests.test_gpu_dft_two_stage import test_two_stage_transform as check

pytestmark = pytest.mark.gpu


# N1 x N2: without conflicts 16 x 257 and 17 x 433 (few rows; long), 17 x 109; with
# N2 + 1 = 4 i, 15 x 163 and 16 x 163; 8 i, 13 x 439 and 14 x 263; 16 i, 10 x 719 and
# 11 x 479
@pytest.mark.parametrize("N", [4112, 7361, 1853, 2445, 2608, 5707, 3682, 7190, 5269])
@pytest.mark.parametrize("n_frames", [1, 5])
def test_rule(N, n_frames):
    check(N, n_frames)
