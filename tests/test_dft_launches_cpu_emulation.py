"""Both forms of the two-stage direct transform under the library's own launches
(dft_launches: the choice of the form, its LDS and its grid), compiled for the CPU
and run under AddressSanitizer and UndefinedBehaviorSanitizer with every buffer,
the dynamic LDS included, allocated to its exact size (test infrastructure; no
GPU; see tests/test_fft_cpu_emulation.py, whose driver this is)."""
import pytest

emu = pytest.importorskip("tests.test_fft_cpu_emulation")
driver = emu.driver         # fixture

# (N, frames, dtype, misaligned, N1): k_window_dft2_few at 8 x 251, 11 x 727, 13 x 331
# and, for its length, 17 x 433; k_window_dft2 with three and four frames a block and
# frame counts that are no multiple of them (8 x 127, 15 x 19, 16 x 17), one frame a
# block (17 x 307) and rows just above the rule's lines (11 x 479, 16 x 163)
INSTANCES = [(2008, 2, 2, 1, 8), (7997, 1, 0, 0, 11), (4303, 2, 1, 0, 13), (7361, 1, 0, 1, 17), (1016, 4, 0, 1, 8),
             (1016, 3, 1, 0, 8), (285, 5, 2, 0, 15), (285, 1, 0, 0, 15), (272, 7, 0, 0, 16), (5219, 2, 0, 0, 17),
             (5269, 1, 2, 0, 11), (2608, 2, 0, 0, 16)]


@pytest.mark.parametrize("N,frames,dtype,mis,n1", INSTANCES)
def test_two_stage_launches_in_bounds_and_correct(driver, tmp_path, N, frames, dtype, mis, n1):
    assert emu.library_factor(N) == n1
    emu.test_direct_transform_kernel_in_bounds_and_correct(driver, tmp_path, N, frames, dtype, mis, n1)
