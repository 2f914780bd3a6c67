// Host driver of the launchers' slicing (test infrastructure only): launch_slices,
// launch_frames, shift_classes and the rule for S3 and S4 in one launch, from the
// library's sources, with counts around and above the blocks one launch takes.
// Prints the first fault and fails.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "ps_fft_extract.inc"

thread_local emu_idx threadIdx, blockIdx;
std::barrier<>* emu_block_barrier = nullptr;
char* emu_dyn_smem = nullptr;

static void check(bool ok, const char* what, int64_t n) {
    if (ok) return;
    fprintf(stderr, "%s, n = %lld\n", what, (long long)n);
    exit(1);
}

int main() {
    const int64_t L = ps::kMaxBlocks;
    check((L + 1) * 256 > 0xffffffffLL && L * 256 <= 0xffffffffLL, "kMaxBlocks is the 2^32-thread limit", L);
    for (int64_t n : {int64_t(0), int64_t(1), L - 1, L, L + 1, 2 * L, 3 * L + 5}) {
        int64_t next = 0;
        const hipError_t e = ps::launch_slices(n, [&](int64_t first, unsigned blocks) {
            check(first == next && blocks >= 1 && blocks <= L, "slice", n);
            next += blocks;
        });
        check(e == hipSuccess && next == n, "slices cover every block once", n);
    }
    for (int frames : {1, 3, 32})
        for (int64_t n : {int64_t(0), int64_t(1), L * frames - 1, L * frames, L * frames + 1, 2 * L * frames + frames - 1}) {
            ps::FftArgs a{};
            a.n_cls = 1;
            a.cls[0].g_lo = 7;
            a.cls[0].g_hi = 7 + n;
            a.cls[0].out_g0 = 7;
            int64_t next = 7;
            ps::launch_frames(a, frames, [&](const ps::FftArgs& b, unsigned blocks) {
                const ps::FftClass& c = b.cls[0];
                check(c.g_lo == next && c.g_hi > c.g_lo && c.out_g0 == 7, "frames of a slice", n);
                check((c.g_hi - c.g_lo + frames - 1) / frames == blocks && blocks <= L, "blocks of a slice", n);
                next = c.g_hi;
            });
            check(next == 7 + n, "slices cover every frame once", n);
        }
    // a block of a slice finds the class and the block within it of the whole
    ps::FftArgs w{};
    w.n_cls = 3;
    w.cls[0].block0 = 0;
    w.cls[1].block0 = 10;
    w.cls[2].block0 = L + 3;
    ps::FftArgs s = w;
    for (int64_t first : {int64_t(0), L}) {
        ps::shift_classes(s, w, first);
        for (int64_t x : {int64_t(0), int64_t(2), int64_t(3), int64_t(9), int64_t(10), L - 1}) {
            auto find = [](const ps::FftArgs& a, int64_t b) {
                int ci = 0;
                for (int i = 1; i < a.n_cls; ++i)
                    if (b >= a.cls[i].block0) ci = i;
                return ci;
            };
            const int cs = find(s, x), cw = find(w, x + first);
            check(cs == cw && x - s.cls[cs].block0 == x + first - w.cls[cw].block0, "class of a block", x + first);
        }
    }
    // S3 and S4 share a launch while their blocks together fit one
    check(ps::s3_s4_supported(1, 1, 10) && !ps::s3_s4_supported(1, 1, 11), "rows", 1);
    check(!ps::s3_s4_supported(0, 5, 10) && !ps::s3_s4_supported(5, 0, 10), "nothing to merge", 0);
    const int64_t half = (L + 1) / 2 - 8;       // a multiple of 8
    check(ps::s3_s4_supported(half, half, 10), "two halves", half);
    check(ps::s3_s4_supported(half, half + 8, 10), "all blocks", half);
    check(!ps::s3_s4_supported(half, half + 9, 10), "one round too many", half);
    check(!ps::s3_s4_supported(half + 8, half + 8, 10), "more than a launch", half);
    check(!ps::s3_s4_supported(L - 7, L - 7, 10), "as many as separate launches take", L);
    return 0;
}
