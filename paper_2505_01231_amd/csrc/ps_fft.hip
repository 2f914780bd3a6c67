// Stage a1: windowed real FFT of every frame (Section 3, eq. a_k), and the
// per-chunk centring a' = a - mean_f a that the k-statistics of Section 4.1
// need in their centred form (Appendix H).
//
//   a_k = sum_{i<N} g_i z_i exp(+2 pi j i k / N),  k < K        (dt folded into the output scale)
//
// The N real samples of a frame are packed as M = N/2 complex points
// x_n = w_{2n} + j w_{2n+1} (w = g z), transformed by a Stockham FFT with the
// +j sign, and unpacked: with X the M-point transform,
//   E_k = (X_k + conj X_{M-k}) / 2,  O_k = (X_k - conj X_{M-k}) / (2j),
//   a_k = E_k + exp(+2 pi j k / N) O_k   (indices of X taken mod M).
// T = M/16 threads per frame each hold 16 points in registers; the passes are
// radix 16 (one radix-2/4/8 pass when log2 M is not a multiple of 4), so a
// 4096-point transform takes three passes through LDS.  The first pass reads
// the windowed samples from global memory straight into registers.  LDS holds
// X with one padding entry per 16 (index i at i + i/16), which keeps the
// first pass's 16-strided writes free of bank conflicts.  A 256-thread block
// transforms 256/T frames.  Twiddles come from tables computed in FP64 on the
// host: exp(+2 pi j t / N) for the unpack, and one table per later pass laid
// out [r][k], so that the twiddles of consecutive threads are consecutive
// entries (a gather from the plain table touches up to one cache line per
// lane).  The stage streams N samples in and K complex values out per frame.
// A complex-valued signal (complex float32 / float64 samples) needs no packing:
// its frames of M samples are windowed and transformed as they are (the same
// passes, instantiated for twice the frame length), and column c of the output
// holds X at bin c - jmax, taken mod M.
#include <algorithm>

#include "ps_internal.h"

namespace ps {
namespace {

constexpr int kFftThreads = 256;
constexpr int kFftLds = kFftThreads * 17;      // float2 entries: 4096 points + padding per block

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 mulj(float2 a) { return make_float2(-a.y, a.x); }   // j a
__device__ __forceinline__ int pad(int i) { return i + (i >> 4); }

// 4-point DFT with the +j sign on v[o], v[o+S], v[o+2S], v[o+3S], in place, natural order.
template <int S>
__device__ __forceinline__ void dft4(float2* v, int o) {
    const float2 a = v[o], b = v[o + S], c = v[o + 2 * S], d = v[o + 3 * S];
    const float2 s02 = cadd(a, c), d02 = csub(a, c), s13 = cadd(b, d), d13 = csub(b, d);
    v[o] = cadd(s02, s13);
    v[o + S] = cadd(d02, mulj(d13));
    v[o + 2 * S] = csub(s02, s13);
    v[o + 3 * S] = csub(d02, mulj(d13));
}
template <int S>
__device__ __forceinline__ void dft2(float2* v, int o) {
    const float2 a = v[o], b = v[o + S];
    v[o] = cadd(a, b);
    v[o + S] = csub(a, b);
}

// exp(+2 pi j q s / 16) for q, s < 4
__device__ __forceinline__ float2 w16(int qs) {
    constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508978f, h = 0.70710678118654752f;
    switch (qs) {
        case 1: return make_float2(c1, s1);
        case 2: return make_float2(h, h);
        case 3: return make_float2(s1, c1);
        case 4: return make_float2(0.f, 1.f);
        case 6: return make_float2(-h, h);
        case 9: return make_float2(-c1, -s1);
        default: return make_float2(1.f, 0.f);
    }
}

// R-point DFT (+j sign) of v[o .. o+R); output k is left at v[o + opos<R>(k)].
template <int R>
__device__ __forceinline__ void dft(float2* v, int o) {
    if constexpr (R == 16) {
        // n = q + 4 r, k = s + 4 t: DFT4 over r, twiddle exp(2 pi j q s / 16), DFT4 over q
#pragma unroll
        for (int q = 0; q < 4; ++q) dft4<4>(v, o + q);
#pragma unroll
        for (int q = 1; q < 4; ++q)
#pragma unroll
            for (int s2 = 1; s2 < 4; ++s2) v[o + q + 4 * s2] = cmul(v[o + q + 4 * s2], w16(q * s2));
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) dft4<1>(v, o + 4 * s2);
    } else if constexpr (R == 8) {
        // n = q + 2 r, k = s + 4 t: DFT4 over r, twiddle exp(2 pi j q s / 8), DFT2 over q
        dft4<2>(v, o);
        dft4<2>(v, o + 1);
        constexpr float h = 0.70710678118654752f;
        v[o + 3] = cmul(v[o + 3], make_float2(h, h));
        v[o + 5] = mulj(v[o + 5]);
        v[o + 7] = cmul(v[o + 7], make_float2(-h, h));
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) dft2<1>(v, o + 2 * s2);
    } else if constexpr (R == 4) {
        dft4<1>(v, o);
    } else {
        dft2<1>(v, o);
    }
}
template <int R>
__device__ __forceinline__ constexpr int opos(int k) {
    return R == 16 ? 4 * (k & 3) + (k >> 2) : R == 8 ? 2 * (k & 3) + (k >> 2) : k;
}

// Pair of consecutive samples (2n, 2n+1) as float2: one vector load when the
// frame is aligned for it, two scalar loads otherwise.  The pointer comes from a
// table of records, so the compiler cannot tell that it is device memory: flat
// loads, an address register pair for each, and of double precision's 16 each
// waited for the one before.  Measured with device-memory loads, the batches of
// load_pairs and of the last columns' twiddles: 9.0 -> 6.2 us (51200 samples in
// double precision, N = 256), 10.6 -> 8.0 (2^20, N = 1024), 21.5 -> 18.5 (2^22),
// 19.5 -> 15.8 (four windows of 2^20, N = 4096), 265 -> 249 (2^27, N = 1024).
template <typename T>
__device__ __forceinline__ float2 sample_pair(const T* __restrict__ xf, int n, bool vec) {
#if defined(__HIP__)
    typedef T T2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) T2 GlobalT2;
    typedef const __attribute__((address_space(1))) T GlobalT;
    if (vec) {
        const T2 d = ((GlobalT2*)xf)[n];
        return make_float2((float)d.x, (float)d.y);
    }
    return make_float2((float)((GlobalT*)xf)[2 * n], (float)((GlobalT*)xf)[2 * n + 1]);
#else
    (void)vec;
    return make_float2((float)xf[2 * n], (float)xf[2 * n + 1]);
#endif
}

// x is computed by here, and what uses t after it is computed later.
__device__ __forceinline__ void formed_here(float2& x, int& t) {
#if defined(__HIP__)
    asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(t));
#else
    (void)x;
    (void)t;
#endif
}

// The 16 pairs t + r Tn.  Double precision's come in two batches, the second
// (and the window) requested once the first is converted: 16 in flight do not
// fit the registers.
template <typename T>
__device__ __forceinline__ void load_pairs(float2 (&x)[16], const T* __restrict__ xf, int& t, int Tn, bool vec) {
    constexpr int B = sizeof(T) == 8 ? 8 : 16;
#pragma unroll
    for (int r0 = 0; r0 < 16; r0 += B) {
#pragma unroll
        for (int r = r0; r < r0 + B; ++r) x[r] = sample_pair(xf, t + r * Tn, vec);
        if (B < 16) {
#pragma unroll
            for (int r = r0; r < r0 + B; ++r) formed_here(x[r], t);
        }
    }
}

template <typename T>
__device__ __forceinline__ void load_first(float2 (&v)[16], const T* __restrict__ xf, const float* __restrict__ g,
                                           int t, int Tn, bool live) {
    if (!live) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = make_float2(0.f, 0.f);
        return;
    }
    // One branch per frame (the alignment is the frame's), not one per load.
    float2 x[16];
    if ((reinterpret_cast<uintptr_t>(xf) % (2 * sizeof(T))) == 0) load_pairs(x, xf, t, Tn, true);
    else load_pairs(x, xf, t, Tn, false);
    const float2* __restrict__ g2 = reinterpret_cast<const float2*>(g);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float2 w = g2[t + r * Tn];
        v[r] = make_float2(w.x * x[r].x, w.y * x[r].y);
    }
}

// Complex samples (n = t + r Tn) times the real window g_n.
template <typename T>
__device__ __forceinline__ void load_first_cplx(float2 (&v)[16], const T* __restrict__ xf,
                                                const float* __restrict__ g, int t, int Tn, bool live) {
    if (!live) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = make_float2(0.f, 0.f);
        return;
    }
    float2 x[16];
    load_pairs(x, xf, t, Tn, true);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float w = g[t + r * Tn];
        v[r] = make_float2(w * x[r].x, w * x[r].y);
    }
}

// Twiddles of a Stockham pass of radix R and span Ns (see fft_pass) for the
// butterflies of thread t: w[b R + r] = exp(+2 pi j r k / (R Ns)), k = j mod Ns,
// from the pass's table tbl[r Ns + k] (consecutive threads read consecutive k).
template <int LOG2M, int R>
__device__ __forceinline__ void pass_twiddles(float2 (&w)[16], int t, int Ns, const float2* __restrict__ tbl) {
    constexpr int M = 1 << LOG2M, Tn = M / 16, B = 16 / R;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int k = (t + b * Tn) & (Ns - 1);
#pragma unroll
        for (int r = 1; r < R; ++r) w[b * R + r] = tbl[r * Ns + k];
    }
}

// Stockham pass of radix R and span Ns over the M points of one frame held in
// LDS at s: butterfly j reads x[j + r M/R], twiddles by exp(+2 pi j r k / (R Ns))
// with k = j mod Ns (w, from pass_twiddles), and writes y[(j - k) R + k + r Ns].
// Thread t owns the 16/R butterflies j = t + b T.  FROM_REGS: the inputs are
// already in v (first pass, Ns = 1, natural order).
template <int LOG2M, int R, bool FROM_REGS>
__device__ __forceinline__ void fft_pass(float2 (&v)[16], const float2 (&w)[16], float2* s, int t, int Ns) {
    constexpr int M = 1 << LOG2M, Tn = M / 16, B = 16 / R;
    if (!FROM_REGS) {
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int r = 0; r < R; ++r) v[b * R + r] = s[pad(t + b * Tn + r * (M / R))];
        lds_barrier();
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int r = 1; r < R; ++r) v[b * R + r] = cmul(v[b * R + r], w[b * R + r]);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) dft<R>(v, b * R);
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int j = t + b * Tn, k = j & (Ns - 1);
        const int base = (j - k) * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r) s[pad(base + r * Ns)] = v[b * R + opos<R>(r)];
    }
    lds_barrier();
}

// One block's frames of one class: block `blk` of the class transforms its
// frames g_lo + blk F + (0..F-1) of channel `c`.
template <int LOG2N, bool CPLX>
__device__ __forceinline__ void window_rfft_block(const FftClass& a, int64_t blk, int c, float2* lds) {
    constexpr int N = 1 << LOG2N;
    constexpr int LOG2M = LOG2N - 1;
    constexpr int M = N / 2, Tn = M / 16, F = kFftThreads / Tn;
    constexpr int P16 = LOG2M / 4, REM = LOG2M % 4;
    // radices of the passes after the first (0: none)
    constexpr int R2 = fft_radix2(LOG2N), R3 = fft_radix3(LOG2N);
    static_assert(P16 <= 3 && !(P16 == 3 && REM), "frame length up to 8192");

    const int fl = threadIdx.x / Tn, t = threadIdx.x % Tn;
    float2* s = lds + fl * (M + M / 16);
    const int64_t gf = a.g_lo + blk * F + fl;     // frame of the class
    const bool live = gf < a.g_hi;
    RecDesc rec = a.single;
    if (a.recs && live) {
        int lo = 0, hi = a.n_recs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.recs[mid].frame0 <= gf) lo = mid;
            else hi = mid - 1;
        }
        rec = a.recs[lo];
    }
    const int64_t off = c * rec.chan_stride + (gf - rec.frame0) * (CPLX ? M : N);
    const float* __restrict__ g = a.g;
    const float2* __restrict__ tw = a.tw;

    // The second pass's twiddles are requested before the samples, the third
    // pass's just before its LDS reads (one pass ahead they spill registers).
    float2 v[16], w2[16], w3[16];
    if constexpr (R2 > 0) pass_twiddles<LOG2M, R2>(w2, t, 16, tw + N);
    if constexpr (CPLX) {
        if (rec.dtype == 3) load_first_cplx(v, static_cast<const float*>(rec.data) + 2 * off, g, t, Tn, live);
        else load_first_cplx(v, static_cast<const double*>(rec.data) + 2 * off, g, t, Tn, live);
    } else {
        if (rec.dtype == 0) load_first(v, static_cast<const float*>(rec.data) + off, g, t, Tn, live);
        else if (rec.dtype == 1) load_first(v, static_cast<const double*>(rec.data) + off, g, t, Tn, live);
        else load_first(v, static_cast<const int16_t*>(rec.data) + off, g, t, Tn, live);
    }

    fft_pass<LOG2M, 16, true>(v, w2, s, t, 1);
    if constexpr (R2 > 0) fft_pass<LOG2M, R2, false>(v, w2, s, t, 16);
    if constexpr (R3 > 0) pass_twiddles<LOG2M, R3>(w3, t, 16 * R2, tw + N + 16 * R2);
    if constexpr (R3 > 0) fft_pass<LOG2M, R3, false>(v, w3, s, t, 16 * R2);

    if (!live) return;
    const int K = a.K;                            // K <= M + 1
    float2* o = a.out + c * a.out_chan_stride + (gf - a.out_g0) * K;
    if constexpr (CPLX) {
        constexpr int KMAX = (M + 1 + Tn - 1) / Tn;
#pragma unroll
        for (int i = 0; i < KMAX; ++i) {
            const int col = t + i * Tn;
            if (col >= K) break;
            o[col] = s[pad((col - a.jmax) & (M - 1))];
        }
        return;
    }
    // Output k = e_k + w_k (X_k - conj X_{M-k}) (-j/2) from X_k and X_{M-k}.  The
    // roundings are spelled out, since which of two products is fused is the
    // compiler's choice: of columns t and M the halves er, ei are formed first, of
    // the others the products with w.
    auto combine = [&](int k, float2 w, bool halves) {
        const float2 xk = s[pad(k & (M - 1))];
        const float2 xm = s[pad((M - k) & (M - 1))];
        const float er = xk.x + xm.x, ei = xk.y - xm.y;
        const float orr = 0.5f * (xk.y + xm.y);   // (X_k - conj X_{M-k}) * (-j/2)
        const float oi = -0.5f * (xk.x - xm.x);
        const float re = halves ? fmaf(w.x, orr, 0.5f * er) : fmaf(0.5f, er, w.x * orr);
        const float im = halves ? fmaf(w.x, oi, 0.5f * ei) : fmaf(0.5f, ei, w.x * oi);
        return make_float2(fmaf(-w.y, oi, re), fmaf(w.y, orr, im));
    };
    // Eight columns at a time, their twiddles requested together and all of them
    // computed before the first is stored (a column after another, each behind
    // its own bounds check, waited for its twiddle each time).
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (8 * h * Tn >= K) break;
        float2 w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = t + (8 * h + i) * Tn;
            w[i] = tw[k < K ? k : K - 1];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = combine(t + (8 * h + i) * Tn, w[i], h + i == 0);
        int l = t;
#pragma unroll
        for (int i = 0; i < 8; ++i) formed_here(w[i], l);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = l + (8 * h + i) * Tn;
            if (k < K) o[k] = w[i];
        }
    }
    if (t + M < K) o[t + M] = combine(t + M, tw[t + M], true);     // column M (t = 0)
}

template <int LOG2N, bool CPLX>
__global__ __launch_bounds__(kFftThreads, 4) void k_window_rfft(FftArgs a) {
    __shared__ float2 lds[kFftLds];
    window_rfft_block<LOG2N, CPLX>(a.cls[0], blockIdx.x, blockIdx.y, lds);
}

// Several frame lengths in one launch (real signals): a block finds its class
// from its index and runs that frame length's transform.
template <int LOG2N>
__device__ __forceinline__ void rfft_class(const FftClass& k, int64_t blk, int c, float2* lds) {
    window_rfft_block<LOG2N, false>(k, blk, c, lds);
}

__global__ __launch_bounds__(kFftThreads, 4) void k_window_rfft_multi(FftArgs a) {
    __shared__ float2 lds[kFftLds];
    int ci = 0;
    for (int i = 1; i < a.n_cls; ++i)
        if ((int64_t)blockIdx.x >= a.cls[i].block0) ci = i;
    const FftClass& k = a.cls[ci];
    const int64_t blk = (int64_t)blockIdx.x - k.block0;
    switch (k.log2n) {
        case 8: rfft_class<8>(k, blk, blockIdx.y, lds); break;
        case 9: rfft_class<9>(k, blk, blockIdx.y, lds); break;
        case 10: rfft_class<10>(k, blk, blockIdx.y, lds); break;
        case 11: rfft_class<11>(k, blk, blockIdx.y, lds); break;
        case 12: rfft_class<12>(k, blk, blockIdx.y, lds); break;
        default: rfft_class<13>(k, blk, blockIdx.y, lds); break;
    }
}

// Frame lengths that are not a power of two: the windowed transform by its
// definition (Section 3, eq. a_k),
//   a_k = sum_{i<N} g_i z_i exp(+2 pi j i k / N),  k < K,
// as the product of the windowed frames [frames x N] with the exponentials
// [N x K], accumulated in FP64; exp(+2 pi j t / N) for t = i k mod N comes from
// an FP64 table of N entries (tw64).  N^2/2 complex products per frame where
// the FFT takes ~N log2 N: the path of the lengths that neither the FFT nor
// the two-stage form below takes (primes, and lengths without a divisor
// between 8 and sqrt(N)).
// A 256-thread block computes kDftFrames frames x kDftBins bins of one
// channel: thread (tf, tb) = (tid / 16, tid % 16) accumulates the frames
// f0 + tf + 16 u (u < 2) at the bins k0 + tb + 16 v (v < 4).  The samples pass
// in steps of kDftStep: each thread stages 4 windowed samples of one frame
// (FP64) and 8 exponentials of the step, then every thread adds the step's
// products.  Grid: x = frame blocks, y = channels, z = bin blocks.
constexpr int kDftFrames = 32, kDftBins = 64, kDftStep = 32;

__device__ __forceinline__ double dft_sample(const RecDesc& rec, int64_t idx) {
    if (rec.dtype == 0) return (double)static_cast<const float*>(rec.data)[idx];
    if (rec.dtype == 1) return static_cast<const double*>(rec.data)[idx];
    return (double)static_cast<const int16_t*>(rec.data)[idx];
}

__global__ __launch_bounds__(256) void k_window_dft(FftArgs args) {
    const FftClass& a = args.cls[0];
    __shared__ double sw[kDftFrames][kDftStep + 1];     // windowed samples of the step
    __shared__ double2 st[kDftStep][kDftBins];          // exponentials of the step

    const int N = a.dft_n, K = a.K;
    const int tid = threadIdx.x;
    const int tf = tid >> 4, tb = tid & 15;
    const int64_t f0 = a.g_lo + (int64_t)blockIdx.x * kDftFrames;
    const int k0 = (int)blockIdx.z * kDftBins;
    const int c = blockIdx.y;

    // staging role: frame lf of the block, samples ls .. ls + 3 of each step
    const int lf = tid >> 3, ls = 4 * (tid & 7);
    const int64_t gf = f0 + lf;
    const bool live = gf < a.g_hi;
    RecDesc rec = a.single;
    if (a.recs && live) {
        int lo = 0, hi = a.n_recs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.recs[mid].frame0 <= gf) lo = mid;
            else hi = mid - 1;
        }
        rec = a.recs[lo];
    }
    const int64_t off = c * rec.chan_stride + (gf - rec.frame0) * N;

    double acc[2][4][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v][0] = acc[u][v][1] = 0.0;

    for (int i0 = 0; i0 < N; i0 += kDftStep) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = i0 + ls + q;
            sw[lf][ls + q] = (live && i < N) ? (double)a.g[i] * dft_sample(rec, off + i) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int e = tid + 256 * q;                     // < kDftStep * kDftBins
            const int s = e / kDftBins, b = e % kDftBins;
            const int i = i0 + s, k = k0 + b;
            st[s][b] = (i < N && k < K) ? a.tw64[(int)(((int64_t)i * k) % N)] : make_double2(0.0, 0.0);
        }
        lds_barrier();
#pragma unroll 4
        for (int s = 0; s < kDftStep; ++s) {
            const double w0 = sw[tf][s], w1 = sw[tf + 16][s];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double2 t = st[s][tb + 16 * v];
                acc[0][v][0] = fma(w0, t.x, acc[0][v][0]);
                acc[0][v][1] = fma(w0, t.y, acc[0][v][1]);
                acc[1][v][0] = fma(w1, t.x, acc[1][v][0]);
                acc[1][v][1] = fma(w1, t.y, acc[1][v][1]);
            }
        }
        lds_barrier();
    }

#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int64_t g = f0 + tf + 16 * u;
        if (g >= a.g_hi) continue;
        float2* o = a.out + c * a.out_chan_stride + (g - a.out_g0) * K;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = k0 + tb + 16 * v;
            if (k < K) o[k] = make_float2((float)acc[u][v][0], (float)acc[u][v][1]);
        }
    }
}

// The same transform in two stages when N = N1 N2 factors well (N1 <= N2,
// both from dft_n1): with n = N2 n1 + n2 and k = k1 + N1 k2 (Cooley-Tukey),
//   Y[k1][n2] = exp(+2 pi j n2 k1 / N) sum_{n1 < N1} w[N2 n1 + n2] exp(+2 pi j n1 k1 / N1),
//   a_{k1 + N1 k2} = sum_{n2 < N2} Y[k1][n2] exp(+2 pi j n2 k2 / N2).
// The windowed samples and Y are FP32 in LDS, every sum is FP64, every
// exponential comes from the FP64 table of exp(+2 pi j t / N)
// (exp(+2 pi j t / N1) = entry t N2, exp(+2 pi j t / N2) = entry t N1).
//
// Stage 1 takes its samples, which are real, in order, each for an output k1
// and its conjugate N1 - k1.  (The order matters: where the exponentials are
// multiples of 60 degrees Y is a dyadic number up to FP64 rounding, often
// halfway between two FP32 values, and another order rounds it the other way.)
// Stage 2 adds the terms n and N2 - n together,
//   sum_n y_n exp(j th n) = y_0 + sum_{n < N2/2} (y_n + y_{N2-n}) cos(th n) + j (y_n - y_{N2-n}) sin(th n)
// (and y_{N2/2} (-1)^{k2}), four FMAs per pair.  A wave takes 64 columns n2
// (rows k1 in stage 2) and a tile of
// frequencies that all its lanes share (nine in stage 1, seven in stage 2: at
// N = 1536 one tile per wave): the exponentials are scalar loads and the
// samples, or the pair's sums, serve the whole tile.  dft2_frames frames per
// block fill the lanes when N1 is small; twice as many, or one, cost 30 and 40 %
// (LDS, idle lanes).
// Bound: nothing saturated; the samples, stage 1, stage 2 and the gathers of
// exp(n2 k1) run one after another, with four blocks per CU to overlap them.
// Measured (2^24 samples, N = 1536, K = 769): 159 us; with a product per output
// and term, its operands from LDS, 346 us.  2^22 samples, N = 296, 1016, 3336,
// 7992: 43, 83, 95 and 180 us against 58, 158, 152 and 377.
constexpr int kDft2Q = 7, kDft2Q1 = 9;
__host__ __device__ constexpr size_t dft2_frame_bytes(int N, int N1) {
    return (size_t)N * 4 + (size_t)N1 * (N / N1 + 1) * 8;
}
// Frames per block: the lanes' 64 rows, at most 40 KB of LDS (four blocks per CU).
__host__ __device__ constexpr int dft2_frames(int N, int N1) {
    const int by_rows = 64 / N1, by_lds = (int)(40960 / dft2_frame_bytes(N, N1));
    const int f = by_rows < by_lds ? by_rows : by_lds;
    return f > 1 ? f : 1;
}
__host__ __device__ constexpr size_t dft2_sx_bytes(int N, int N1) {
    return ((size_t)dft2_frames(N, N1) * N * 4 + 15) / 16 * 16;
}
// LDS (dynamic): the frames' windowed samples (FP32), then Y, N1 rows of N2 + 1 per frame.
__host__ __device__ constexpr size_t dft2_lds_bytes(int N, int N1) {
    return dft2_sx_bytes(N, N1) + (size_t)dft2_frames(N, N1) * N1 * (N / N1 + 1) * 8;
}

// A frame's windowed samples, six of a thread's in flight at once.
template <typename T>
__device__ __forceinline__ void dft2_stage(float* sx, const T* x, const float* g, int N) {
    constexpr int kBatch = 6;
    for (int i0 = threadIdx.x; i0 < N; i0 += 256 * kBatch) {
        T v[kBatch];
        float w[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = i0 + 256 * u;
            v[u] = i < N ? x[i] : T(0);
            w[u] = i < N ? g[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (i0 + 256 * u < N) sx[i0 + 256 * u] = (float)((double)w[u] * (double)v[u]);
    }
}

__global__ __launch_bounds__(256) void k_window_dft2(FftArgs args) {
    const FftClass& a = args.cls[0];
    HIP_DYNAMIC_SHARED(double2, dyn)
    const int N = a.dft_n, N1 = a.dft_n1, N2 = N / N1, K = a.K, F = dft2_frames(N, N1);
    float* sx = reinterpret_cast<float*>(dyn);                        // windowed samples [F][N]
    float2* sy = reinterpret_cast<float2*>(reinterpret_cast<char*>(dyn) + dft2_sx_bytes(N, N1));    // Y [F][N1][N2 + 1]
    // exp(+2 pi j t / N) by the byte offset 16 t, the same in all lanes; a step
    // mod the table's length (both below it: the smaller of the sum and,
    // unsigned, the sum less the length).  Packed copies of either stage's
    // entries measured the same.
    const uint32_t wrap = 16u * N;
    ConstMem<char>* tw = const_mem(reinterpret_cast<const char*>(a.tw64));
    auto step = [wrap](uint32_t t, uint32_t by) {
        const uint32_t u = t + by, v = u - wrap;
        return v < u ? v : u;
    };
    auto twiddle = [tw](uint32_t t) {
        typedef double pair_t __attribute__((vector_size(16)));
        const pair_t w = *reinterpret_cast<ConstMem<pair_t>*>(tw + t);
        return make_double2(w[0], w[1]);
    };

    const int tid = threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6);
    const int64_t g0 = a.g_lo + (int64_t)blockIdx.x * F;
    const int c = blockIdx.y;
    if (g0 >= a.g_hi) return;                            // (block-uniform)
    const int nf = (int)(a.g_hi - g0 < F ? a.g_hi - g0 : F);
    for (int f = 0; f < nf; ++f) {
        RecDesc rec = a.single;
        if (a.recs) {
            int lo = 0, hi = a.n_recs - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (a.recs[mid].frame0 <= g0 + f) lo = mid;
                else hi = mid - 1;
            }
            rec = a.recs[lo];
        }
        const int64_t off = c * rec.chan_stride + (g0 + f - rec.frame0) * N;
        if (rec.dtype == 0) dft2_stage(sx + f * N, static_cast<const float*>(rec.data) + off, a.g, N);
        else if (rec.dtype == 1) dft2_stage(sx + f * N, static_cast<const double*>(rec.data) + off, a.g, N);
        else dft2_stage(sx + f * N, static_cast<const int16_t*>(rec.data) + off, a.g, N);
    }
    lds_barrier();

    // stage 1: frequencies q and N1 - q, q <= N1 / 2, of 64 columns (frame, n2)
    {
        const int n_tiles = (N1 / 2 + kDft2Q1) / kDft2Q1, n_cols = nf * N2;
        const int n_items = n_tiles * ((n_cols + 63) / 64);
        for (int it = wave; it < n_items; it += 4) {
            const int q0 = it % n_tiles * kDft2Q1, col = it / n_tiles * 64 + lane;
            const bool live = col < n_cols;
            const int f = live ? col / N2 : 0, n2 = live ? col - f * N2 : 0;
            const float* x = sx + f * N + n2;
            double re[kDft2Q1], im[kDft2Q1];
            uint32_t t[kDft2Q1], by[kDft2Q1];            // entries n q N2 and q N2 mod N
#pragma unroll
            for (int j = 0; j < kDft2Q1; ++j) {
                re[j] = im[j] = 0.0;
                t[j] = 0;
                by[j] = 16u * N2 * ((q0 + j) % N1);
            }
            for (int n = 0; n < N1; ++n) {
                const double u = x[n * N2];
#pragma unroll
                for (int j = 0; j < kDft2Q1; ++j) {
                    const double2 w = twiddle(t[j]);
                    t[j] = step(t[j], by[j]);
                    re[j] = fma(u, w.x, re[j]);
                    im[j] = fma(u, w.y, im[j]);
                }
            }
            if (!live) continue;
            float2* y = sy + f * N1 * (N2 + 1) + n2;
#pragma unroll
            for (int j = 0; j < kDft2Q1; ++j) {
                const int q = q0 + j;
                if (2 * q > N1) break;
                const double2 w = a.tw64[n2 * q];        // n2 k1 < N
                y[q * (N2 + 1)] = make_float2((float)fma(re[j], w.x, -(im[j] * w.y)), (float)fma(im[j], w.x, re[j] * w.y));
                if (q == 0 || 2 * q == N1) continue;
                const double2 z = a.tw64[n2 * (N1 - q)];
                y[(N1 - q) * (N2 + 1)] =
                    make_float2((float)fma(re[j], z.x, im[j] * z.y), (float)fma(-im[j], z.x, re[j] * z.y));
            }
        }
    }
    lds_barrier();

    // stage 2: coefficients k = k1 + N1 k2 < K of 64 rows (frame, k1)
    const int n_k2 = (K + N1 - 1) / N1, n_tiles = (n_k2 + kDft2Q - 1) / kDft2Q, n_rows = nf * N1;
    const int n_items = n_tiles * ((n_rows + 63) / 64);
    for (int it = wave; it < n_items; it += 4) {
        const int q0 = it % n_tiles * kDft2Q, row = it / n_tiles * 64 + lane;
        const bool live = row < n_rows;
        const int f = live ? row / N1 : 0, k1 = live ? row - f * N1 : 0;
        const float2* y = sy + (f * N1 + k1) * (N2 + 1);
        double xr[kDft2Q], xi[kDft2Q];
        uint32_t t[kDft2Q], by[kDft2Q];                  // entries n k2 N1 and k2 N1 mod N
        const float2 y0 = y[0], ym = N2 % 2 ? make_float2(0.f, 0.f) : y[N2 / 2];
#pragma unroll
        for (int j = 0; j < kDft2Q; ++j) {
            const double s = (q0 + j) & 1 ? -1.0 : 1.0;
            xr[j] = fma(s, (double)ym.x, (double)y0.x);
            xi[j] = fma(s, (double)ym.y, (double)y0.y);
            t[j] = 0;
            by[j] = 16u * N1 * ((q0 + j) % N2);
        }
        for (int n = 1; n < N2 - n; ++n) {
            const float2 u = y[n], v = y[N2 - n];
            const double er = (double)u.x + (double)v.x, ei = (double)u.y + (double)v.y;
            const double dr = (double)u.x - (double)v.x, di = (double)u.y - (double)v.y;
#pragma unroll
            for (int j = 0; j < kDft2Q; ++j) {
                t[j] = step(t[j], by[j]);
                const double2 w = twiddle(t[j]);
                xr[j] = fma(er, w.x, fma(-di, w.y, xr[j]));
                xi[j] = fma(ei, w.x, fma(dr, w.y, xi[j]));
            }
        }
        if (!live) continue;
        float2* o = a.out + c * a.out_chan_stride + (g0 + f - a.out_g0) * K;
#pragma unroll
        for (int j = 0; j < kDft2Q; ++j) {
            const int k = k1 + N1 * (q0 + j);
            if (k < K) o[k] = make_float2((float)xr[j], (float)xi[j]);
        }
    }
}

// The two stages with a product per term and outputs spread over all threads,
// whatever N1: for lengths with a small N1 and a large N2 (8 x 1021), whose
// block holds too few rows for the lanes of k_window_dft2 (dft2_takes_few).
// LDS (dynamic): the N samples (FP32), the exponentials of the two stages
// exp(+2 pi j t / N1), t < N1, and exp(+2 pi j t / N2), t < N2 (FP64), then Y.
__host__ __device__ constexpr size_t dft2_few_sx_bytes(int N) { return ((size_t)N * 4 + 15) / 16 * 16; }
__host__ __device__ constexpr size_t dft2_few_lds_bytes(int N, int N1) {
    return dft2_few_sx_bytes(N) + (size_t)(N1 + N / N1) * 16 + (size_t)N1 * (N / N1 + 1) * 8;
}

__global__ __launch_bounds__(256) void k_window_dft2_few(FftArgs args) {
    const FftClass& a = args.cls[0];
    HIP_DYNAMIC_SHARED(double2, dyn)
    const int N = a.dft_n, N1 = a.dft_n1, N2 = N / N1, K = a.K;
    float* sx = reinterpret_cast<float*>(dyn);                        // windowed samples of the frame
    double2* sw1 = dyn + dft2_few_sx_bytes(N) / 16;                       // exp(+2 pi j t / N1)
    double2* sw2 = sw1 + N1;                                          // exp(+2 pi j t / N2)
    float2* sy = reinterpret_cast<float2*>(sw2 + N2);                 // Y, N1 rows of N2 + 1

    const int tid = threadIdx.x;
    const int64_t gf = a.g_lo + (int64_t)blockIdx.x;
    const int c = blockIdx.y;
    if (gf >= a.g_hi) return;                            // (block-uniform)
    RecDesc rec = a.single;
    if (a.recs) {
        int lo = 0, hi = a.n_recs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.recs[mid].frame0 <= gf) lo = mid;
            else hi = mid - 1;
        }
        rec = a.recs[lo];
    }
    const int64_t off = c * rec.chan_stride + (gf - rec.frame0) * N;
    for (int i = tid; i < N; i += 256) sx[i] = (float)((double)a.g[i] * dft_sample(rec, off + i));
    for (int t = tid; t < N1; t += 256) sw1[t] = a.tw64[t * N2];
    for (int t = tid; t < N2; t += 256) sw2[t] = a.tw64[t * N1];
    lds_barrier();

    // stage 1: (k1, n2) = (e / N2, e % N2), e < N
    for (int e = tid; e < N; e += 256) {
        const int k1 = e / N2, n2 = e - k1 * N2;
        double yr = 0.0, yi = 0.0;
        int t = 0;                                       // n1 k1 mod N1
        for (int n1 = 0; n1 < N1; ++n1) {
            const double x = sx[N2 * n1 + n2];
            const double2 w = sw1[t];
            yr = fma(x, w.x, yr);
            yi = fma(x, w.y, yi);
            t += k1;
            if (t >= N1) t -= N1;
        }
        const double2 w = a.tw64[n2 * k1];               // n2 k1 < N
        sy[k1 * (N2 + 1) + n2] = make_float2((float)(yr * w.x - yi * w.y), (float)(yr * w.y + yi * w.x));
    }
    lds_barrier();

    // stage 2: coefficient k = k1 + N1 k2 < K
    float2* o = a.out + c * a.out_chan_stride + (gf - a.out_g0) * K;
    for (int k = tid; k < K; k += 256) {
        const int k2 = k / N1, k1 = k - k2 * N1;
        const float2* y = sy + k1 * (N2 + 1);
        const int step = k2 % N2;
        double xr = 0.0, xi = 0.0;
        int t = 0;                                       // n2 k2 mod N2
        for (int n2 = 0; n2 < N2; ++n2) {
            const float2 v = y[n2];
            const double2 w = sw2[t];
            xr = fma((double)v.x, w.x, fma(-(double)v.y, w.y, xr));
            xi = fma((double)v.x, w.y, fma((double)v.y, w.x, xi));
            t += step;
            if (t >= N2) t -= N2;
        }
        o[k] = make_float2((float)xr, (float)xi);
    }
}

// One frame length's frames, `frames` a block: launch(args, blocks) per slice.
template <typename Launch>
hipError_t launch_frames(const FftArgs& a, int frames, Launch launch) {
    FftArgs b = a;
    const int64_t lo = a.cls[0].g_lo, hi = a.cls[0].g_hi;
    return launch_slices((hi - lo + frames - 1) / frames, [&](int64_t first, unsigned blocks) {
        b.cls[0].g_lo = lo + first * frames;
        b.cls[0].g_hi = std::min<int64_t>(hi, b.cls[0].g_lo + (int64_t)blocks * frames);
        launch(b, blocks);
    });
}

// Whether a two-stage length takes k_window_dft2_few: by the rows that a block of
// k_window_dft2 has for its 64 lanes, and by the bank conflicts of k_window_dft2_few,
// whose rows of Y lie N2 + 1 pairs apart.  Measured at 335 lengths (2^22 samples,
// time of k_window_dft2 over k_window_dft2_few): below 11 rows 1.1 to 3.5, with
// N2 + 1 = 16 i 0.9 to 1.7; 11 to 13 rows 1.1 to 2.5, 16 i 0.5 to 0.7, 16 i + 8 0.85
// and 1.14; 14 and 15 rows 1.1 to 1.5, 8 i 0.3 to 0.7; 16 rows 1.03 to 1.3, 4 i 0.8;
// from 17 rows on 0.3 to 1.07, but 0.9 to 1.3 beyond N2 = 320 without conflicts,
// where stage 2 is long and few blocks fit a CU (N = 7361: 484 us against 627).
bool dft2_takes_few(int N, int N1) {
    const int N2 = N / N1, rows = dft2_frames(N, N1) * N1, stride = (N2 + 1) % 16;
    if (stride == 0) return rows < 11;
    if (stride == 8) return rows < 14;
    return rows < (stride % 4 == 0 ? 16 : 17) || N2 > 320;
}

// The direct transform's launches: launch(kernel, grid, bytes of LDS, arguments).
template <typename Launch>
hipError_t dft_launches(const FftArgs& a, Launch launch) {
    const FftClass& c = a.cls[0];
    const int N = c.dft_n, N1 = c.dft_n1;
    if (N < 2 || !c.tw64 || c.K < 1) return hipErrorInvalidValue;
    if (N1 > 0) {                       // two stages, N = N1 N2
        if (N / N1 * N1 != N || N1 > N / N1) return hipErrorInvalidValue;
        const bool few = dft2_takes_few(N, N1);
        const size_t lds = few ? dft2_few_lds_bytes(N, N1) : dft2_lds_bytes(N, N1);
        if (lds > 160 * 1024) return hipErrorInvalidValue;
        return launch_frames(a, few ? 1 : dft2_frames(N, N1), [&](const FftArgs& b, unsigned blocks) {
            launch(few ? k_window_dft2_few : k_window_dft2, dim3(blocks, b.n_channels), lds, b);
        });
    }
    const unsigned bz = (c.K + kDftBins - 1) / kDftBins;
    return launch_frames(a, kDftFrames, [&](const FftArgs& b, unsigned blocks) {
        launch(k_window_dft, dim3(blocks, b.n_channels, bz), 0, b);
    });
}

hipError_t launch_dft(const FftArgs& a, hipStream_t st) {
    return dft_launches(a, [&](void (*kernel)(FftArgs), dim3 grid, size_t lds, const FftArgs& b) {
        kernel<<<grid, 256, lds, st>>>(b);
    });
}

template <int LOG2N>
hipError_t launch_n(const FftArgs& a, hipStream_t st) {
    constexpr int M = (1 << LOG2N) / 2, F = kFftThreads / (M / 16);
    if (a.cplx && LOG2N < 9) return hipErrorInvalidValue;
    return launch_frames(a, F, [&](const FftArgs& b, unsigned blocks) {
        const dim3 grid(blocks, b.n_channels);
        if constexpr (LOG2N >= 9)
            if (b.cplx) {
                k_window_rfft<LOG2N, true><<<grid, kFftThreads, 0, st>>>(b);
                return;
            }
        k_window_rfft<LOG2N, false><<<grid, kFftThreads, 0, st>>>(b);
    });
}

// a_k(f) -= (1/m) sum_{f' in chunk} a_k(f'), in place, one thread per (chunk, k).
// Chunks of up to kCentreRegs frames stay in registers between the mean and
// the subtraction, so each coefficient is read from HBM once.
//
// For the c3^(opt) estimator of S3 (Section 4.1) the same pass also writes the
// rows S3 multiplies: with x_f, y_f, z_f the chunk's three factors, x' = x - mean
// and P = sum over the three pairs of (1/m) sum_f x'_f y'_f times the third
// factor's mean, R = the product of the three means,
//   c3opt = ((m+4) M3' + 4 P + (4 - 2m) R) / (m + 1),  M3' = (1/m) sum x'y'z'.
// Since sum_f x'_f = 0, the rows x'_f + alpha mean with alpha = 4/(m+4) give
//   (1/m) sum_f (x' + alpha xm)(y' + alpha ym)(z' + alpha zm) = M3' + alpha P + alpha^3 R,
// and one more row mu mean per chunk, mu^3 = m ((4 - 2m)/(m+4) - alpha^3), adds
// the rest of R: the plain S3 sum over the m + 1 rows, times (m+4)/((m+1) m),
// is c3opt.
// float16 word pair (lo, hi), each rounded to nearest even.
typedef _Float16 f16x2_v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f16_pair(float lo, float hi) {
    const f16x2_v v = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// The operand records of the matrix-core S4 kernel for one column of one
// chunk (see kOpWords): piece i of value v (Re, Im, P) of column k at the
// 16-byte unit (3 v + i) op4_cols + k of the chunk's block, and the pair
// (p = sum_f P, s^2) at p4[chunk][k].  v holds the chunk's m <= kOpFrames
// uncentred values; a column without coefficients (k >= K, padding up to
// op4_cols) gets zero records, p = 0 and s = 1.
__device__ __forceinline__ void write_op_records(const CentreClass& cl, int64_t chunk, int k, int m,
                                                 const float2 (&v)[kCentreRegs], float mr, float mi, bool live) {
    const int64_t ngp = cl.op4_cols;
    uint4* rec = reinterpret_cast<uint4*>(cl.op4 + blockIdx.y * cl.op4_cs + chunk * (3 * kOpWords) * ngp) + k;
    float re[kOpFrames], im[kOpFrames], amax = 0.f;
#pragma unroll
    for (int f = 0; f < kOpFrames; ++f) {
        const bool on = live && f < m;
        re[f] = on ? v[f].x - mr : 0.f;                     // the centred values written to coef
        im[f] = on ? v[f].y - mi : 0.f;
        amax = fmaxf(amax, fmaxf(fabsf(re[f]), fabsf(im[f])));
    }
    const float s = pow2_above(amax);
    const float inv_s = 1.0f / s, inv_s2 = inv_s * inv_s;    // exact: powers of two
    float psum = 0.f;
#pragma unroll
    for (int val = 0; val < 3; ++val) {
        uint32_t w[10];
#pragma unroll
        for (int f = 0; f < kOpFrames; f += 2) {
            float x[2], l[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float P = fmaf(re[f + u], re[f + u], im[f + u] * im[f + u]);
                if (val == 2) psum += P;
                x[u] = val == 0 ? re[f + u] * inv_s : val == 1 ? im[f + u] * inv_s : P * inv_s2;
                l[u] = x[u] - (float)(_Float16)x[u];
            }
            w[f >> 1] = f16_pair(x[0], x[1]);
            w[5 + (f >> 1)] = f16_pair(l[0], l[1]);
        }
        uint4* dst = rec + val * kOpPieces * ngp;
        dst[0] = make_uint4(w[0], w[1], w[2], w[3]);                // H: h words 0..3
        dst[ngp] = make_uint4(w[5], w[6], w[7], w[8]);              // L: l words 0..3
        dst[2 * ngp] = make_uint4(w[4], w[9], 0u, 0u);              // T: h word 4, l word 4
    }
    double2* pp = reinterpret_cast<double2*>(cl.p4 + blockIdx.y * cl.p4_cs + chunk * 2 * ngp) + k;
    *pp = make_double2((double)psum, (double)(s * s));
}

// Grid: x = the classes' (chunk, 256-wide k block) pairs, chunk-major within
// each class; y = channel (the chunk count can exceed the 65536 limit of the y
// and z grid dimensions).
__global__ __launch_bounds__(256) void k_centre(CentreArgs a) {
    int ci = 0;
    for (int i = 1; i < a.n_cls; ++i)
        if ((int64_t)blockIdx.x >= a.cls[i].block0) ci = i;
    const CentreClass& cl = a.cls[ci];
    const int K = cl.K, m = a.m;
    const int kblocks = (K + 255) / 256;
    const int64_t local = (int64_t)blockIdx.x - cl.block0;
    const int64_t chunk = local / kblocks;
    const int k = (int)(local - chunk * kblocks) * 256 + threadIdx.x;
    if (k >= K) {
        if (cl.op4 && k < cl.op4_cols) {            // padding columns of the S4 operand records
            float2 z[kCentreRegs];
#pragma unroll
            for (int f = 0; f < kCentreRegs; ++f) z[f] = make_float2(0.f, 0.f);
            write_op_records(cl, chunk, k, m, z, 0.f, 0.f, false);
        }
        return;
    }
    float2* p = cl.coef + blockIdx.y * cl.coef_chan_stride + chunk * m * K + k;
    // c3^(opt): the chunk's rows for S3, frames shifted by alpha mean, then mu mean
    float2* q = cl.out3 ? cl.out3 + blockIdx.y * cl.out3_cs + chunk * (m + 1) * K + k : nullptr;
    const float inv = 1.0f / (float)m;
    const float alpha = a.alpha, mu = a.mu;
    // S1: the chunk's mean of a_0 (real for a real signal)
    auto keep_mean = [&](float mr, float mi) {
        if (a.s1 && k == a.s1_col) a.s1[blockIdx.y * a.s1_cs + cl.s1_chunk0 + chunk] = make_float2(mr, mi);
        if (q) q[(int64_t)m * K] = make_float2(mu * mr, mu * mi);
    };
    auto put = [&](int f, float2 v, float mr, float mi) {
        const float2 c = make_float2(v.x - mr, v.y - mi);
        p[(int64_t)f * K] = c;
        if (q) q[(int64_t)f * K] = make_float2(fmaf(alpha, mr, c.x), fmaf(alpha, mi, c.y));
    };
    if (m <= kCentreRegs) {
        float2 v[kCentreRegs];
        float sr = 0.f, si = 0.f;
#pragma unroll
        for (int f = 0; f < kCentreRegs; ++f) {
            if (f < m) {
                v[f] = p[(int64_t)f * K];
                sr += v[f].x;
                si += v[f].y;
            }
        }
        const float mr = sr * inv, mi = si * inv;
        keep_mean(mr, mi);
#pragma unroll
        for (int f = 0; f < kCentreRegs; ++f)
            if (f < m) put(f, v[f], mr, mi);
        const int ks = k - a.s2_col0, e = a.s2_entry[blockIdx.y][blockIdx.y];
        if (cl.s2c && e >= 0 && (unsigned)ks < (unsigned)cl.s2_n) {
            float re = 0.f;
#pragma unroll
            for (int f = 0; f < kCentreRegs; ++f) {
                const float x = v[f].x - mr, y = v[f].y - mi;
                if (f < m) re += fmaf(x, x, y * y);
            }
            cl.s2c[(e * cl.n_chunks + chunk) * cl.s2_n + ks] = make_float2(re, 0.f);
        }
        if (cl.op4 && k < cl.op4_cols) write_op_records(cl, chunk, k, m, v, mr, mi, true);
        return;
    }
    float sr = 0.f, si = 0.f;
    for (int f = 0; f < m; ++f) {
        const float2 v = p[(int64_t)f * K];
        sr += v.x;
        si += v.y;
    }
    const float mr = sr * inv, mi = si * inv;
    keep_mean(mr, mi);
    for (int f = 0; f < m; ++f) put(f, p[(int64_t)f * K], mr, mi);
}

// S1 and S2 alone (no other kernel reads the centred coefficients): the chunk's
// frames of all C channels are held in registers, centred there, and every
// wanted pair's chunk term is stored, with the arithmetic of k_s2.  One read of
// the coefficients in place of a read and a write here and another read in
// k_s2.  Bound: HBM.  Measured (2^27 samples, N = 1024, 513 columns, m = 10):
// 121 us (4.6 TB/s), against 200 us for k_centre and 142 for k_s2 (27 from the
// chunk terms).
template <int C, int R>
__global__ __launch_bounds__(256) void k_power(CentreArgs a) {
    int ci = 0;
    for (int i = 1; i < a.n_cls; ++i)
        if ((int64_t)blockIdx.x >= a.cls[i].block0) ci = i;
    const CentreClass& cl = a.cls[ci];
    const int K = cl.K, m = a.m;
    const int kblocks = (K + 255) / 256;
    const int64_t local = (int64_t)blockIdx.x - cl.block0;
    const int64_t chunk = local / kblocks;
    const int k = (int)(local - chunk * kblocks) * 256 + threadIdx.x;
    if (k >= K) return;
    const float inv = 1.0f / (float)m;
    float2 v[C][R];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float2* p = cl.coef + c * cl.coef_chan_stride + chunk * m * K + k;
#pragma unroll
        for (int f = 0; f < R; ++f)
            if (f < m) v[c][f] = p[(int64_t)f * K];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        float sr = 0.f, si = 0.f;
#pragma unroll
        for (int f = 0; f < R; ++f)
            if (f < m) sr += v[c][f].x, si += v[c][f].y;
        const float mr = sr * inv, mi = si * inv;
        if (a.s1 && k == a.s1_col) a.s1[c * a.s1_cs + cl.s1_chunk0 + chunk] = make_float2(mr, mi);
#pragma unroll
        for (int f = 0; f < R; ++f) v[c][f] = make_float2(v[c][f].x - mr, v[c][f].y - mi);
    }
    const int ks = k - a.s2_col0;
    if (!cl.s2c || (unsigned)ks >= (unsigned)cl.s2_n) return;
#pragma unroll
    for (int x = 0; x < C; ++x)
#pragma unroll
        for (int y = 0; y < C; ++y) {
            const int e = a.s2_entry[x][y];
            if (e < 0) continue;
            float re = 0.f, im = 0.f;
#pragma unroll
            for (int f = 0; f < R; ++f)
                if (f < m) {
                    const float2 p = v[x][f], q = v[y][f];
                    re += fmaf(p.x, q.x, p.y * q.y);
                    // (of one channel, chunks of up to kS2Regs frames: |a'|^2, real)
                    if (x != y || R > 16) im += fmaf(p.y, q.x, -(p.x * q.y));
                }
            cl.s2c[(e * cl.n_chunks + chunk) * cl.s2_n + ks] = make_float2(re, im);
        }
}

// Blocks of a centring launch (0: nothing to do, < 0: invalid).
int64_t centre_blocks(const CentreArgs& a) {
    if (a.n_cls > kMaxClasses) return -1;
    int64_t nx = 0;
    for (int i = 0; i < a.n_cls; ++i) {
        const CentreClass& c = a.cls[i];
        if (c.block0 != nx || c.n_chunks < 0) return -1;
        nx += (int64_t)((c.K + 255) / 256) * c.n_chunks;
    }
    return nx;
}

// Slice arguments of a launch whose classes are block ranges: the slice's
// block 0 is block `first` of the whole.
template <typename Args>
void shift_classes(Args& slice, const Args& whole, int64_t first) {
    for (int i = 0; i < whole.n_cls; ++i) slice.cls[i].block0 = whole.cls[i].block0 - first;
}

}  // namespace

hipError_t launch_power(const CentreArgs& a, hipStream_t s) {
    const int64_t nx = centre_blocks(a);
    if (nx == 0) return hipSuccess;
    if (nx < 0 || !power_supported(a.n_channels, a.m)) return hipErrorInvalidValue;
    void (*kernel)(CentreArgs) = nullptr;
    switch (a.n_channels * 2 + (a.m > 16)) {
        case 2: kernel = k_power<1, 16>; break;
        case 3: kernel = k_power<1, 32>; break;
        case 4: kernel = k_power<2, 16>; break;
        case 5: kernel = k_power<2, 32>; break;
        case 6: kernel = k_power<3, 16>; break;
        case 8: kernel = k_power<4, 16>; break;
        default: return hipErrorInvalidValue;
    }
    CentreArgs b = a;
    return launch_slices(nx, [&](int64_t first, unsigned blocks) {
        shift_classes(b, a, first);
        kernel<<<blocks, 256, 0, s>>>(b);
    });
}

hipError_t launch_window_rfft(const FftArgs& a, hipStream_t s) {
    if (a.n_cls <= 0 || a.n_channels <= 0) return hipSuccess;
    if (a.n_cls > 1) {          // several frame lengths: one launch, a class per block range
        if (a.cplx || a.n_cls > kMaxClasses) return hipErrorInvalidValue;
        for (int i = 0; i < a.n_cls; ++i)
            if (a.cls[i].dft_n) return hipErrorInvalidValue;
        int64_t blocks = 0;
        for (int i = 0; i < a.n_cls; ++i) {
            const FftClass& c = a.cls[i];
            const int F = kFftThreads / ((1 << c.log2n) / 32);
            if (c.block0 != blocks || c.g_hi < c.g_lo || c.log2n < 8 || c.log2n > 13) return hipErrorInvalidValue;
            blocks += (c.g_hi - c.g_lo + F - 1) / F;
        }
        FftArgs b = a;
        return launch_slices(blocks, [&](int64_t first, unsigned n) {
            shift_classes(b, a, first);
            k_window_rfft_multi<<<dim3(n, a.n_channels), kFftThreads, 0, s>>>(b);
        });
    }
    const FftClass& c0 = a.cls[0];
    if (c0.g_hi <= c0.g_lo || c0.n_recs <= 0) return hipSuccess;
    if (c0.dft_n) {            // N not a power of two: the direct transform
        if (a.cplx) return hipErrorInvalidValue;
        return launch_dft(a, s);
    }
    switch (c0.log2n) {
        case 8: return launch_n<8>(a, s);
        case 9: return launch_n<9>(a, s);
        case 10: return launch_n<10>(a, s);
        case 11: return launch_n<11>(a, s);
        case 12: return launch_n<12>(a, s);
        case 13: return launch_n<13>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_centre(const CentreArgs& a, hipStream_t s) {
    const int64_t nx = centre_blocks(a);
    if (nx == 0) return hipSuccess;
    if (nx < 0) return hipErrorInvalidValue;
    CentreArgs b = a;
    return launch_slices(nx, [&](int64_t first, unsigned blocks) {
        shift_classes(b, a, first);
        k_centre<<<dim3(blocks, a.n_channels), 256, 0, s>>>(b);
    });
}

}  // namespace ps
