// Cross-power map formation on gfx950: the step before the template search that turns two
// detectors' strain into the complex SNR maps it scores (Sec. II, Eq. 7, and the formalism
// appendix), with time slides of one detector for background maps (Sec. IV-V).
//
//   k_col_fft     one workgroup per column: M Hann-weighted samples (columns overlap by half),
//                 a length-M/2 complex FFT in LDS over the even/odd sample pairs, then the
//                 real-FFT split for the kept bins only; s~ = dt * DFT.
//   k_psd         P'(t; f): mean of (2 / Nrm) |s~|^2 over the columns 2 .. nb+1 away.
//   k_form_maps   per (t, f) and per slide: Y = (2 / Nrm) conj(s~_I) s~_J(t + shift) and
//                 sigma = sqrt(P'_I P'_J(t + shift) / 2), written to the caller's maps.
//
// Twiddles e^{-2 pi i j / M} (j < M/2) and the window sin^2(pi n / M) come from a table the
// host fills in FP64 and rounds once to FP32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stt {

constexpr int kFftThreads = 256;   // at most; a column of N points uses N / 8
constexpr int kMaxFftM = 8192;     // samples per column; the complex FFT has M/2 points in LDS
constexpr int kSlidesPerLaunch = 64;  // 20 bytes each of the 4 KB of kernel arguments
constexpr int64_t kPsdPixels = (int64_t)2 << 20;  // T F from which k_psd takes four columns per lane

struct SlideArgs {
    float2 *Y[kSlidesPerLaunch];
    float *sigma[kSlidesPerLaunch];
    int32_t shift[kSlidesPerLaunch];  // in [0, T)
    int32_t n;
};

// LDS word of FFT element i. Passes touch elements 2^s apart from lanes 8 or 64 elements apart; the
// pad spreads both over the banks.
__host__ __device__ __forceinline__ constexpr int fft_slot(int i) { return i + (i >> 5) + ((i >> 6) << 3); }

// Stages s .. s+G-1 of the radix-2 decimation in time on the 2^G elements v[j] at i0 + j 2^s, low =
// i0 mod 2^s: stage s+q joins blocks of 2^(s+q) elements, e^{-2 pi i p / 2^(s+q+1)} = tw[p M / 2^(s+q+1)].
template <int G>
__device__ __forceinline__ void fft_stages(float2 *v, int s, int low, int M, const float2 *__restrict__ tw)
{
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const int tstep = M >> (s + q + 1);
#pragma unroll
        for (int p = 0; p < (1 << q); ++p) {
            const float2 w = tw[(low + (p << s)) * tstep];
#pragma unroll
            for (int j = p; j < (1 << G); j += 2 << q) {
                const float2 a = v[j], c = v[j + (1 << q)];
                const float cr = w.x * c.x - w.y * c.y, ci = w.x * c.y + w.y * c.x;
                v[j] = make_float2(a.x + cr, a.y + ci);
                v[j + (1 << q)] = make_float2(a.x - cr, a.y - ci);
            }
        }
    }
}

// First pass: 2^G windowed samples straight from the strain. Element r of the bit-reversed order
// holds sample pair bitrev(r); lane w takes r = 2^G bitrev(w) + j, sample pairs w + bitrev(j) N/2^G.
template <int G>
__device__ __forceinline__ void fft_load_pass(float2 *z, const float2 *__restrict__ seg, const float2 *__restrict__ win2,
                                              int M, int lg, const float2 *__restrict__ tw)
{
    const int items = 1 << (lg - G);
    for (int w = threadIdx.x; w < items; w += blockDim.x) {
        float2 v[1 << G];
#pragma unroll
        for (int j = 0; j < (1 << G); ++j) {
            const int i = w + (int)(__builtin_bitreverse32((unsigned)j) >> (32 - G)) * items;
            const float2 x = seg[i], h = win2[i];
            v[j] = make_float2(x.x * h.x, x.y * h.y);
        }
        fft_stages<G>(v, 0, 0, M, tw);
        const int r = lg > G ? (int)(__builtin_bitreverse32((unsigned)w) >> (32 - (lg - G))) << G : 0;
#pragma unroll
        for (int j = 0; j < (1 << G); ++j) z[fft_slot(r + j)] = v[j];
    }
}

template <int G>
__device__ __forceinline__ void fft_pass(float2 *z, int s, int M, int lg, const float2 *__restrict__ tw)
{
    __syncthreads();
    for (int w = threadIdx.x; w < 1 << (lg - G); w += blockDim.x) {
        const int low = w & ((1 << s) - 1);
        const int i0 = ((w >> s) << (s + G)) + low;
        float2 v[1 << G];
#pragma unroll
        for (int j = 0; j < (1 << G); ++j) v[j] = z[fft_slot(i0 + (j << s))];
        fft_stages<G>(v, s, low, M, tw);
#pragma unroll
        for (int j = 0; j < (1 << G); ++j) z[fft_slot(i0 + (j << s))] = v[j];
    }
}

// x: strain (8-byte aligned); tab: M/2 twiddles (float2) followed by M window values (float);
// spec: [T][F] complex64. Grid: T workgroups, fft_slot(N) float2 of LDS, N = M/2 = 2^lg >= 4.
// Bound by latency: a stage at a time through LDS was 11 barriers and a twiddle gather in front of
// each at M = 4096. Three stages at a time stay in registers (the same butterflies in the same
// order; contracted otherwise, so spectra agree to rounding), and the first three take the samples straight from memory.
__global__ __launch_bounds__(kFftThreads) void k_col_fft(const float *__restrict__ x, int M, int lg, int k_lo, int F,
                                                         float dt, const float2 *__restrict__ tab,
                                                         float2 *__restrict__ spec)
{
    extern __shared__ float2 z[];
    const int N = M >> 1;
    const float2 *tw = tab;
    const float2 *win2 = reinterpret_cast<const float2 *>(tab + N);  // window pairs (w[2i], w[2i+1])
    const int t = blockIdx.x;
    // even/odd sample pairs as one complex sequence
    const float2 *seg = reinterpret_cast<const float2 *>(x + (int64_t)t * N);
    int s;
    if (lg >= 3) {
        fft_load_pass<3>(z, seg, win2, M, lg, tw);
        s = 3;
    } else {
        fft_load_pass<2>(z, seg, win2, M, lg, tw);
        s = 2;
    }
    for (; s + 3 <= lg; s += 3) fft_pass<3>(z, s, M, lg, tw);
    if (lg - s == 2) fft_pass<2>(z, s, M, lg, tw);
    else if (lg - s == 1) fft_pass<1>(z, s, M, lg, tw);
    __syncthreads();
    // X[k] = E[k] + e^{-2 pi i k / M} O[k] with E = (Z[k] + conj Z[N-k]) / 2 (even samples) and
    // O = (Z[k] - conj Z[N-k]) / 2i (odd samples); only the kept bins k_lo .. k_lo+F-1 (< N)
    for (int f = threadIdx.x; f < F; f += blockDim.x) {
        const int k = k_lo + f;
        const float2 a = z[fft_slot(k)], b = z[fft_slot((N - k) & (N - 1))];
        const float er = 0.5f * (a.x + b.x), ei = 0.5f * (a.y - b.y);
        const float orr = 0.5f * (a.y + b.y), oi = -0.5f * (a.x - b.x);
        const float2 w = tw[k];
        const float xr = er + (w.x * orr - w.y * oi), xi = ei + (w.x * oi + w.y * orr);
        spec[(int64_t)t * F + f] = make_float2(xr * dt, xi * dt);
    }
}

// |s~|^2 as every size sums it: the contraction is written out, and sums add it as it is.
__device__ __forceinline__ float power(float2 v)
{
#pragma clang fp contract(off)
    return __builtin_fmaf(v.x, v.x, v.y * v.y);
}

// P'(t; f) = scale * mean |spec(t', f)|^2 over 2 <= |t' - t| <= nb + 1 inside [0, T).
// Grid: (ceil(F / 256), ceil(T / C)); every column has a neighbour (T >= 4, checked by the host). A
// lane sums C columns, and every sum runs over t' in ascending order, so C changes no bit.
// Spectra that stay in the L2s are bound by latency: one column per lane, its neighbours in flight
// together (us for C = 1 and 4 at nb = 4: 2.3 and 3.0 at 100 x 60, 3.9 and 4.5 at 500 x 800, 5.9 and
// 6.4 at 1000 x 1000). Larger ones are bound by the reads: four columns read each neighbour once for
// all of them, 3.5 reads per column instead of 8 (13.7 and 14.2 at 1500 x 2000, 23.7 and 19.4 with
// nb = 8; 24.2 and 19.7 at 1500 x 2660, 35.2 and 24.8 at 1500 x 3840).
template <int C>
__global__ __launch_bounds__(256) void k_psd(const float2 *__restrict__ spec, int T, int F, int nb, float scale,
                                             float *__restrict__ psd)
{
#pragma clang fp contract(off)
    const int f = blockIdx.x * 256 + threadIdx.x;
    const int t0 = blockIdx.y * C;
    if (f >= F) return;
    float acc[C] = {};
    const int lo = max(t0 - nb - 1, 0), hi = min(t0 + C + nb, T - 1);
    if constexpr (C == 1) {
#pragma unroll 4
        for (int u = lo; u <= t0 - 2; ++u) acc[0] += power(spec[(int64_t)u * F + f]);
#pragma unroll 4
        for (int u = t0 + 2; u <= hi; ++u) acc[0] += power(spec[(int64_t)u * F + f]);
    } else {
#pragma unroll 4
        for (int u = lo; u <= hi; ++u) {
            const float q = power(spec[(int64_t)u * F + f]);
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const int d = u > t0 + j ? u - t0 - j : t0 + j - u;
                if (d >= 2 && d <= nb + 1) acc[j] += q;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int t = t0 + j;
        if (t >= T) break;
        const int cnt = max(0, min(nb, t - 1)) + max(0, min(nb, T - 2 - t));
        psd[(int64_t)t * F + f] = scale * acc[j] / (float)cnt;
    }
}

// Order of an XCD's workgroups over the n slides of a launch, `per` of them per slide: runs of
// kFormRun bins (`run` workgroups), every slide's part of a run before the next run. Workgroup b of
// the XCD takes place `at` of its part of slide k.
struct SlideItem {
    uint32_t k, at;
};
constexpr uint32_t kFormRun = 131072;

__host__ __device__ __forceinline__ SlideItem slide_item(uint32_t b, uint32_t per, uint32_t n, uint32_t run)
{
    run = run < per ? run : per;
    const uint32_t base = b / (run * n) * run, size = run < per - base ? run : per - base;
    const uint32_t rem = b - base * n, k = rem / size;
    return {k, base + rem - k * size};
}

// One launch writes up to kSlidesPerLaunch slide maps, one after the other: a workgroup takes 256 P
// consecutive bins of one slide (rows of F bins end to end; P = 2 when F and ld are even and the
// buffers 16-byte aligned: one 16-byte and one 8-byte store per lane), so that the workgroups in
// flight write a map or two front to back. Stores past the caches in that order reach the rate of a
// fill: 256 maps of 1000 x 1000 in 448 us, 6.9 TB/s of the card's 6.9. A workgroup that wrote its
// bins to 16 maps in turn scattered the stores over 16 maps at once (915 us; past the caches 765);
// two slides per workgroup take 511 us, stores through the caches 723. Workgroups go round-robin to
// the 8 XCDs; the remap gives each XCD one contiguous part of every slide, so its I columns, and for
// neighbouring shifts its J columns, stay in its own L2 (shifts in random order: 677 us). 131072 bins
// of both spectra are 3 MB of an L2's 4: a part larger than that is written in runs of so many bins,
// all slides of a run before the next run. Slide by slide, larger spectra come from beyond the L2s
// for every slide again (1500 x 2000, 4 slides: 51 us, in runs 29; 1500 x 3840: 96 and 57, 16 slides
// 376 and 184; runs of 262144 bins 44, 95 and 364, of 65536 28, 57 and 191).
// Stores past the caches leave the maps in memory: one 1000 x 1000 map and a reading pass over it take
// 10.9 us, 10.5 with stores through the caches, 8 maps 50.2 and 51.8, 4 of 1500 x 2000 62.2 and 66.0.
// Grid: 1-D, 8 * ceil(nchunk / 8) * a.n workgroups of 256 lanes, nchunk = ceil(T F / (256 P)).
// RUNS: parts larger than a run (the order's divisions cost 256 maps of 1000 x 1000 4 us of 448).
template <int P, bool RUNS>
__global__ __launch_bounds__(256) void k_form_maps(const float2 *__restrict__ si, const float *__restrict__ pi,
                                                   const float2 *__restrict__ sj, const float *__restrict__ pj,
                                                   int T, int F, float scale, int64_t ld, SlideArgs a)
{
    const uint32_t n = (uint32_t)T * (uint32_t)F;  // < 2^29 (T < 2^16, F <= kMaxFftM / 2)
    const uint32_t nchunk = (n + 256 * P - 1) / (256 * P);
    const uint32_t per = (nchunk + 7) / 8;
    const uint32_t b = blockIdx.x / 8;
    SlideItem w;
    if constexpr (RUNS) {
        w = slide_item(b, per, (uint32_t)a.n, kFormRun / (256 * P));
    } else {
        w.k = b / per;
        w.at = b - w.k * per;
    }
    const uint32_t k = w.k, L = (blockIdx.x % 8) * per + w.at;
    if (L >= nchunk) return;
    const uint32_t i = P * (L * 256 + threadIdx.x);
    if (i >= n) return;
    uint32_t j = i + (uint32_t)a.shift[k] * (uint32_t)F;  // column t + shift, modulo T
    if (j >= n) j -= n;
    typedef float fv __attribute__((ext_vector_type(2 * P)));  // P complex values
    typedef float pv __attribute__((ext_vector_type(P)));      // P powers
    const fv u = *reinterpret_cast<const fv *>(si + i), v = *reinterpret_cast<const fv *>(sj + j);
    const pv pu = *reinterpret_cast<const pv *>(pi + i), pq = *reinterpret_cast<const pv *>(pj + j);
    fv y;
    pv sg;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const float ur = u[2 * q], ui = u[2 * q + 1], vr = v[2 * q], vi = v[2 * q + 1];
        y[2 * q] = scale * (ur * vr + ui * vi);
        y[2 * q + 1] = scale * (ur * vi - ui * vr);
        sg[q] = sqrtf(0.5f * pu[q] * pq[q]);
    }
    const int64_t o = ld == F ? (int64_t)i : (int64_t)(i / (uint32_t)F) * (ld - F) + i;
    __builtin_nontemporal_store(y, reinterpret_cast<fv *>(a.Y[k] + o));
    __builtin_nontemporal_store(sg, reinterpret_cast<pv *>(a.sigma[k] + o));
}

}  // namespace stt
