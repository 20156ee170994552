// kernels.hpp -- the libstt device kernels for gfx950 (wave64, 160 KB LDS per CU).
//
// Hot path of the template search (paper Sec. III, Eq. 6 and Eq. 8):
//   k_make_tracks   materialise templates (Philox4x32-10 + exact unranking)
//   k_bin_count     \  counting sort of templates by (start, end) column bucket,
//   k_bin_scan       | so that a workgroup's templates cover nearly the same
//   k_bin_group      | columns and its lanes stay busy through a time sweep;
//   k_bin_fine      /  scattered in two passes, to groups of buckets, then buckets
//   k_fold_polar    p = Y/sigma of every pixel in polar form (|p|, arg p in
//                   2^-32 turn), the layout the scorers stage: one cosine per term
//   k_score_slab    time-slab scorer: the workgroup copies slabs of consecutive
//                   columns of the folded map into LDS (LDS DMA, double-buffered)
//                   and every lane gathers its templates' pixels there
//   k_score_direct, k_score_wave  one lane or one wave per template, pixels
//                   gathered straight from global memory (small calls, very wide maps)
//   k_reduce_keys   max of the slab scorer's per-workgroup best keys
//   k_argmax        max/argmax of an existing score array
// Reductions use the packed 64-bit key (score bits, ~index), so results do not
// depend on scheduling: wave shuffles, then across the workgroup through LDS
// (slab scorers) or one 64-bit atomic max per wave (small kernels).
#pragma once

#include <hip/hip_fp16.h>

#include "dev_common.hpp"

namespace stt {

struct MapP {
    const float2 *Y;   // [T][ld] complex64 (FP32 map) -- or __half2 p (FP16 map)
    const float *sig;  // [T][ld] sigma (FP32 map only)
    int32_t T, F;
    int64_t ld;
    int32_t fq4_lo, dfq4;
    float scale;       // FP16 map: p = stored * scale (a power of two)
};

// Map element formats: the caller's (Y, sigma) FP32 map; the caller's FP16 map
// (one 32-bit word per pixel: arg p in 2^-16 turn in the low half, |p| * 2^-e
// as binary16 in the high half); p = Y/sigma folded into complex64 by k_fold_p
// (read by the smooth statistic); p folded into polar form by k_fold_polar
// (read by every scorer of Eq. 8 on an FP32 map): |p| as FP32 and arg p as a
// 32-bit fraction of a turn, 8 bytes per pixel; and the FP16 map's words copied
// into the folded layout (read by every scorer on an FP16 map), 4 bytes per
// pixel. Folded maps pad columns to whole 1 KB pieces (128 or 256 pixels) so
// that slabs can be copied into LDS by 1 KB LDS-DMA instructions.
enum : int { kMapF32 = 0, kMapP16 = 1, kMapPF = 2, kMapPol = 3, kMapPolH = 4 };
constexpr int kDmaBytes = 1024;  // bytes one wave moves per LDS-DMA instruction (64 lanes x 16 B)

// Element type of a map format in registers and LDS.
template <int MAPT> struct ElemOf { using type = float2; };
template <> struct ElemOf<kMapPolH> { using type = uint32_t; };
template <int MAPT> using elem_t = typename ElemOf<MAPT>::type;
template <int MAPT> constexpr int kDmaPix = kDmaBytes / (int)sizeof(elem_t<MAPT>);  // pixels per 1 KB piece

// binary16 bits of the high half of a word, as FP32 (exact)
__device__ __forceinline__ float half_hi(uint32_t w)
{
    return __half2float(__ushort_as_half((unsigned short)(w >> 16)));
}

// The complex SNR p = Y/sigma of pixel element e (Eq. 7 with the appendix's rho = Y/sigma).
// FP16 map: |p| 2^e exp(2 pi i arg) evaluated in FP64 and rounded once per component.
template <int MAPT>
__device__ __forceinline__ float2 load_p(const MapP &m, int64_t e)
{
    if constexpr (MAPT == kMapP16) {
        const uint32_t w = reinterpret_cast<const uint32_t *>(m.Y)[e];
        const double mag = (double)half_hi(w) * (double)m.scale;
        double sn, cs;
        sincospi((double)(w & 0xFFFFu) * (1.0 / 32768.0), &sn, &cs);
        return make_float2((float)(mag * cs), (float)(mag * sn));
    } else if constexpr (MAPT == kMapPF || MAPT == kMapPol) {
        return m.Y[e];  // (a polar map's element is returned as stored)
    } else {
        const float2 y = m.Y[e];
        const float w = 1.0f / m.sig[e];
        return make_float2(y.x * w, y.y * w);
    }
}

// One element of a map as its scorers hold it: a word of a folded FP16 map, p otherwise.
template <int MAPT>
__device__ __forceinline__ elem_t<MAPT> load_e(const MapP &m, int64_t e)
{
    if constexpr (MAPT == kMapPolH) return reinterpret_cast<const uint32_t *>(m.Y)[e];
    else return load_p<MAPT>(m, e);
}

// p of every pixel into a complex64 map with column stride ld_out (pixels
// F..ld_out-1 of a column are zero): Y/sigma of an FP32 map, or the exact FP32
// value of an FP16 map's entry. The same expression as load_p's, so scores do
// not depend on whether the map was folded first.
template <int MAPT>
__global__ __launch_bounds__(256) void k_fold_p(MapP m, float2 *out, int64_t ld_out)
{
    const int64_t n = (int64_t)m.T * ld_out;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t t = i / ld_out, r = i - t * ld_out;
        out[i] = r < m.F ? load_p<MAPT>(m, t * m.ld + r) : make_float2(0.0f, 0.0f);
    }
}

// arg (x + iy) as a 32-bit fraction of a turn, from FP32 components. The first
// octant's angle atan(a), a = min(|x|, |y|) / max(|x|, |y|), is reduced to
// |t| <= tan(pi/8) (atan(a) = pi/4 + atan((a - 1)/(a + 1)) above), evaluated as
// atan(t)/(2 pi) = t P(t^2) in FP32 (coefficients from gen_atan_coeffs.py) and
// rounded to 2^-32 turn; the octant and quadrant are then undone in integers
// (eighths of a turn are exact). The polynomial in FP32 is within 41 units of
// 2^-32 turn; with the FP32 division and reduction about 100 units (2.3e-8
// turn) in all -- well below the 2^-24-turn rounding of the phase each term
// takes before its cosine. arg 0 = 0 (its magnitude is 0 then).
__device__ __forceinline__ uint32_t arg_turns(float x, float y)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const bool swap = ay > ax;  // the angle from the nearer axis is atan(min/max)
    const float num = swap ? ax : ay, den = swap ? ay : ax;
    const float a = den > 0.0f ? num / den : 0.0f;
    const bool hi = a > 0.41421356f;
    const float t = hi ? (a - 1.0f) / (a + 1.0f) : a;
    const float s = t * t;
    float q = -9.602202103e-03f;
    q = fmaf(q, s, 1.682715677e-02f);
    q = fmaf(q, s, -2.266363613e-02f);
    q = fmaf(q, s, 3.182814270e-02f);
    q = fmaf(q, s, -5.305160582e-02f);
    q = fmaf(q, s, 1.591549367e-01f);
    const int32_t f = (int32_t)rintf(t * q * 4294967296.0f);  // |t q| <= 1/16 turn
    uint32_t u = (uint32_t)((hi ? (1 << 29) : 0) + f);        // first-octant angle
    if (swap) u = (1u << 30) - u;                               // first quadrant
    if (x < 0.0f) u = (1u << 31) - u;                           // second quadrant
    if (y < 0.0f) u = 0u - u;                                   // lower half, modulo one turn
    return u;
}

// Polar form of p: (|p| rounded to FP32, arg p in 2^-32 turn as the bits of the second word).
// The FP32 components square exactly in FP64, so |p|^2 = x^2 + y^2 is rounded once, its square
// root once more and the result once to FP32.
__device__ __forceinline__ float2 polar_of(float2 p)
{
    const double x = p.x, y = p.y;
    const float mag = (float)sqrt(fma(x, x, y * y));
    return make_float2(mag, __uint_as_float(arg_turns(p.x, p.y)));
}

constexpr int kFoldRows = 4;  // rows per thread of the fold kernels: all their loads in flight at once

// Column t, rows r0 + 256 i + threadIdx.x (i < kFoldRows) of a fold: every load first, then the
// polar forms and stores (pixels F .. ld_out-1 zero).
template <int MAPT>
__device__ __forceinline__ void fold_rows(const MapP &m, int64_t t, int64_t r0, float2 *out, int64_t ld_out)
{
    float2 p[kFoldRows];
#pragma unroll
    for (int i = 0; i < kFoldRows; ++i) {
        const int64_t r = r0 + i * 256 + threadIdx.x;
        p[i] = r < m.F ? load_p<MAPT>(m, t * m.ld + r) : make_float2(0.0f, 0.0f);
    }
#pragma unroll
    for (int i = 0; i < kFoldRows; ++i) {
        const int64_t r = r0 + i * 256 + threadIdx.x;
        if (r < ld_out) out[t * ld_out + r] = r < m.F ? polar_of(p[i]) : make_float2(0.0f, 0.0f);
    }
}

// The same rows of an FP16 map: its words as they are.
__device__ __forceinline__ void fold_words_rows(const MapP &m, int64_t t, int64_t r0, uint32_t *out, int64_t ld_out)
{
    const uint32_t *w = reinterpret_cast<const uint32_t *>(m.Y);
    uint32_t v[kFoldRows];
#pragma unroll
    for (int i = 0; i < kFoldRows; ++i) {
        const int64_t r = r0 + i * 256 + threadIdx.x;
        v[i] = r < m.F ? w[t * m.ld + r] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kFoldRows; ++i) {
        const int64_t r = r0 + i * 256 + threadIdx.x;
        if (r < ld_out) out[t * ld_out + r] = v[i];
    }
}

// p of every pixel in polar form into a map with column stride ld_out (pixels F..ld_out-1 of a
// column are zero): from Y/sigma of an FP32 map, or from the exact FP32 values of an FP16 map's
// entries (load_p's expression). Grid: column blockIdx.x, y strides over its rows.
template <int MAPT>
__global__ __launch_bounds__(256) void k_fold_polar(MapP m, float2 *out, int64_t ld_out)
{
    for (int64_t r0 = (int64_t)blockIdx.y * 256 * kFoldRows; r0 < ld_out; r0 += (int64_t)gridDim.y * 256 * kFoldRows)
        fold_rows<MAPT>(m, blockIdx.x, r0, out, ld_out);
}

// The words of an FP16 map into the folded layout (column stride ld_out, pixels F..ld_out-1 zero).
// Grid: column blockIdx.x, y strides over its rows.
__global__ __launch_bounds__(256) void k_fold_words(MapP m, uint32_t *out, int64_t ld_out)
{
    for (int64_t r0 = (int64_t)blockIdx.y * 256 * kFoldRows; r0 < ld_out; r0 += (int64_t)gridDim.y * 256 * kFoldRows)
        fold_words_rows(m, blockIdx.x, r0, out, ld_out);
}

// One fold of a batch: map src into dst (column stride ld_out); its columns are col0 .. col0 +
// T - 1 of the batch's column run (col0 ascending over the maps).
struct FoldJob {
    MapP src;
    void *dst;
    int64_t ld_out;
    uint32_t col0;
};

// Every map of a batch in one launch: blockIdx.x runs over the batch's columns, each workgroup
// finds its map once by bisection of col0 (jobs[n_jobs].col0 = the total), y strides over rows.
// FP32 maps fold to polar form (k_fold_polar), FP16 maps copy their words (k_fold_words).
template <int MAPT>
__global__ __launch_bounds__(256) void k_fold_batch(const FoldJob *jobs, int n_jobs)
{
    const uint32_t col = blockIdx.x;
    int lo = 0, hi = n_jobs;  // jobs[lo].col0 <= col < jobs[hi].col0
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (jobs[mid].col0 <= col) lo = mid; else hi = mid;
    }
    const FoldJob &j = jobs[lo];
    const int64_t t = (int64_t)(col - j.col0);
    for (int64_t r0 = (int64_t)blockIdx.y * 256 * kFoldRows; r0 < j.ld_out; r0 += (int64_t)gridDim.y * 256 * kFoldRows) {
        if constexpr (MAPT == kMapP16)
            fold_words_rows(j.src, t, r0, (uint32_t *)j.dst, j.ld_out);
        else
            fold_rows<MAPT>(j.src, t, r0, (float2 *)j.dst, j.ld_out);
    }
}

constexpr int kMaxDt = 2895;  // Dt * Dt * 256 < 2^31
// FP32 partial sums are flushed into the FP64 total after every column c with
// c % kFlush == kFlush - 1: a fixed grid of absolute columns, so a template's
// arithmetic does not depend on which workgroup or scorer handles it.
constexpr int kFlush = 16;
constexpr int kWG = 256;      // threads per workgroup of the scorers

__device__ __forceinline__ bool track_ok(const Trk &t, const MapP &m)
{
    const uint32_t frange = (uint32_t)m.F << 8;
    return t.t0 >= 0 && t.t2 < m.T && t.t2 > t.t0 && t.t2 - t.t0 <= kMaxDt && t.f0 < frange &&
           t.f1 < frange && t.f2 < frange;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}

// Wave-wide min/max, returned as a wave-uniform (scalar) value so that loop
// bounds and addresses derived from it stay off the vector ALU.
__device__ __forceinline__ int wave_min_i32(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off));
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ int wave_max_i32(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off));
    return __builtin_amdgcn_readfirstlane(v);
}

// Max of the keys of a workgroup of 256 lanes into *best: waves by shuffles, the four waves
// through LDS, one atomic per workgroup. (Atomics on one address complete one after the other,
// 11 ns each on gfx950: with one per wave, calls of one template per wave took 11.4 ns per template.)
__device__ __forceinline__ void merge_key(uint64_t *best, uint64_t key)
{
    __shared__ uint64_t kmax[4];
    if (!best) return;  // uniform over the launch
    key = wave_max_u64(key);
    if ((threadIdx.x & 63) == 0) kmax[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) key = kmax[w] > key ? kmax[w] : key;
        if (key) atomicMax((unsigned long long *)best, (unsigned long long)key);
    }
}

// z of a template from its FP64 sum S of terms in units of `scale` (2^e of an FP16 map, else 1).
__device__ __forceinline__ float finish(double S, int32_t N, int32_t norm, float scale)
{
    S *= (double)scale;
    return (float)(norm == 1 ? S / (double)N : S / sqrt((double)N));
}

// Phase constants of one template: its Eq. 8 phase at row r is pa + r*pb in
// units of 2^-32 turn, exact with 32-bit wrap-around.
struct PhaseK {
    uint32_t pa, pb;
};

__device__ __forceinline__ PhaseK phase_k(const MapP &m, int32_t dtau)
{
    return PhaseK{phase_a(m.fq4_lo, dtau), phase_b(m.dfq4, dtau)};
}

// part + Re[exp(2 pi i phase(row)) p], the template's Eq. 8 term at this row.
// HW: the exact 32-bit phase rounded once to FP32 turns (phase_turns) feeds
// the hardware sine and cosine, which take turns; measured on gfx950 over 2^22
// phases spanning a turn: at most 1.25e-7 absolute error, rms 3.5e-8, no bias.
// The two products are added to the running sum by fused multiply-adds.
// HW = false: the polynomial of rot_re (about 1.5e-7 absolute).
template <bool HW>
__device__ __forceinline__ float add_term(float part, const PhaseK &k, int32_t row, float2 p)
{
    if constexpr (HW) {
        const float x = phase_turns(k.pa, k.pb, row);
        part = fmaf(__builtin_amdgcn_cosf(x), p.x, part);
        return fmaf(-__builtin_amdgcn_sinf(x), p.y, part);
    } else {
        return part + rot_re(k.pa + (uint32_t)row * k.pb, p.x, p.y);
    }
}

// The same term from the polar form (|p|, arg p): Re[exp(2 pi i phase) p] = |p| cos(2 pi (phase +
// arg p)). The two phases add exactly in 32-bit turns, so one cosine and one fused multiply-add
// replace the sine, the cosine and the two products of the Cartesian form. HW: the hardware cosine
// of the sum rounded once to FP32 turns; HW = false: the polynomial of rot_re.
// Polar elements: (|p|, arg p) of an FP32 map's fold, or an FP16 map's word (|p| 2^-e and arg p
// in 2^-16 turn, which shifted left by 16 is the same 32-bit fraction of a turn, exactly).
__device__ __forceinline__ float pol_mag(float2 v) { return v.x; }
__device__ __forceinline__ uint32_t pol_arg(float2 v) { return __float_as_uint(v.y); }
__device__ __forceinline__ float pol_mag(uint32_t w) { return half_hi(w); }
__device__ __forceinline__ uint32_t pol_arg(uint32_t w) { return w << 16; }

template <bool HW, typename E>
__device__ __forceinline__ float add_term_pol(float part, const PhaseK &k, int32_t row, E v)
{
    const uint32_t arg = pol_arg(v);
    if constexpr (HW) {
        const float x = phase_turns(k.pa + arg, k.pb, row);
        return fmaf(__builtin_amdgcn_cosf(x), pol_mag(v), part);
    } else {
        return part + rot_re(k.pa + arg + (uint32_t)row * k.pb, pol_mag(v), 0.0f);
    }
}

// The Eq. 8 term of one pixel element of map format MAPT (polar or Cartesian).
template <bool HW, int MAPT>
__device__ __forceinline__ float add_term_m(float part, const PhaseK &k, int32_t row, elem_t<MAPT> v)
{
    if constexpr (MAPT == kMapPol || MAPT == kMapPolH) return add_term_pol<HW>(part, k, row, v);
    else return add_term<HW>(part, k, row, v);
}

// A fill kernel rather than a memset node, so that captured graphs replay it faithfully.
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------- generation

__global__ __launch_bounds__(256) void k_make_tracks(GenP g, uint64_t first, int64_t n, Trk *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = draw_track(g, first + (uint64_t)i);
}

// ---------------------------------------------------------------- direct scorers
// Calls too small for the slab scorer, and maps too wide for it: pixels gathered straight from
// global memory. Both scorers walk a template by flush groups (kFlush aligned columns): all rows of
// a group first, then its 16 gathers, all in flight at once, then its terms in column order, so a
// template costs one memory latency per group instead of one per column (search map, 20 000
// templates: 297 us with a gather at a time). Columns of a group outside the template gather the
// template's first pixel's column and drop the term.

// Element e of the map a direct scorer reads, in the polar form of its terms: a folded map, an FP16
// map's own words, or an FP32 map folded here (the expression of k_fold_polar, so the same bits).
template <int MAPT> struct PolOf { using type = float2; };
template <> struct PolOf<kMapPolH> { using type = uint32_t; };
template <> struct PolOf<kMapP16> { using type = uint32_t; };
template <int MAPT> using pol_t = typename PolOf<MAPT>::type;

template <int MAPT>
__device__ __forceinline__ pol_t<MAPT> load_pol(const MapP &m, int64_t e)
{
    if constexpr (MAPT == kMapPolH || MAPT == kMapP16) return reinterpret_cast<const uint32_t *>(m.Y)[e];
    else if constexpr (MAPT == kMapF32) return polar_of(load_p<kMapF32>(m, e));
    else return m.Y[e];
}

// The FP32 sum of a template's terms over the flush group that starts at column cb (a multiple of
// kFlush), for a row walk st standing at cb; st is advanced past the group. t0 .. t2: its columns.
// G gathers at a time are in flight (the sums are the same for every G).
template <bool HW, int MAPT, int G = kFlush>
__device__ __forceinline__ float group_sum(const MapP &m, const PhaseK &pk, int32_t cb, int32_t t0, int32_t t2, DdaF &st)
{
    float part = 0.0f;
#pragma unroll
    for (int j0 = 0; j0 < kFlush; j0 += G) {
        int32_t row[G];
        pol_t<MAPT> v[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = cb + j0 + j;
            const bool act = c >= t0 && c <= t2;
            row[j] = act ? ddaf_row(st) : 0;
            v[j] = load_pol<MAPT>(m, (int64_t)(act ? c : t0) * m.ld + row[j]);
            ddaf_step(st);
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = cb + j0 + j;
            const float p = add_term_pol<HW>(part, pk, row[j], v[j]);
            part = c >= t0 && c <= t2 ? p : part;
        }
        if (G < kFlush) __builtin_amdgcn_sched_barrier(0);
    }
    return part;
}

// One lane per template. G: a flush group's gathers at a time, or one at a time where many lanes walk a
// map larger than an L2 (lane_gathers).
template <bool EXPL, bool HW, int MAPT, int G>
__global__ __launch_bounds__(kWG) void k_score_direct(MapP m, GenP g, const Trk *tr, uint64_t first, int64_t n,
                                                      int32_t norm, float *snr, uint64_t *best)
{
    const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
    uint64_t key = 0;
    if (i < n) {
        const Trk t = EXPL ? tr[i] : draw_track(g, first + (uint64_t)i);
        float z = __builtin_nanf("");
        if (!EXPL || track_ok(t, m)) {
            const PhaseK pk = phase_k(m, t.dtau);
            int32_t cb = t.t0 & ~(kFlush - 1);
            DdaF st = ddaf_init_at(t, cb - t.t0);
            double acc = 0.0;
            for (; cb <= t.t2; cb += kFlush) acc += group_sum<HW, MAPT, G>(m, pk, cb, t.t0, t.t2, st);
            z = finish(acc, t.t2 - t.t0 + 1, norm, m.scale);
        }
        if (snr) snr[i] = z;
        key = key_encode(z, (uint32_t)(first + (uint64_t)i));
    }
    merge_key(best, key);
}

// One wave per template, for calls too small to fill the chip with one lane
// per template: lane l takes the template's groups l, l + 64, ... The FP64 sum
// over groups runs in column order (read lane by lane), so the score is
// bit-identical to the other scorers'. Four waves (templates at a time) per
// workgroup, which strides over the templates.
constexpr int kWaveGroups = (STT_MAX_T + kFlush - 1) / kFlush + 1;  // groups a template can touch
constexpr int kWaveRounds = (kWaveGroups + 63) / 64;

// The sum in order of gp[r] of lanes 0 .. over rounds r: ng group sums.
__device__ __forceinline__ double wave_ordered_sum(const float (&gp)[kWaveRounds], int ng)
{
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < kWaveRounds; ++r) {
        const int cnt = min(64, ng - r * 64);
        for (int l = 0; l < cnt; ++l)
            acc += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gp[r]), l));
    }
    return acc;
}

template <bool EXPL, bool HW, int MAPT>
__global__ __launch_bounds__(256) void k_score_wave(MapP m, GenP g, const Trk *tr, uint64_t first, int64_t n,
                                                    int32_t norm, float *snr, uint64_t *best)
{
    const int lane = threadIdx.x & 63;
    uint64_t key = 0;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {  // wave-uniform
        const Trk t = EXPL ? tr[i] : draw_track(g, first + (uint64_t)i);
        float z = __builtin_nanf("");
        if (!EXPL || track_ok(t, m)) {
            const PhaseK pk = phase_k(m, t.dtau);
            const int gfirst = t.t0 / kFlush, glast = t.t2 / kFlush;
            float gp[kWaveRounds];
#pragma unroll
            for (int r = 0; r < kWaveRounds; ++r) {
                gp[r] = 0.0f;
                const int gi = gfirst + r * 64 + lane;
                if (gi > glast) continue;
                DdaF st = ddaf_init_at(t, gi * kFlush - t.t0);
                gp[r] = group_sum<HW, MAPT>(m, pk, gi * kFlush, t.t0, t.t2, st);
            }
            z = finish(wave_ordered_sum(gp, glast - gfirst + 1), t.t2 - t.t0 + 1, norm, m.scale);
        }
        if (lane == 0 && snr) snr[i] = z;
        const uint64_t k = key_encode(z, (uint32_t)(first + (uint64_t)i));
        key = k > key ? k : key;
    }
    merge_key(best, key);
}

// ---------------------------------------------------------------- argmax of an array

__global__ __launch_bounds__(256) void k_argmax(const float *z, int64_t n, uint64_t first, uint64_t *best)
{
    uint64_t key = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const uint64_t k = key_encode(z[i], (uint32_t)(first + (uint64_t)i));
        key = k > key ? k : key;
    }
    merge_key(best, key);
}

// ---------------------------------------------------------------- binning by time extent
// Bucket of a template: b0 = t0 >> wb, b2 = t2 >> wb (b0 <= b2), nb buckets
// per axis, numbered by bucket_number: four classes of extents, longest first,
// and by start within a class. Blocks of binned templates are dispatched in
// that order. Blocks that run together then stage the same columns: on the
// search map (1000 x 1000, 10^7 templates, 512 x 4 workgroups) the scorer takes
// 1.39 ms; numbered by extent alone, 1.69 ms (classes of 20, 24, 42, 48 and 64
// of the 126 extents: 1.59, 1.55, 1.42, 1.43, 1.46). Invalid given templates go
// to bucket 0 (they are skipped when scored).
//
// The sort: count, scans, two scatters. Buckets form groups of 2^kGroupShift
// consecutive ones. The count (one workgroup per chunk of kBinChunk templates)
// draws each template's bucket once and keeps it (2 bytes, in the space the
// binned order fills last), adds its chunk's bucket histogram to the totals
// and writes the chunk's count per group. The scans give every bucket its
// start, every group its region and every chunk its run in each group. The
// first scatter moves each index, with its bucket within the group, to its
// chunk's run in its group's region (no cursor atomics: the place of every run
// is known). The second takes each group's region in chunks of kFineChunk and
// moves each index to its bucket, the runs reserved by atomics on the bucket
// cursors. Each scatter workgroup first orders its chunk by key in LDS, then
// stores it run by run: consecutive lanes write consecutive addresses, so a
// store instruction touches one or two cache lines (a single scatter into all
// buckets would store about one index per bucket per workgroup: one cache
// line per lane).

constexpr int kBinPerThread = 32;                 // templates per thread of the count (256 lanes)
constexpr int kBinChunk = 256 * kBinPerThread;    // templates per sort chunk: count, first scatter
constexpr int kFineChunk = 4096;                  // templates per chunk of the second scatter
constexpr int kScatterWG = 512;                   // lanes of a scatter workgroup
constexpr int kMaxBins = 128 * 129 / 2;           // at most 128 buckets per axis
constexpr int kGroupShift = 6;                    // buckets per group: 64
constexpr int kGroupMask = (1 << kGroupShift) - 1;
constexpr int kMaxGroups = (kMaxBins + kGroupMask) >> kGroupShift;
constexpr int kGroupSlots = kMaxGroups + 1 + (kMaxGroups & 1 ? 0 : 1);  // groups + 1 entries, an even count
static_assert(kMaxGroups << kGroupShift == kMaxBins, "bucket tables are whole groups");
static_assert(kMaxGroups <= 3 * 64, "one wave scans the group table");

// The slot of item in a table of ascending starts: start[k] <= item < start[k + 1], 0 <= k < n.
__device__ __forceinline__ int find_slot(const uint32_t *start, int n, uint32_t item)
{
    int lo = 0, hi = n;  // start[lo] <= item < start[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= item) lo = mid; else hi = mid;
    }
    return lo;
}

// Exclusive prefix sums by one wave (the caller's lanes 0..63) of val(0 .. cnt-1),
// cnt <= 192: out[k] = val(0) + ... + val(k-1), out[cnt] = the total.
template <typename F>
__device__ __forceinline__ void wave_prefix(F val, int cnt, uint32_t *out)
{
    const int lane = threadIdx.x & 63;
    uint32_t v[3], s = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int k = 3 * lane + j;
        v[j] = k < cnt ? val(k) : 0u;
        s += v[j];
    }
    uint32_t incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    uint32_t run = incl - s;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int k = 3 * lane + j;
        if (k < cnt) out[k] = run;
        run += v[j];
    }
    if (lane == 63) out[cnt] = incl;
}

template <bool EXPL>
__device__ __forceinline__ uint32_t bin_of(const GenP &g, const Trk *tr, const MapP &m, uint64_t first, int64_t i,
                                           int wb, uint32_t cw)
{
    int32_t t0, t2;
    if (EXPL) {
        const Trk t = tr[i];
        if (!track_ok(t, m)) return 0;
        t0 = t.t0;
        t2 = t.t2;
    } else {
        draw_extent(g, first + (uint64_t)i, t0, t2);
    }
    const uint32_t b0 = (uint32_t)t0 >> wb, b2 = (uint32_t)t2 >> wb;
    const uint32_t nb = ((uint32_t)(m.T - 1) >> wb) + 1;
    return bucket_number(nb - 1 - (b2 - b0), b0, cw, nb);
}

// The count's step for one chunk, after its histogram hist[0 .. nbins-1] is
// complete in LDS: totals[b] += hist[b], and ccnt[k * stride] = the chunk's
// templates in group k (a thread per group; thread k starts its sum at bucket
// k mod 64 of the group, so the lanes of a wave read 64 different banks).
__device__ __forceinline__ void count_out(const uint32_t *hist, int nbins, uint32_t *totals, uint32_t *ccnt,
                                          size_t stride)
{
    for (int b = threadIdx.x; b < nbins; b += 256)
        if (hist[b]) atomicAdd(&totals[b], hist[b]);
    const int ngroups = (nbins + kGroupMask) >> kGroupShift;
    for (int k = threadIdx.x; k < ngroups; k += 256) {
        const int b0 = k << kGroupShift, nb = min(1 << kGroupShift, nbins - b0);
        uint32_t v = 0;
#pragma unroll 8
        for (int i = 0; i <= kGroupMask; ++i) {
            const int j = (i + k) & kGroupMask;
            if (j < nb) v += hist[b0 + j];
        }
        ccnt[(size_t)k * stride] = v;
    }
}

// Count: bins[i] = the bucket of template i; count_out for workgroup (chunk) c
// at ccnt + c with stride gridDim.x (row k of ccnt: group k's count per chunk).
template <bool EXPL>
__global__ __launch_bounds__(256) void k_bin_count(MapP m, GenP g, const Trk *tr, uint64_t first, int64_t n, int wb,
                                                   uint32_t cw, int nbins, uint32_t *totals, uint16_t *bins,
                                                   uint32_t *ccnt)
{
    __shared__ uint32_t hist[kMaxBins];
    for (int b = threadIdx.x; b < nbins; b += 256) hist[b] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kBinChunk;
    for (int q = 0; q < kBinPerThread; ++q) {
        const int64_t i = base + q * 256 + threadIdx.x;
        if (i < n) {
            const uint32_t b = bin_of<EXPL>(g, tr, m, first, i, wb, cw);
            bins[i] = (uint16_t)b;
            atomicAdd(&hist[b], 1u);
        }
    }
    __syncthreads();
    count_out(hist, nbins, totals, ccnt + blockIdx.x, gridDim.x);
}

// The bucket scan of one call or map by NT threads (nbins <= kMaxBins):
// cursor[b] = base + the templates in buckets before b; gstart[k] = cursor of
// group k's first bucket, gstart[ngroups] = base + all; fitem[k] = the first
// second-scatter chunk of group k, fitem[ngroups] = their count.
template <int NT>
__device__ __forceinline__ void scan_buckets(const uint32_t *totals, int nbins, uint32_t base, uint32_t *cursor,
                                             uint32_t *gstart, uint32_t *fitem)
{
    constexpr int kPer = (kMaxBins + NT - 1) / NT;
    __shared__ uint32_t wsum[NT / 64];
    __shared__ uint32_t gs[kGroupSlots];
    const int per = (nbins + NT - 1) / NT;
    const int lo = threadIdx.x * per;
    uint32_t v[kPer], s = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int b = lo + j;
        v[j] = j < per && b < nbins ? totals[b] : 0u;
        s += v[j];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t run = base + incl - s;
    for (int w = 0; w < wv; ++w) run += wsum[w];
    const int ngroups = (nbins + kGroupMask) >> kGroupShift;
    if (threadIdx.x == NT - 1) gs[ngroups] = run + s;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int b = lo + j;
        if (j < per && b < nbins) {
            if (!(b & kGroupMask)) gs[b >> kGroupShift] = run;
            cursor[b] = run;
            run += v[j];
        }
    }
    __syncthreads();
    if ((int)threadIdx.x <= ngroups) gstart[threadIdx.x] = gs[threadIdx.x];
    if (threadIdx.x < 64)
        wave_prefix([&](int k) { return (gs[k + 1] - gs[k] + (uint32_t)kFineChunk - 1) / (uint32_t)kFineChunk; }, ngroups,
                    fitem);
}

// Exclusive scan, in place, of row[0 .. len-1] by one workgroup of 256 threads.
__device__ __forceinline__ void scan_row(uint32_t *row, int len)
{
    __shared__ uint32_t wsum[4];
    uint32_t carry = 0;
    for (int t0 = 0; t0 < len; t0 += 1024) {
        const int lo = t0 + 4 * (int)threadIdx.x;
        uint32_t v[4], s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = lo + j < len ? row[lo + j] : 0u;
            s += v[j];
        }
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        uint32_t incl = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t run = carry + incl - s;
        for (int w = 0; w < wv; ++w) run += wsum[w];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (lo + j < len) {
                row[lo + j] = run;
                run += v[j];
            }
        carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
}

// The scans of one call: workgroup 0 scans the buckets (scan_buckets), and
// workgroup k + 1 scans row k of ccnt (nchunks long), which becomes the offset
// of each chunk's run within group k's region.
__global__ __launch_bounds__(256) void k_bin_scan(const uint32_t *totals, int nbins, uint32_t *cursor, uint32_t *gstart,
                                                  uint32_t *fitem, uint32_t *ccnt, int nchunks)
{
    if (blockIdx.x == 0)
        scan_buckets<256>(totals, nbins, 0u, cursor, gstart, fitem);
    else
        scan_row(ccnt + (size_t)(blockIdx.x - 1) * nchunks, nchunks);
}

// The common steps of both scatters, for one chunk of count <= NT * PER
// templates: element q of a thread (present when q*NT + threadIdx.x < count)
// has value kv[q] < 2^16 whose key is kv[q] >> shift (< nkeys <= kMaxGroups).
// Ranks the elements within their keys (kv[q] gets its rank in the high half),
// sets lst[k] = the first position of key k in the chunk ordered by key, and
// cnt[k] = start(k, c) for each key k present c times: the global start of the
// chunk's run of key k. Called by all NT threads; cnt is read back only after
// a later barrier.
template <int PER, typename StartF, int NT>
__device__ __forceinline__ void rank_chunk(uint32_t *cnt, uint32_t *lst, int nkeys, int count, uint32_t (&kv)[PER],
                                           int shift, StartF start)
{
    for (int b = threadIdx.x; b < nkeys; b += NT) cnt[b] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + (int)threadIdx.x < count) kv[q] |= atomicAdd(&cnt[kv[q] >> shift], 1u) << 16;
    __syncthreads();
    if (threadIdx.x < 64) wave_prefix([&](int k) { return cnt[k]; }, nkeys, lst);
    __syncthreads();
    static_assert(kMaxGroups <= 256, "one key per thread");
    if ((int)threadIdx.x < nkeys) {
        const uint32_t c = cnt[threadIdx.x];
        if (c) cnt[threadIdx.x] = start((int)threadIdx.x, c);
    }
}

// LDS of a first-scatter workgroup: the chunk ordered by group, each entry
// (position in the chunk << 16) | bucket.
struct GroupLds {
    uint32_t cnt[kGroupSlots];
    uint32_t lst[kGroupSlots];
    uint32_t sval[kBinChunk];
};

// LDS of a second-scatter workgroup: the chunk ordered by bucket (index and
// bucket within the group).
struct FineLds {
    uint32_t cnt[kGroupSlots];
    uint32_t lst[kGroupSlots];
    uint32_t sidx[kFineChunk];
    uint8_t skey[kFineChunk];
};

// First scatter of chunk c: templates base + j (j < count), buckets bins[base
// + j], to tmp at gstart[k] + crun[k * stride] (group k's region, this chunk's
// run in it) in the order of their ranks; the bucket within the group to tsub
// at the same position.
template <int NT>
__device__ __forceinline__ void group_chunk(GroupLds &L, int ngroups, int64_t base, int count, const uint16_t *bins,
                                            const uint32_t *gstart, const uint32_t *crun, size_t stride, uint32_t *tmp,
                                            uint8_t *tsub)
{
    constexpr int PER = kBinChunk / NT;
    uint32_t kv[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = q * NT + threadIdx.x;
        kv[q] = j < count ? bins[base + j] : 0u;
    }
    auto st = [&](int k, uint32_t) { return gstart[k] + crun[(size_t)k * stride]; };
    rank_chunk<PER, decltype(st), NT>(L.cnt, L.lst, ngroups, count, kv, kGroupShift, st);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = q * NT + threadIdx.x;
        if (j < count) {
            const uint32_t b = kv[q] & 0xffffu;
            L.sval[L.lst[b >> kGroupShift] + (kv[q] >> 16)] = ((uint32_t)j << 16) | b;
        }
    }
    __syncthreads();
    for (int p = threadIdx.x; p < count; p += NT) {
        const uint32_t v = L.sval[p], b = v & 0xffffu, k = b >> kGroupShift;
        const uint32_t at = L.cnt[k] + ((uint32_t)p - L.lst[k]);
        tmp[at] = (uint32_t)(base + (v >> 16));
        tsub[at] = (uint8_t)(b & kGroupMask);
    }
}

// Second scatter of one chunk: entries src[j] (index) and ssub[j] (bucket
// within the group), j < count, to order at their bucket's cursor cur[sub].
template <int NT>
__device__ __forceinline__ void fine_chunk(FineLds &L, int nkeys, int count, const uint32_t *src, const uint8_t *ssub,
                                           uint32_t *cur, uint32_t *order)
{
    constexpr int PER = kFineChunk / NT;
    uint32_t idx[PER], kv[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = q * NT + threadIdx.x;
        idx[q] = j < count ? src[j] : 0u;
        kv[q] = j < count ? ssub[j] : 0u;
    }
    auto st = [&](int k, uint32_t c) { return atomicAdd(&cur[k], c); };
    rank_chunk<PER, decltype(st), NT>(L.cnt, L.lst, nkeys, count, kv, 0, st);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + (int)threadIdx.x < count) {
            const uint32_t k = kv[q] & 0xffffu, p = L.lst[k] + (kv[q] >> 16);
            L.sidx[p] = idx[q];
            L.skey[p] = (uint8_t)k;
        }
    __syncthreads();
    for (int p = threadIdx.x; p < count; p += NT) {
        const uint32_t k = L.skey[p];
        order[L.cnt[k] + ((uint32_t)p - L.lst[k])] = L.sidx[p];
    }
}

// First scatter: workgroup c takes the chunk of templates c * kBinChunk .. of
// the call (ccnt as scanned by k_bin_scan, row stride gridDim.x).
__global__ __launch_bounds__(kScatterWG) void k_bin_group(int64_t n, int ngroups, const uint16_t *bins, const uint32_t *gstart,
                                                   const uint32_t *ccnt, uint32_t *tmp, uint8_t *tsub)
{
    __shared__ GroupLds L;
    const int64_t base = (int64_t)blockIdx.x * kBinChunk;
    group_chunk<kScatterWG>(L, ngroups, base, (int)min<int64_t>(kBinChunk, n - base), bins, gstart, ccnt + blockIdx.x, gridDim.x,
                tmp, tsub);
}

// Second scatter: workgroup w takes chunk w - fitem[k] (of kFineChunk) of group
// k's region of tmp (fitem[k] <= w < fitem[k + 1]) to the group's buckets;
// workgroups from fitem[ngroups] on have nothing to do.
__global__ __launch_bounds__(kScatterWG) void k_bin_fine(int nbins, const uint32_t *gstart, const uint32_t *fitem,
                                                  uint32_t *cursor, const uint32_t *tmp, const uint8_t *tsub,
                                                  uint32_t *order)
{
    __shared__ FineLds L;
    const int ngroups = (nbins + kGroupMask) >> kGroupShift;
    const uint32_t w = blockIdx.x;
    if (w >= fitem[ngroups]) return;
    const int k = find_slot(fitem, ngroups, w);
    const uint32_t e0 = gstart[k] + (w - fitem[k]) * (uint32_t)kFineChunk;
    const int b0 = k << kGroupShift;
    fine_chunk<kScatterWG>(L, min(1 << kGroupShift, nbins - b0), (int)min<uint32_t>(kFineChunk, gstart[k + 1] - e0), tmp + e0,
               tsub + e0, cursor + b0, order);
}

// LDS byte address of a pointer into LDS, and the 4- or 8-byte map element at one.
__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
template <typename E> __device__ __forceinline__ E lds_elem(uint32_t addr);
template <> __device__ __forceinline__ float2 lds_elem<float2>(uint32_t addr)
{
    typedef float f2 __attribute__((ext_vector_type(2)));  // one 8-byte read
    const f2 v = *(const __attribute__((address_space(3))) f2 *)(uintptr_t)addr;
    return make_float2(v.x, v.y);
}
template <> __device__ __forceinline__ uint32_t lds_elem<uint32_t>(uint32_t addr)
{
    return *(const __attribute__((address_space(3))) uint32_t *)(uintptr_t)addr;
}

// LDS-DMA staging of columns of a folded map by a workgroup of NW waves. A wave moves 1 KB pieces
// (16 bytes per lane): pieces w, w + NW, ... of a run of columns, which lies contiguous in the map
// and in LDS. The copies are inline assembly so that the compiler does not tie them to the LDS
// reads of the other slab buffer: its wait-count pass cannot tell the buffers apart and would
// stall each wave's first read of a slab until its prefetch of the next one had landed; slab_sync
// waits for them. Addresses stay scalar (base in SGPRs, the lane's 16 bytes as the vector offset):
// with the 64-bit vector address and the generic LDS pointer of a plain builtin the loop around a
// copy took 52 scalar instructions per wave and slab, and the search scorer 6-8 % more time.
// The compiler keeps no wait states inside an asm block: gfx9 wants one between a scalar write of M0 and
// the copy that reads it, and five between a vector instruction's write of a scalar register and a vector
// memory address in it. The move of the address in between is the one, and makes a scalar write of the other.
template <int NW>
struct SlabDma {
    const char *src;    // this wave's first piece of column 0
    uint32_t col_bytes; // bytes per column (whole pieces)
    uint32_t wave_off;  // 1024 * wave
    uint32_t lane_off;  // 16 * lane

    __device__ __forceinline__ SlabDma(const MapP &m, int esize)
    {
        wave_off = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (uint32_t)kDmaBytes;
        const uint64_t y = (uint64_t)m.Y;  // wave-uniform, also where it was loaded through a vector register
        const uint32_t ylo = __builtin_amdgcn_readfirstlane((uint32_t)y);
        const uint32_t yhi = __builtin_amdgcn_readfirstlane((uint32_t)(y >> 32));
        src = reinterpret_cast<const char *>((uint64_t)yhi << 32 | ylo) + wave_off;
        col_bytes = __builtin_amdgcn_readfirstlane((uint32_t)m.ld * (uint32_t)esize);
        lane_off = (threadIdx.x & 63) * 16;
    }

    // columns c0 .. c0 + ncol - 1 to LDS address dst (c0, ncol and dst wave-uniform)
    __device__ __forceinline__ void issue(int c0, int ncol, uint32_t dst) const
    {
        const uint32_t bytes = (uint32_t)__builtin_amdgcn_readfirstlane(ncol) * col_bytes;
        const char *p = src + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(c0) * col_bytes;
        const uint32_t d = __builtin_amdgcn_readfirstlane(dst);
        for (uint32_t o = wave_off; o < bytes; o += NW * kDmaBytes, p += NW * kDmaBytes) {
            const char *q;
            asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                         : "=&s"(q) : "v"(lane_off), "s"(p), "s"(d + o) : "memory", "m0");
        }
    }
};

// Between two slabs: this wave's copies have landed and its LDS reads are done, then everyone's.
__device__ __forceinline__ void slab_sync()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
}

// ---------------------------------------------------------------- time-slab scorer
// One workgroup = WG lanes x TPT templates taken consecutively from the binned
// order; wave w owns the 64*TPT consecutive entries starting at w*64*TPT, so a
// wave's templates start and end in nearly the same columns. The workgroup
// sweeps the union of its waves' column ranges in slabs of columns staged into
// LDS, and each wave walks its own column range through them. Every template's
// row walk is started at its wave's first column (rewound when the template
// starts later), so all lanes step together: no divergent branches in the inner
// loop, the pixels outside a template are masked by a select and their LDS
// address clamped into the column. Per-template partial sums are FP32 between
// flush columns and FP64 across them.

// Walk columns ca..cb of the current slab (column c0 at slab[0]) for the TPT
// templates of this lane. MASK = false is the wave's core, where every
// template of the wave covers every column: no select and no clamp.
template <int TPT, bool MASK, bool HW, int MAPT>
__device__ __forceinline__ void walk(int ca, int cb, int c0, const elem_t<MAPT> *slab, int ldc, const int32_t (&t0)[TPT],
                                     const uint32_t (&span)[TPT], const PhaseK (&pk)[TPT], DdaF (&st)[TPT],
                                     float (&part)[TPT], double (&acc)[TPT])
{
    // segments end at the flush columns (c = 15 mod 16), so the inner loop has no flush test
    for (int c = ca; c <= cb;) {
        const int ce = min(cb, c | (kFlush - 1));
        for (; c <= ce; ++c) {
            const elem_t<MAPT> *col = slab + (c - c0) * ldc;
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                const int32_t row = ddaf_row(st[q]);
                if (MASK) {
                    const bool act = (uint32_t)c - (uint32_t)t0[q] <= span[q];
                    const float v = add_term_m<HW, MAPT>(part[q], pk[q], row, col[act ? row : 0]);
                    part[q] = act ? v : part[q];
                } else {
                    part[q] = add_term_m<HW, MAPT>(part[q], pk[q], row, col[row]);
                }
                ddaf_step(st[q]);
            }
        }
        if ((ce & (kFlush - 1)) == kFlush - 1) {  // wave-uniform
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                acc[q] += part[q];
                part[q] = 0.0f;
            }
        }
    }
}

// Row walks and sums of a lane's TPT templates in the LDS-DMA scorer. Rows are carried as
// kRowHi + row (the low word of exact_row and the high word of lazy_row), which the LDS
// address and the phase constant absorb: pa holds phase_a - kRowHi * phase_b (plus the rounding
// half unit of phase_turns with the hardware cosine).
template <int TPT>
struct SlabTpl {
    double num[TPT], del[TPT], dd[TPT], invq[TPT], Y[TPT];
    uint32_t pa[TPT], pb[TPT];
    uint32_t ext[TPT];  // first column | (columns - 1) << 16; kNoExtent: no template, never active
    float part[TPT];
};
constexpr uint32_t kNoExtent = 0xFFFFu;

// part + the Eq. 8 term (add_term_pol) of a pixel at kRowHi + row = r, pa as in SlabTpl.
template <bool HW, typename E>
__device__ __forceinline__ float add_term_hi(float part, uint32_t pa, uint32_t pb, uint32_t r, E v)
{
    const uint32_t ph = r * pb + pa + pol_arg(v);
    if constexpr (HW) {
        const float x = __builtin_bit_cast(float, __builtin_amdgcn_alignbit(0x7Fu, ph, 9u));
        return fmaf(__builtin_amdgcn_cosf(x), pol_mag(v), part);
    } else {
        return part + rot_re(ph, pol_mag(v), 0.0f);
    }
}

enum : int { kWalkMask = 0, kWalkExact = 1, kWalkLazy = 2 };

// Walk of one aligned slab of SC columns c0 .. c0 + SC - 1 at LDS address base (col_bytes per
// column): straight-line code, SC columns x TPT templates.
//   kWalkMask   some template of the wave does not cover every column: exact rows, selects
//   kWalkExact  the wave's core, exact rows
//   kWalkLazy   the wave's core, rows from the lazily seeded Y (one FP64 operation fewer per pixel)
// A column's rows and LDS reads are issued before the previous column's terms are evaluated (the
// scheduling barriers keep that order), so a gather has a column's worth of work to land behind:
// 1.17 -> 1.12 ms on the search map with 1024 x 2, 1.17 -> 1.15 with 512 x 4.
template <int SC, int TPT, bool HW, typename E, int KIND>
__device__ __forceinline__ void walk_slab(uint32_t c0, uint32_t base, uint32_t col_bytes, SlabTpl<TPT> &s)
{
    constexpr uint32_t kShift = sizeof(E) == 8 ? 3 : 2;
    uint32_t r[2][TPT];
    E v[2][TPT];
    bool act[2][TPT];
    auto fetch = [&](int j) {
        const int b = j & 1;
        const uint32_t col = base + (uint32_t)j * col_bytes - (kRowHi << kShift);
        uint32_t c = c0 + (uint32_t)j;
        if constexpr (KIND == kWalkMask) asm("" : "+s"(c));  // else j - t0 of every column is kept in registers
#pragma unroll
        for (int q = 0; q < TPT; ++q) {
            r[b][q] = KIND == kWalkLazy ? lazy_row(s.Y[q]) : exact_row(s.num[q], s.invq[q]);
            if constexpr (KIND == kWalkMask) {
                act[b][q] = c - (s.ext[q] & 0xFFFFu) <= s.ext[q] >> 16;
                r[b][q] = act[b][q] ? r[b][q] : kRowHi;
            }
            v[b][q] = lds_elem<E>((r[b][q] << kShift) + col);
            if constexpr (KIND == kWalkLazy) s.Y[q] = lazy_step(s.Y[q], s.del[q], s.invq[q]);
            else s.num[q] += s.del[q];
            s.del[q] += s.dd[q];
        }
    };
    fetch(0);
#pragma unroll
    for (int j = 0; j < SC; ++j) {
        if (j + 1 < SC) fetch(j + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < TPT; ++q) {
            const float p = add_term_hi<HW>(s.part[q], s.pa[q], s.pb[q], r[j & 1][q], v[j & 1][q]);
            s.part[q] = KIND != kWalkMask || act[j & 1][q] ? p : s.part[q];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // the sums are used here: without this the compiler moves the slab's terms into the block that
    // reads them next, with every gathered element spilled on the way
#pragma unroll
    for (int q = 0; q < TPT; ++q) asm volatile("" : "+v"(s.part[q]));
}

// The block's best key from its lanes' keys: waves by shuffles, then across waves through LDS.
template <int WG>
__device__ __forceinline__ uint64_t block_best(uint64_t key, uint64_t *kred)
{
    key = wave_max_u64(key);
    if ((threadIdx.x & 63) == 0) kred[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < WG / 64; ++w) key = kred[w] > key ? kred[w] : key;
    return key;  // valid in thread 0
}

// One block of WG*TPT consecutive entries of `order` (block index b): the
// whole slab sweep for those templates. slab is the dynamic LDS, bnd two LDS
// ints. Callable repeatedly by a persistent workgroup. Templates are drawn
// (tr == NULL) or read from tr and validated. The folded map (kMapPol: 8 bytes
// per pixel, kMapPolH: 4 bytes; columns padded to whole 1 KB pieces) is staged
// with LDS DMA into two slab buffers of SC columns (double buffering: slab k+1
// streams in while slab k is walked). Slabs are aligned to multiples of SC on the
// absolute column grid, so the FP32 partial sums are flushed between slabs and
// a slab is one straight-line walk_slab; each wave starts its rows at its first
// aligned column (columns before a template's start and after its end are
// masked, so the extra columns change nothing). A wave passes its slabs in
// phases, each a loop of its own so that no state is copied between branches:
// waiting for its first column, masked, core, masked, waiting for the others.
// What bounds it: vector-ALU issue (0.82 ms of the search map's 1.12 with neither LDS reads,
// staging nor barriers), then the random 8-byte LDS gathers (7 clocks each) and the staging.
template <int WG, int TPT, bool HW, int MAPT, int SC>
__device__ __forceinline__ uint64_t score_block(const MapP &m, const GenP &g, const Trk *tr, const uint32_t *order,
                                                uint64_t first, int64_t n, int64_t b, int32_t norm, float *snr,
                                                float2 *slab_raw, int *bnd, uint64_t *kred)
{
    static_assert(kFlush % SC == 0, "slabs must tile the flush grid");
    using E = elem_t<MAPT>;
    __syncthreads();  // LDS of a previous block is no longer read
    if (threadIdx.x == 0) { bnd[0] = 0x7fffffff; bnd[1] = -1; }

    const int lane = threadIdx.x & 63;
    const int64_t wbase = b * (WG * TPT) + (int64_t)(threadIdx.x >> 6) * (64 * TPT) + lane;
    const bool expl = tr != nullptr;
    SlabTpl<TPT> s;
    double acc[TPT];
    Trk tk[TPT];
    int lo = 0x7fffffff, hi = -1;        // union of this wave's templates
    int clo = -1, chi = 0x7fffffff;      // intersection (the core)
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const int64_t e = wbase + q * 64;
        const bool live = e < n;
        const uint32_t idx = live ? order[e] : 0u;
        Trk t = expl ? tr[idx] : draw_track(g, first + idx);
        const bool ok = live && (!expl || track_ok(t, m));
        if (!ok) t = Trk{0, 1, 0u, 0u, 0u, 0};
        tk[q] = t;
        s.ext[q] = ok ? (uint32_t)t.t0 | (uint32_t)(t.t2 - t.t0) << 16 : kNoExtent;
        const PhaseK pk = phase_k(m, t.dtau);
        s.pb[q] = pk.pb;
        s.pa[q] = pk.pa - kRowHi * pk.pb + (HW ? 256u : 0u);
        s.part[q] = 0.0f;
        acc[q] = 0.0;
        if (ok) {
            lo = min(lo, t.t0);
            hi = max(hi, t.t2);
            clo = max(clo, t.t0);
            chi = min(chi, t.t2);
        } else {
            clo = 0x7fffffff;  // a lane without a template: no unmasked core for this wave
            chi = -1;
        }
    }
    int dmax = 0;  // longest template
#pragma unroll
    for (int q = 0; q < TPT; ++q) dmax = max(dmax, (int)(s.ext[q] >> 16));
    lo = wave_min_i32(lo);
    hi = wave_max_i32(hi);
    clo = wave_max_i32(clo);
    chi = wave_min_i32(chi);
    const int seed_cols = lazy_period(wave_max_i32(dmax));
    // the rows start at the wave's first column, aligned down to a slab boundary
    const int start = lo == 0x7fffffff ? 0 : lo & ~(SC - 1);
    // core slabs lie in [core0, core1)
    int core0 = hi + 1, core1 = hi + 1;
    if (clo <= chi) {
        const int a0 = (clo + SC - 1) & ~(SC - 1), a1 = (chi + 1) & ~(SC - 1);
        if (a0 < a1) { core0 = a0; core1 = a1; }
    }
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const DdaF d = ddaf_init_at(tk[q], start - tk[q].t0);
        s.num[q] = d.num;
        s.del[q] = d.del;
        s.dd[q] = d.dd;
        s.invq[q] = d.invq;
    }
    __syncthreads();
    if (lane == 0) {
        atomicMin(&bnd[0], lo);
        atomicMax(&bnd[1], hi);
    }
    __syncthreads();
    const int c_first = __builtin_amdgcn_readfirstlane(bnd[0]), c_last = __builtin_amdgcn_readfirstlane(bnd[1]);
    const SlabDma<WG / 64> dma(m, (int)sizeof(E));
    const uint32_t col_bytes = dma.col_bytes, buf0 = lds_addr(slab_raw), buf1 = buf0 + SC * col_bytes;
    int c0 = c_first & ~(SC - 1);
    if (c_first <= c_last) dma.issue(c0, min(SC, c_last - c0 + 1), buf0);
    uint32_t cur = buf1;
    // slab c0: its copies have landed, the next one's are on their way; returns its LDS address
    auto next_slab = [&](int c) {
        slab_sync();
        const uint32_t other = cur;
        cur = buf0 + buf1 - cur;
        if (c + SC <= c_last) dma.issue(c + SC, min(SC, c_last - c - SC + 1), other);
        return cur;
    };
    auto flush = [&](int c) {
        if (((c + SC) & (kFlush - 1)) == 0) {  // wave-uniform: the slab ends a flush group
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                acc[q] += s.part[q];
                s.part[q] = 0.0f;
            }
        }
    };
    for (; c0 < start && c0 <= c_last; c0 += SC) next_slab(c0);
    for (; c0 < core0 && c0 <= hi; c0 += SC) {
        walk_slab<SC, TPT, HW, E, kWalkMask>(c0, next_slab(c0), col_bytes, s);
        flush(c0);
    }
    // seeds lie between slabs: on slabs wider than the period (16 columns from 1021 columns of extent on, 8
    // from 1440) the core takes exact rows, at the speed of the code before the lazy ones
    if (seed_cols >= SC) {
        int seeded = c0;  // the column of num
        auto seed = [&](int c) {
            const double d = (double)(c - seeded), e = -0.5 * d * (d + 1.0);
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                s.num[q] = fma(e, s.dd[q], fma(d, s.del[q], s.num[q]));
                s.Y[q] = lazy_seed(s.num[q], s.invq[q]);
            }
            seeded = c;
        };
        if (c0 < core1) seed(c0);
        for (; c0 < core1; c0 += SC) {
            walk_slab<SC, TPT, HW, E, kWalkLazy>(c0, next_slab(c0), col_bytes, s);
            flush(c0);
            if (((c0 + SC) & (seed_cols - 1)) == 0) seed(c0 + SC);
        }
        if (seeded != c0) seed(c0);
    } else {
        for (; c0 < core1; c0 += SC) {
            walk_slab<SC, TPT, HW, E, kWalkExact>(c0, next_slab(c0), col_bytes, s);
            flush(c0);
        }
    }
    for (; c0 <= hi; c0 += SC) {
        walk_slab<SC, TPT, HW, E, kWalkMask>(c0, next_slab(c0), col_bytes, s);
        flush(c0);
    }
    for (; c0 <= c_last; c0 += SC) next_slab(c0);

    uint64_t key = 0;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const int64_t e = wbase + q * 64;
        if (e >= n) continue;
        const uint32_t idx = order[e];
        const float z = s.ext[q] != kNoExtent ? finish(acc[q] + s.part[q], (int32_t)(s.ext[q] >> 16) + 1, norm, m.scale)
                                        : __builtin_nanf("");
        if (snr) snr[idx] = z;
        const uint64_t k = key_encode(z, (uint32_t)(first + idx));
        key = k > key ? k : key;
    }
    return block_best<WG>(key, kred);
}

// The same for maps whose columns do not fit two DMA slabs (or with DMA staging off): the lanes
// stage S columns through registers into one buffer and walk them column by column.
template <int WG, int TPT, bool HW, int MAPT>
__device__ __forceinline__ uint64_t score_block_regs(const MapP &m, const GenP &g, const Trk *tr, const uint32_t *order,
                                                uint64_t first, int64_t n, int64_t b, int S, int32_t norm, float *snr,
                                                float2 *slab_raw, int *bnd, uint64_t *kred)
{
    // element format of the slab: the map's own for the folded formats, p in Cartesian form otherwise
    constexpr int SM = (MAPT == kMapPol || MAPT == kMapPolH) ? MAPT : kMapPF;
    using E = elem_t<SM>;
    __syncthreads();  // LDS of a previous block is no longer read
    if (threadIdx.x == 0) { bnd[0] = 0x7fffffff; bnd[1] = -1; }

    const int lane = threadIdx.x & 63;
    const int64_t wbase = b * (WG * TPT) + (int64_t)(threadIdx.x >> 6) * (64 * TPT);
    const bool expl = tr != nullptr;
    Trk tk[TPT];
    int32_t t0[TPT];
    uint32_t span[TPT], idx[TPT];
    PhaseK pk[TPT];
    bool ok[TPT], live[TPT];
    int lo = 0x7fffffff, hi = -1;        // union of this wave's templates
    int clo = -1, chi = 0x7fffffff;      // intersection (the core)
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const int64_t e = wbase + q * 64 + lane;
        live[q] = e < n;
        idx[q] = live[q] ? order[e] : 0u;
        Trk t = expl ? tr[idx[q]] : draw_track(g, first + idx[q]);
        ok[q] = live[q] && (!expl || track_ok(t, m));
        if (!ok[q]) t = Trk{0, 1, 0u, 0u, 0u, 0};  // never active: (c - t0) > span below
        tk[q] = t;
        t0[q] = ok[q] ? t.t0 : 0x7fffffff;
        span[q] = ok[q] ? (uint32_t)(t.t2 - t.t0) : 0u;
        pk[q] = phase_k(m, t.dtau);
        if (ok[q]) {
            lo = min(lo, t.t0);
            hi = max(hi, t.t2);
            clo = max(clo, t.t0);
            chi = min(chi, t.t2);
        } else {
            clo = 0x7fffffff;  // a lane without a template: no unmasked core for this wave
            chi = -1;
        }
    }
    lo = wave_min_i32(lo);
    hi = wave_max_i32(hi);
    clo = wave_max_i32(clo);
    chi = wave_min_i32(chi);
    if (clo > chi) {  // empty core: everything goes through the masked walk
        clo = hi + 1;
        chi = hi;
    }
    DdaF st[TPT];
    float part[TPT];
    double acc[TPT];
    const int start = lo == 0x7fffffff ? 0 : lo;  // the rows start at the wave's first column
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        st[q] = ddaf_init_at(tk[q], start - tk[q].t0);
        part[q] = 0.0f;
        acc[q] = 0.0;
    }
    __syncthreads();
    if (lane == 0) {
        atomicMin(&bnd[0], lo);
        atomicMax(&bnd[1], hi);
    }
    __syncthreads();
    const int c_first = __builtin_amdgcn_readfirstlane(bnd[0]), c_last = __builtin_amdgcn_readfirstlane(bnd[1]);
    const int F = m.F;

    E *slab = reinterpret_cast<E *>(slab_raw);
    // staging walk: element e = tid + i*WG of the slab is (column e / F, row e % F)
    const int dcol = WG / F, drow = WG % F;
    const int col0 = threadIdx.x / F, row0 = threadIdx.x % F;
    for (int c0 = c_first; c0 <= c_last; c0 += S) {
        const int ncol = min(S, c_last - c0 + 1);
        __syncthreads();  // the previous slab has been consumed
        {
            int col = col0, r = row0;
            const int64_t base = (int64_t)c0 * m.ld;
#pragma unroll 4
            for (int e = threadIdx.x; e < ncol * F; e += WG) {
                slab[col * F + r] = load_e<MAPT>(m, base + (int64_t)col * m.ld + r);
                r += drow;
                col += dcol;
                if (r >= F) { r -= F; ++col; }
            }
        }
        __syncthreads();
        const int ca = max(c0, lo), cb = min(c0 + ncol - 1, hi);  // this wave's columns in the slab
        walk<TPT, true, HW, SM>(ca, min(cb, clo - 1), c0, slab, F, t0, span, pk, st, part, acc);
        walk<TPT, false, HW, SM>(max(ca, clo), min(cb, chi), c0, slab, F, t0, span, pk, st, part, acc);
        walk<TPT, true, HW, SM>(max(ca, chi + 1), cb, c0, slab, F, t0, span, pk, st, part, acc);
    }

    uint64_t key = 0;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        if (!live[q]) continue;
        const float z = ok[q] ? finish(acc[q] + part[q], (int32_t)span[q] + 1, norm, m.scale) : __builtin_nanf("");
        if (snr) snr[idx[q]] = z;
        const uint64_t k = key_encode(z, (uint32_t)(first + idx[q]));
        key = k > key ? k : key;
    }
    return block_best<WG>(key, kred);
}

// One block of binned templates per workgroup. Each workgroup stores its best
// key in its own slot of wg_keys (no atomics: many same-address atomics from
// every wave serialise across the chip); k_reduce_keys folds the slots.
// Four templates per lane: at least 4 waves per SIMD (at most 128 VGPRs), so that two workgroups
// of 512 lanes, or four of 256, can share a CU when their slabs fit its LDS. Two per lane with DMA
// staging: 8 waves (64 VGPRs, two workgroups of 1024 lanes). These bounds are kept by spilling state that
// the lazy and the masked loops do not touch: 10 VGPRs for 1024 x 2 on SC = 4, 31 for its batch, whose exact
// core (kWalkExact) loads and stores two words per slab.
template <int TPT, int SC> constexpr int kSlabWavesPerSimd = TPT <= 2 && SC > 0 ? 8 : 4;

template <int WG, int TPT, bool HW, int MAPT, int SC>
__device__ __forceinline__ uint64_t score_block_any(const MapP &m, const GenP &g, const Trk *tr, const uint32_t *order,
                                                    uint64_t first, int64_t n, int64_t b, int S, int32_t norm,
                                                    float *snr, float2 *slab, int *bnd, uint64_t *kred)
{
    if constexpr (SC > 0)
        return score_block<WG, TPT, HW, MAPT, SC>(m, g, tr, order, first, n, b, norm, snr, slab, bnd, kred);
    else
        return score_block_regs<WG, TPT, HW, MAPT>(m, g, tr, order, first, n, b, S, norm, snr, slab, bnd, kred);
}

template <int WG, int TPT, bool HW, int MAPT, int SC>
__global__ __launch_bounds__(WG, (kSlabWavesPerSimd<TPT, SC>)) void k_score_slab(MapP m, GenP g, const Trk *tr,
                                                                      const uint32_t *order, uint64_t first,
                                                                      int64_t n, int S, int32_t norm, float *snr,
                                                                      uint64_t *wg_keys)
{
    extern __shared__ float2 slab[];
    __shared__ int bnd[2];
    __shared__ uint64_t kred[WG / 64];
    const uint64_t key = score_block_any<WG, TPT, HW, MAPT, SC>(m, g, tr, order, first, n, (int64_t)blockIdx.x, S,
                                                                norm, snr, slab, bnd, kred);
    if (threadIdx.x == 0) wg_keys[blockIdx.x] = key;
}

// Max of n keys into *best (max-merged with what it holds), in one workgroup.
__global__ __launch_bounds__(1024) void k_reduce_keys(const uint64_t *keys, int64_t n, uint64_t *best)
{
    __shared__ uint64_t kred[16];
    uint64_t key = 0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) key = keys[i] > key ? keys[i] : key;
    key = wave_max_u64(key);
    if ((threadIdx.x & 63) == 0) kred[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) key = kred[w] > key ? kred[w] : key;
        if (key) atomicMax((unsigned long long *)best, (unsigned long long)key);
    }
}

// ---------------------------------------------------------------- templates with a free t_mid
// A free-t_mid template's rows have no recurrence: each column's row is an
// independent root (row_tm). Both scorers below walk a template's columns on
// the flush grid of the plain scorers (FP32 partial sums per group of kFlush
// aligned columns, FP64 across groups in column order), so they give the same
// bits: k_score_tm_slab (binned templates, LDS slabs, like k_score_md_slab) for
// generated templates, k_score_tm (one wave per template, lanes over groups,
// like k_score_wave) for small calls and given lists.

__device__ __forceinline__ bool track_tm_ok(const TrkTm &t, const MapP &m)
{
    const uint32_t lim = (uint32_t)m.F << 8;
    return t.t0 >= 0 && t.t0 < t.t2 && t.t2 < m.T && t.t1 >= t.t0 && t.t1 <= t.t2 && t.f0 < lim && t.f1 < lim &&
           t.f2 < lim;
}

__global__ __launch_bounds__(256) void k_make_tracks_tm(GenP g, uint64_t first, int64_t n, TrkTm *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = draw_track_tm(g, first + (uint64_t)i);
}

// A wave per template, lanes over flush groups (as k_score_wave, with an independent row per column): the
// FP32 pass over the whole group, then one copy of the exact path for the columns that it leaves open, each
// lane its own next one, then the gathers. Compiled in at each of the 16 columns the exact path was half of
// the code (5600 instructions, now 3400): lists of 16 to 50 000 templates take 10 % less on average.
template <bool EXPL, bool HW, int MAPT>
__global__ __launch_bounds__(256) void k_score_tm(MapP m, GenP g, const TrkTm *tr, uint64_t first, int64_t n,
                                                  int32_t norm, float *snr, uint64_t *best)
{
    const int lane = threadIdx.x & 63;
    uint64_t key = 0;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {  // wave-uniform
        const TrkTm t = EXPL ? tr[i] : draw_track_tm(g, first + (uint64_t)i);
        float z = __builtin_nanf("");
        if (!EXPL || track_tm_ok(t, m)) {
            const RowTm k = row_tm_init(t);
            const PhaseK pk = phase_k(m, t.dtau);
            const int gfirst = t.t0 / kFlush, glast = t.t2 / kFlush;
            float gp[kWaveRounds];
#pragma unroll
            for (int r = 0; r < kWaveRounds; ++r) {
                gp[r] = 0.0f;
                const int gi = gfirst + r * 64 + lane;
                if (gi > glast) continue;
                const int32_t cb = gi * kFlush;
                int32_t row[kFlush];
                uint32_t open = 0;  // columns that the FP32 pass leaves open
#pragma unroll
                for (int j = 0; j < kFlush; ++j) {
                    const bool act = cb + j >= t.t0 && cb + j <= t.t2;
                    bool ok;
                    const int32_t r = row_tm_fp32(k, act ? cb + j - t.t0 : 1, ok);
                    row[j] = act ? r : 0;
                    open |= act && !ok ? 1u << j : 0u;
                }
                // one copy of the exact path, each lane at its own next column
#pragma unroll 1
                while (open) {
                    const int32_t q = __builtin_ctz(open);
                    const int32_t r = row_tm_fallback(k, cb + q - t.t0);
#pragma unroll
                    for (int j = 0; j < kFlush; ++j) row[j] = j == q ? r : row[j];
                    open &= open - 1;
                }
                pol_t<MAPT> v[kFlush];
#pragma unroll
                for (int j = 0; j < kFlush; ++j) {
                    const bool act = cb + j >= t.t0 && cb + j <= t.t2;
                    v[j] = load_pol<MAPT>(m, (int64_t)(act ? cb + j : t.t0) * m.ld + row[j]);
                }
                float part = 0.0f;
#pragma unroll
                for (int j = 0; j < kFlush; ++j) {
                    const int32_t c = gi * kFlush + j;
                    const float p = add_term_pol<HW>(part, pk, row[j], v[j]);
                    part = c >= t.t0 && c <= t.t2 ? p : part;
                }
                gp[r] = part;
            }
            z = finish(wave_ordered_sum(gp, glast - gfirst + 1), t.t2 - t.t0 + 1, norm, m.scale);
        }
        if (lane == 0 && snr) snr[i] = z;
        const uint64_t k = key_encode(z, (uint32_t)(first + (uint64_t)i));
        key = k > key ? k : key;
    }
    merge_key(best, key);
}

// Column walk of the free-t_mid slab scorer (as walk, with an independent row per column). The
// FP32 pass takes every template's row of the column, with D = b^2 + 4 a dt and 2 dt carried from
// column to column by one add each (Dc, dt2c: their values at column ca, advanced past cb on
// return, so that the wave's walks over consecutive column ranges carry them through); where it
// does not stand for some lane (about one template pixel in a thousand on the search band), the
// whole wave takes one uniform branch in which those lanes settle their rows exactly. A lane
// outside its template's columns works on column t0 + 1 (valid for every template) and drops the
// term.
template <int TPT, bool MASK, bool HW, typename E>
__device__ __forceinline__ void walk_tm(int ca, int cb, int c0, const E *slab, int ldc, const int32_t (&t0)[TPT],
                                        const uint32_t (&span)[TPT], const RowTm (&rk)[TPT],
                                        const PhaseK (&pk)[TPT], int32_t (&Dc)[TPT], float (&dt2c)[TPT],
                                        float (&part)[TPT], double (&acc)[TPT])
{
    for (int c = ca; c <= cb;) {
        const int ce = min(cb, c | (kFlush - 1));
        for (; c <= ce; ++c) {
            int32_t row[TPT];
            bool act[TPT], ok[TPT];
            bool redo = false;
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                act[q] = !MASK || (uint32_t)(c - t0[q]) <= span[q];
                const int32_t D = act[q] ? Dc[q] : rk[q].bb + rk[q].a4;
                row[q] = row_tm_fp32_d(rk[q], D, act[q] ? dt2c[q] : 2.0f, ok[q]);
                ok[q] = ok[q] || !act[q];
                redo = redo || !ok[q];
                Dc[q] = (int32_t)((uint32_t)Dc[q] + (uint32_t)rk[q].a4);
                dt2c[q] += 2.0f;
            }
            if (__builtin_amdgcn_ballot_w64(redo)) {  // wave-uniform
                // the column through readfirstlane: no induction variables for this rare branch
                // are kept up to date in the loop
                const int cu = __builtin_amdgcn_readfirstlane(c);
#pragma unroll
                for (int q = 0; q < TPT; ++q)
                    if (!ok[q]) row[q] = row_tm_fallback(rk[q], cu - t0[q]);
            }
            const E *col = slab + (c - c0) * ldc;
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                const int32_t r = MASK && !act[q] ? 0 : row[q];
                const float v = add_term_pol<HW>(part[q], pk[q], r, col[r]);
                part[q] = act[q] ? v : part[q];
            }
        }
        if ((ce & (kFlush - 1)) == kFlush - 1) {  // wave-uniform
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                acc[q] += part[q];
                part[q] = 0.0f;
            }
        }
    }
}

// With one template per lane the scorer fits 64 VGPRs, so that 8 waves share each SIMD (two
// workgroups of 1024 lanes per CU with 80 KB of slabs each): the more waves, the more of the
// latency of the root's square root and reciprocal and of the LDS gathers is hidden.
template <int WG, int TPT, bool HW, int MAPT>
__global__ __launch_bounds__(WG, TPT == 1 ? 8 : 1) void k_score_tm_slab(MapP m, GenP g, const uint32_t *order,
                                                                         uint64_t first, int64_t n, int S, int32_t norm,
                                                                         float *snr, uint64_t *wg_keys)
{
    extern __shared__ float2 slab[];
    __shared__ int bnd[2];
    __shared__ uint64_t kred[WG / 64];
    if (threadIdx.x == 0) { bnd[0] = 0x7fffffff; bnd[1] = -1; }
    const int lane = threadIdx.x & 63;
    const int64_t wbase = (int64_t)blockIdx.x * (WG * TPT) + (int64_t)(threadIdx.x >> 6) * (64 * TPT);
    int32_t t0[TPT];
    uint32_t span[TPT], idx[TPT];
    bool live[TPT];
    RowTm rk[TPT];
    PhaseK pk[TPT];
    int lo = 0x7fffffff, hi = -1, clo = -1, chi = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const int64_t e = wbase + q * 64 + lane;
        live[q] = e < n;
        idx[q] = live[q] ? order[e] : 0u;
        TrkTm t = draw_track_tm(g, first + idx[q]);
        if (!live[q]) t = TrkTm{0, 0, 1, 0u, 0u, 0u, 0};  // never active: (c - t0) > span below
        rk[q] = row_tm_init(t);
        pk[q] = phase_k(m, t.dtau);
        t0[q] = live[q] ? t.t0 : 0x7fffffff;
        span[q] = live[q] ? (uint32_t)(t.t2 - t.t0) : 0u;
        if (live[q]) {
            lo = min(lo, t.t0);
            hi = max(hi, t.t2);
            clo = max(clo, t.t0);
            chi = min(chi, t.t2);
        } else {
            clo = 0x7fffffff;
            chi = -1;
        }
    }
    lo = wave_min_i32(lo);
    hi = wave_max_i32(hi);
    clo = wave_max_i32(clo);
    chi = wave_min_i32(chi);
    if (clo > chi) { clo = hi + 1; chi = hi; }
    float part[TPT];
    double acc[TPT];
    // D and 2 dt at the wave's first column; the walks then carry them column by column. Modulo
    // 2^32: a lane that holds no template (t0 = INT_MAX) only ever takes the masked walk.
    int32_t Dc[TPT];
    float dt2c[TPT];
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        part[q] = 0.0f;
        acc[q] = 0.0;
        const uint32_t dt = (uint32_t)lo - (uint32_t)t0[q];
        Dc[q] = (int32_t)((uint32_t)rk[q].bb + (uint32_t)rk[q].a4 * dt);
        dt2c[q] = 2.0f * (float)(int32_t)dt;
    }
    __syncthreads();
    if (lane == 0) {
        atomicMin(&bnd[0], lo);
        atomicMax(&bnd[1], hi);
    }
    __syncthreads();
    const int c_first = __builtin_amdgcn_readfirstlane(bnd[0]), c_last = __builtin_amdgcn_readfirstlane(bnd[1]);
    using E = elem_t<MAPT>;
    const int ldc = (int)m.ld;
    const SlabDma<WG / 64> dma(m, (int)sizeof(E));
    const uint32_t buf0 = lds_addr(slab), slab_bytes = (uint32_t)S * dma.col_bytes;
    if (c_first <= c_last) dma.issue(c_first, min(S, c_last - c_first + 1), buf0);
    int kk = 0;
    for (int c0 = c_first; c0 <= c_last; c0 += S, ++kk) {
        slab_sync();  // slab kk has landed and slab kk-1 is no longer read
        if (c0 + S <= c_last) dma.issue(c0 + S, min(S, c_last - c0 - S + 1), buf0 + ((kk + 1) & 1) * slab_bytes);
        const E *cur = reinterpret_cast<const E *>(reinterpret_cast<const char *>(slab) + (size_t)(kk & 1) * slab_bytes);
        const int ncol = min(S, c_last - c0 + 1);
        const int ca = max(c0, lo), cb = min(c0 + ncol - 1, hi);
        walk_tm<TPT, true, HW>(ca, min(cb, clo - 1), c0, cur, ldc, t0, span, rk, pk, Dc, dt2c, part, acc);
        walk_tm<TPT, false, HW>(max(ca, clo), min(cb, chi), c0, cur, ldc, t0, span, rk, pk, Dc, dt2c, part, acc);
        walk_tm<TPT, true, HW>(max(ca, chi + 1), cb, c0, cur, ldc, t0, span, rk, pk, Dc, dt2c, part, acc);
    }
    uint64_t key = 0;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        if (!live[q]) continue;
        const float z = finish(acc[q] + part[q], (int32_t)span[q] + 1, norm, m.scale);
        if (snr) snr[idx[q]] = z;
        const uint64_t k = key_encode(z, (uint32_t)(first + idx[q]));
        key = k > key ? k : key;
    }
    key = wave_max_u64(key);
    if (lane == 0) kred[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < WG / 64; ++w) key = kred[w] > key ? kred[w] : key;
        wg_keys[blockIdx.x] = key;
    }
}

// ---------------------------------------------------------------- delay-maximised scoring
// The maximum of Eq. 8 over a grid of delays per template (a reading of
// "phase-maximised"): the template keeps its geometry and its own delay is
// replaced by dtau_m = d0 + m * step. A launch handles kMD consecutive delays
// m0 .. m0 + cnt - 1 of the grid for every template: the row walk and the
// pixel gather are shared, each delay has its own (wave-uniform) phase
// constants and accumulators, on the same flush grid as the other scorers.
// The running maximum and its index live in snr / tidx between launches.
constexpr int kMD = 8;

// The grid is uniform, so at row r the phase of delay k of a launch is
// phase_0(r) + k * dphase(r) (32-bit, exact). The map is in polar form, so the
// term of delay k is |p| cos(theta_k) with theta_k = 2 pi (phase_k + arg p):
// the first delay's term is the plain scorer's (add_term_pol, the same bits),
// and each further (cos, sin) theta_k is the previous one rotated by
// exp(2 pi i dphase(r)), one complex multiply (at most kMD - 1 = 7 in a row, a
// few 1e-7 relative).
struct DelayGrid {
    PhaseK k0;       // phase constants of the launch's first delay
    PhaseK dk;       // phase constants of the grid step
    int32_t m0, cnt;
};

__device__ __forceinline__ DelayGrid delay_grid(const MapP &m, int32_t d0, int32_t step, int32_t m0, int32_t cnt)
{
    DelayGrid dg;
    dg.m0 = m0;
    dg.cnt = cnt;
    const int32_t d = (int32_t)((uint32_t)d0 + (uint32_t)m0 * (uint32_t)step);  // in range (checked by the host)
    dg.k0 = phase_k(m, d);
    dg.dk = phase_k(m, step);
    return dg;
}

// Adds the template's Eq. 8 terms at `row` for all kMD delays of the launch.
template <bool HW, bool MASK, typename E>
__device__ __forceinline__ void add_terms_md(float (&part)[kMD], const DelayGrid &dg, int32_t row, E pp, bool act)
{
    const float v0 = add_term_pol<HW>(part[0], dg.k0, row, pp);
    part[0] = !MASK || act ? v0 : part[0];
    const uint32_t arg = pol_arg(pp);
    const float mag = pol_mag(pp);
    float c, s, cr, sr;
    if constexpr (HW) {
        const float x0 = phase_turns(dg.k0.pa + arg, dg.k0.pb, row), xr = phase_turns(dg.dk.pa, dg.dk.pb, row);
        c = __builtin_amdgcn_cosf(x0);
        s = __builtin_amdgcn_sinf(x0);
        cr = __builtin_amdgcn_cosf(xr);
        sr = __builtin_amdgcn_sinf(xr);
    } else {
        const uint32_t ph0 = dg.k0.pa + arg + (uint32_t)row * dg.k0.pb, phr = dg.dk.pa + (uint32_t)row * dg.dk.pb;
        c = rot_re(ph0, 1.0f, 0.0f);
        s = rot_re(ph0 - 0x40000000u, 1.0f, 0.0f);  // cos(x - pi/2) = sin x
        cr = rot_re(phr, 1.0f, 0.0f);
        sr = rot_re(phr - 0x40000000u, 1.0f, 0.0f);
    }
#pragma unroll
    for (int k = 1; k < kMD; ++k) {
        const float cn = fmaf(c, cr, -s * sr), sn = fmaf(s, cr, c * sr);
        c = cn;
        s = sn;
        const float v = fmaf(c, mag, part[k]);
        part[k] = !MASK || act ? v : part[k];
    }
}

// The best of this launch's delays for one template, merged with the running
// maximum of earlier launches (strictly greater wins, so ties keep the lowest
// index). A NaN score (from NaN map data) makes the result NaN with index -1.
__device__ __forceinline__ void merge_delays(const double (&acc)[kMD], const float (&part)[kMD], int32_t N,
                                             int32_t norm, float scale, const DelayGrid &dg, bool ok, float &z,
                                             int32_t &mi)
{
    z = __builtin_nanf("");
    mi = -1;
    if (!ok) return;
    bool nan = false;
#pragma unroll
    for (int k = 0; k < kMD; ++k) {
        if (k >= dg.cnt) break;
        const float v = finish(acc[k] + part[k], N, norm, scale);
        if (v != v) nan = true;
        else if (mi < 0 || v > z) { z = v; mi = dg.m0 + k; }
    }
    if (nan) { z = __builtin_nanf(""); mi = -1; }
}

__device__ __forceinline__ void merge_running(float &z, int32_t &mi, float zp, int32_t mp, bool first_launch)
{
    if (first_launch) return;
    if (zp != zp || mp < 0 || z != z) { z = __builtin_nanf(""); mi = -1; return; }
    if (!(z > zp)) { z = zp; mi = mp; }
}

// The FP32 sums, for the launch's delays, of a template's terms over the flush group that starts at
// column cb, for a row walk standing there (as group_sum).
template <bool HW, int MAPT, int G = kFlush>
__device__ __forceinline__ void group_sums_md(const MapP &m, const DelayGrid &dg, int32_t cb, int32_t t0, int32_t t2,
                                              DdaF &st, float (&part)[kMD])
{
#pragma unroll
    for (int k = 0; k < kMD; ++k) part[k] = 0.0f;
#pragma unroll
    for (int j0 = 0; j0 < kFlush; j0 += G) {
        int32_t row[G];
        pol_t<MAPT> v[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = cb + j0 + j;
            const bool act = c >= t0 && c <= t2;
            row[j] = act ? ddaf_row(st) : 0;
            v[j] = load_pol<MAPT>(m, (int64_t)(act ? c : t0) * m.ld + row[j]);
            ddaf_step(st);
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = cb + j0 + j;
            add_terms_md<HW, true>(part, dg, row[j], v[j], c >= t0 && c <= t2);
        }
        if (G < kFlush) __builtin_amdgcn_sched_barrier(0);
    }
}

// One lane per template, direct gathers (maps too wide for LDS, medium calls).
template <bool EXPL, bool HW, int MAPT, int G>
__global__ __launch_bounds__(kWG) void k_score_md_direct(MapP m, GenP g, const Trk *tr, uint64_t first, int64_t n,
                                                         int32_t norm, int32_t d0, int32_t step, int32_t m0,
                                                         int32_t cnt, int32_t last, float *snr, int32_t *tidx,
                                                         uint64_t *best)
{
    const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
    const DelayGrid dg = delay_grid(m, d0, step, m0, cnt);
    uint64_t key = 0;
    if (i < n) {
        const Trk t = EXPL ? tr[i] : draw_track(g, first + (uint64_t)i);
        const bool ok = !EXPL || track_ok(t, m);
        double acc[kMD];
        float part[kMD];
#pragma unroll
        for (int k = 0; k < kMD; ++k) { acc[k] = 0.0; part[k] = 0.0f; }
        if (ok) {
            int32_t cb = t.t0 & ~(kFlush - 1);
            DdaF st = ddaf_init_at(t, cb - t.t0);
            for (; cb <= t.t2; cb += kFlush) {
                group_sums_md<HW, MAPT, G>(m, dg, cb, t.t0, t.t2, st, part);
#pragma unroll
                for (int q = 0; q < kMD; ++q) { acc[q] += part[q]; part[q] = 0.0f; }
            }
        }
        float z;
        int32_t mi;
        merge_delays(acc, part, t.t2 - t.t0 + 1, norm, m.scale, dg, ok, z, mi);
        merge_running(z, mi, m0 ? snr[i] : 0.0f, m0 ? tidx[i] : 0, m0 == 0);
        snr[i] = z;
        tidx[i] = mi;
        if (last) key = key_encode(z, (uint32_t)(first + (uint64_t)i));
    }
    if (last) merge_key(best, key);
}

// Between a wave's LDS stores and its lanes' loads of each other's values (or the other way round). The
// LDS serves a wave in order; the fences keep the compiler to that order and cost no instruction.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per template for small calls: lanes over flush groups as k_score_wave, each group's kMD
// partial sums through LDS to kMD lanes, which add them in column order (the same bits as the other
// scorers). Four waves per workgroup, which strides over the templates.
template <bool EXPL, bool HW, int MAPT>
__global__ __launch_bounds__(256) void k_score_md_wave(MapP m, GenP g, const Trk *tr, uint64_t first, int64_t n,
                                                       int32_t norm, int32_t d0, int32_t step, int32_t m0, int32_t cnt,
                                                       int32_t last, float *snr, int32_t *tidx, uint64_t *best)
{
    __shared__ float gsum[4][64][kMD + 1];  // one round of groups per wave; padded rows spread the banks
    const DelayGrid dg = delay_grid(m, d0, step, m0, cnt);
    const int lane = threadIdx.x & 63;
    float (*gs)[kMD + 1] = gsum[threadIdx.x >> 6];
    uint64_t key = 0;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {  // wave-uniform
        const Trk t = EXPL ? tr[i] : draw_track(g, first + (uint64_t)i);
        float z = __builtin_nanf("");
        int32_t mi = -1;
        if (!EXPL || track_ok(t, m)) {
            const int gfirst = t.t0 / kFlush, glast = t.t2 / kFlush;
            double acc = 0.0;  // of delay `lane` in lanes 0 .. kMD - 1
            for (int r0 = gfirst; r0 <= glast; r0 += 64) {
                const int gi = r0 + lane;
                if (gi <= glast) {
                    DdaF st = ddaf_init_at(t, gi * kFlush - t.t0);
                    float part[kMD];
                    group_sums_md<HW, MAPT>(m, dg, gi * kFlush, t.t0, t.t2, st, part);
#pragma unroll
                    for (int q = 0; q < kMD; ++q) gs[lane][q] = part[q];
                }
                wave_lds_sync();
                if (lane < kMD)
                    for (int l = 0; l < min(64, glast - r0 + 1); ++l) acc += gs[l][lane];
                wave_lds_sync();
            }
            const int32_t N = t.t2 - t.t0 + 1;
            const float v = lane < dg.cnt ? finish(acc, N, norm, m.scale) : -__builtin_inff();
            if (!__builtin_amdgcn_ballot_w64(v != v)) {
                // largest score, then lowest delay: the scores' ordered bits with the delay's complement
                const uint64_t kq = lane < dg.cnt ? key_encode(v, (uint32_t)lane) : 0;
                const uint64_t top = wave_max_u64(kq);
                mi = (int32_t)(0xFFFFFFFFu - (uint32_t)top);
                z = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), mi));
                mi += dg.m0;
            }
        }
        merge_running(z, mi, m0 ? snr[i] : 0.0f, m0 ? tidx[i] : 0, m0 == 0);
        if (lane == 0) {
            snr[i] = z;
            tidx[i] = mi;
        }
        if (last) {
            const uint64_t k = key_encode(z, (uint32_t)(first + (uint64_t)i));
            key = k > key ? k : key;
        }
    }
    if (last) merge_key(best, key);
}

// Column walk of the delay-maximised slab scorer (as walk, with kMD delays).
template <int TPT, bool MASK, bool HW, typename E>
__device__ __forceinline__ void walk_md(int ca, int cb, int c0, const E *slab, int ldc,
                                        const int32_t (&t0)[TPT], const uint32_t (&span)[TPT], const DelayGrid &dg,
                                        DdaF (&st)[TPT], float (&part)[TPT][kMD], double (&acc)[TPT][kMD])
{
    for (int c = ca; c <= cb;) {
        const int ce = min(cb, c | (kFlush - 1));
        for (; c <= ce; ++c) {
            const E *col = slab + (c - c0) * ldc;
#pragma unroll
            for (int q = 0; q < TPT; ++q) {
                const int32_t row = ddaf_row(st[q]);
                const bool act = !MASK || (uint32_t)c - (uint32_t)t0[q] <= span[q];
                const E p = col[act ? row : 0];
                add_terms_md<HW, MASK>(part[q], dg, row, p, act);
                ddaf_step(st[q]);
            }
        }
        if ((ce & (kFlush - 1)) == kFlush - 1) {  // wave-uniform
#pragma unroll
            for (int q = 0; q < TPT; ++q)
#pragma unroll
                for (int k = 0; k < kMD; ++k) { acc[q][k] += part[q][k]; part[q][k] = 0.0f; }
        }
    }
}

// Slab scorer of the delay grid: the folded map streamed into LDS by DMA as in
// score_block, WG lanes x TPT binned templates per workgroup; on the last launch
// each workgroup stores its best key in wg_keys[blockIdx.x].
template <int WG, int TPT, bool EXPL, bool HW, int MAPT>
__global__ __launch_bounds__(WG) void k_score_md_slab(MapP m, GenP g, const Trk *tr, const uint32_t *order,
                                                      uint64_t first, int64_t n, int S, int32_t norm, int32_t d0,
                                                      int32_t step, int32_t m0, int32_t cnt, int32_t last, float *snr,
                                                      int32_t *tidx, uint64_t *wg_keys)
{
    extern __shared__ float2 slab[];
    __shared__ int bnd[2];
    __shared__ uint64_t kred[WG / 64];
    if (threadIdx.x == 0) { bnd[0] = 0x7fffffff; bnd[1] = -1; }
    const DelayGrid dg = delay_grid(m, d0, step, m0, cnt);
    const int lane = threadIdx.x & 63;
    const int64_t wbase = (int64_t)blockIdx.x * (WG * TPT) + (int64_t)(threadIdx.x >> 6) * (64 * TPT);
    Trk tk[TPT];
    int32_t t0[TPT];
    uint32_t span[TPT], idx[TPT];
    bool ok[TPT], live[TPT];
    int lo = 0x7fffffff, hi = -1, clo = -1, chi = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        const int64_t e = wbase + q * 64 + lane;
        live[q] = e < n;
        idx[q] = live[q] ? order[e] : 0u;
        Trk t = EXPL ? tr[idx[q]] : draw_track(g, first + idx[q]);
        ok[q] = live[q] && (!EXPL || track_ok(t, m));
        if (!ok[q]) t = Trk{0, 1, 0u, 0u, 0u, 0};
        tk[q] = t;
        t0[q] = ok[q] ? t.t0 : 0x7fffffff;
        span[q] = ok[q] ? (uint32_t)(t.t2 - t.t0) : 0u;
        if (ok[q]) {
            lo = min(lo, t.t0);
            hi = max(hi, t.t2);
            clo = max(clo, t.t0);
            chi = min(chi, t.t2);
        } else {
            clo = 0x7fffffff;
            chi = -1;
        }
    }
    lo = wave_min_i32(lo);
    hi = wave_max_i32(hi);
    clo = wave_max_i32(clo);
    chi = wave_min_i32(chi);
    if (clo > chi) { clo = hi + 1; chi = hi; }
    DdaF st[TPT];
    float part[TPT][kMD];
    double acc[TPT][kMD];
    const int start = lo == 0x7fffffff ? 0 : lo;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        st[q] = ddaf_init_at(tk[q], start - tk[q].t0);
#pragma unroll
        for (int k = 0; k < kMD; ++k) { part[q][k] = 0.0f; acc[q][k] = 0.0; }
    }
    __syncthreads();
    if (lane == 0) {
        atomicMin(&bnd[0], lo);
        atomicMax(&bnd[1], hi);
    }
    __syncthreads();
    const int c_first = __builtin_amdgcn_readfirstlane(bnd[0]), c_last = __builtin_amdgcn_readfirstlane(bnd[1]);
    using E = elem_t<MAPT>;
    const int ldc = (int)m.ld;
    const SlabDma<WG / 64> dma(m, (int)sizeof(E));
    const uint32_t buf0 = lds_addr(slab), slab_bytes = (uint32_t)S * dma.col_bytes;
    if (c_first <= c_last) dma.issue(c_first, min(S, c_last - c_first + 1), buf0);
    int kk = 0;
    for (int c0 = c_first; c0 <= c_last; c0 += S, ++kk) {
        slab_sync();  // slab kk has landed and slab kk-1 is no longer read
        if (c0 + S <= c_last) dma.issue(c0 + S, min(S, c_last - c0 - S + 1), buf0 + ((kk + 1) & 1) * slab_bytes);
        const E *cur = reinterpret_cast<const E *>(reinterpret_cast<const char *>(slab) + (size_t)(kk & 1) * slab_bytes);
        const int ncol = min(S, c_last - c0 + 1);
        const int ca = max(c0, lo), cb = min(c0 + ncol - 1, hi);
        walk_md<TPT, true, HW>(ca, min(cb, clo - 1), c0, cur, ldc, t0, span, dg, st, part, acc);
        walk_md<TPT, false, HW>(max(ca, clo), min(cb, chi), c0, cur, ldc, t0, span, dg, st, part, acc);
        walk_md<TPT, true, HW>(max(ca, chi + 1), cb, c0, cur, ldc, t0, span, dg, st, part, acc);
    }
    uint64_t key = 0;
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
        if (!live[q]) continue;
        float z;
        int32_t mi;
        merge_delays(acc[q], part[q], (int32_t)span[q] + 1, norm, m.scale, dg, ok[q], z, mi);
        merge_running(z, mi, m0 ? snr[idx[q]] : 0.0f, m0 ? tidx[idx[q]] : 0, m0 == 0);
        snr[idx[q]] = z;
        tidx[idx[q]] = mi;
        const uint64_t k = key_encode(z, (uint32_t)(first + idx[q]));
        key = k > key ? k : key;
    }
    if (!last) return;  // uniform: every workgroup of a launch has the same flag
    key = wave_max_u64(key);
    if (lane == 0) kred[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < WG / 64; ++w) key = kred[w] > key ? kred[w] : key;
        wg_keys[blockIdx.x] = key;
    }
}

// ---------------------------------------------------------------- batches of maps
// A batch scores n_m generated templates on each map m (the paper's n_ts
// time-shifted background maps, Sec. V). Map m's templates are binned within
// the map; its blocks of WG*TPT binned templates are the work items
// [item0[m], item0[m+1]). One persistent launch: each workgroup takes the
// next item from an atomic queue until the queue is empty, so maps of uneven
// length share the machine without a tail per map.

struct BatchMap {
    MapP m;
    GenP g;
    int64_t n;          // templates on this map
    uint64_t order0;    // offset of this map's binned order in the shared order array
    uint64_t bin0;      // offset of this map's bucket counters
    int32_t wb, nbins;  // bucket shift and count of this map
    int32_t S;          // slab columns
    int32_t chunk0;     // first sort chunk of this map
    uint64_t cc0;       // offset of this map's counts per group and sort chunk
    float *snr;         // optional per-template output
};

__global__ __launch_bounds__(256) void k_bin_count_batch(const BatchMap *maps, int n_maps, const uint32_t *chunk_start,
                                                         uint32_t *totals, uint16_t *bins, uint32_t *ccnt)
{
    __shared__ uint32_t hist[kMaxBins];
    const int mi = find_slot(chunk_start, n_maps, blockIdx.x);
    const BatchMap &d = maps[mi];
    for (int b = threadIdx.x; b < d.nbins; b += 256) hist[b] = 0;
    __syncthreads();
    const uint32_t c = blockIdx.x - chunk_start[mi], cw = bucket_class(((uint32_t)(d.m.T - 1) >> d.wb) + 1);
    const int64_t base = (int64_t)c * kBinChunk;
    for (int q = 0; q < kBinPerThread; ++q) {
        const int64_t i = base + q * 256 + threadIdx.x;
        if (i < d.n) {
            const uint32_t b = bin_of<false>(d.g, nullptr, d.m, 0, i, d.wb, cw);
            bins[d.order0 + i] = (uint16_t)b;
            atomicAdd(&hist[b], 1u);
        }
    }
    __syncthreads();
    count_out(hist, d.nbins, totals + d.bin0, ccnt + d.cc0 + c, chunk_start[mi + 1] - chunk_start[mi]);
}

// The scans of a batch, 1 + max_groups workgroups per map: the first scans the
// map's buckets, offset by its order0 (tables at gstart/fitem + map index *
// kGroupSlots); workgroup k + 1 scans row k of the map's chunk counts.
__global__ __launch_bounds__(256) void k_bin_scan_batch(const BatchMap *maps, const uint32_t *chunk_start,
                                                        int max_groups, const uint32_t *totals, uint32_t *cursor,
                                                        uint32_t *gstart, uint32_t *fitem, uint32_t *ccnt)
{
    const int mi = blockIdx.x / (max_groups + 1), k = (int)(blockIdx.x % (max_groups + 1)) - 1;
    const BatchMap &d = maps[mi];
    if (k < 0) {
        const size_t t0 = (size_t)mi * kGroupSlots;
        scan_buckets<256>(totals + d.bin0, d.nbins, (uint32_t)d.order0, cursor + d.bin0, gstart + t0, fitem + t0);
    } else if (k < (d.nbins + kGroupMask) >> kGroupShift) {
        const uint32_t nc = chunk_start[mi + 1] - chunk_start[mi];
        scan_row(ccnt + d.cc0 + (size_t)k * nc, (int)nc);
    }
}

// The scatters of k_bin_group and k_bin_fine, each workgroup on one map's
// templates: sort chunks in map order (chunk_start), and for the second,
// fine_start[mi] = the map's first workgroup (it has its second-scatter chunk
// count plus its group count of them, an upper bound of its chunks of group
// regions).
__global__ __launch_bounds__(kScatterWG) void k_bin_group_batch(const BatchMap *maps, int n_maps, const uint32_t *chunk_start,
                                                         const uint16_t *bins, const uint32_t *gstart,
                                                         const uint32_t *ccnt, uint32_t *tmp, uint8_t *tsub)
{
    __shared__ GroupLds L;
    const int mi = find_slot(chunk_start, n_maps, blockIdx.x);
    const BatchMap &d = maps[mi];
    const uint32_t c = blockIdx.x - chunk_start[mi];
    const int64_t base = (int64_t)c * kBinChunk;
    group_chunk<kScatterWG>(L, (d.nbins + kGroupMask) >> kGroupShift, base, (int)min<int64_t>(kBinChunk, d.n - base),
                bins + d.order0, gstart + (size_t)mi * kGroupSlots, ccnt + d.cc0 + c,
                chunk_start[mi + 1] - chunk_start[mi], tmp, tsub);
}

__global__ __launch_bounds__(kScatterWG) void k_bin_fine_batch(const BatchMap *maps, int n_maps, const uint32_t *fine_start,
                                                        const uint32_t *gstart, const uint32_t *fitem, uint32_t *cursor,
                                                        const uint32_t *tmp, const uint8_t *tsub, uint32_t *order)
{
    __shared__ FineLds L;
    const int mi = find_slot(fine_start, n_maps, blockIdx.x);
    const BatchMap &d = maps[mi];
    const int ngroups = (d.nbins + kGroupMask) >> kGroupShift;
    const uint32_t *fi = fitem + (size_t)mi * kGroupSlots;
    const uint32_t *gs = gstart + (size_t)mi * kGroupSlots;
    const uint32_t w = blockIdx.x - fine_start[mi];
    if (w >= fi[ngroups]) return;
    const int k = find_slot(fi, ngroups, w);
    const uint32_t e0 = gs[k] + (w - fi[k]) * (uint32_t)kFineChunk;
    const int b0 = k << kGroupShift;
    fine_chunk<kScatterWG>(L, min(1 << kGroupShift, d.nbins - b0), (int)min<uint32_t>(kFineChunk, gs[k + 1] - e0), tmp + e0,
               tsub + e0, cursor + d.bin0 + b0, order);
}

// A record read by every lane at one address, kept in scalar registers (its plain loads would hold
// it in vector registers, which the scorer needs).
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    uint32_t w[sizeof(T) / 4];
    const uint32_t *src = reinterpret_cast<const uint32_t *>(p);
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(src[i]);
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

template <int WG, int TPT, bool HW, int MAPT, int SC>
__global__ __launch_bounds__(WG, (kSlabWavesPerSimd<TPT, SC>)) void k_score_batch(const BatchMap *maps, int n_maps,
                                                                       const uint32_t *item_start, uint32_t *queue,
                                                                       const uint32_t *order, int32_t norm,
                                                                       uint64_t *best)
{
    extern __shared__ float2 slab[];
    __shared__ int bnd[2];
    __shared__ uint64_t kred[WG / 64];
    __shared__ uint32_t item_s;
    const uint32_t total = item_start[n_maps];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) item_s = atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(item_s);
        if (item >= total) break;  // every workgroup reaches this: the queue only grows
        const int mi = __builtin_amdgcn_readfirstlane(find_slot(item_start, n_maps, item));
        const BatchMap d = load_uniform(maps + mi);
        const uint64_t key = score_block_any<WG, TPT, HW, MAPT, SC>(d.m, d.g, nullptr, order + d.order0, 0, d.n,
                                                                   (int64_t)(item - __builtin_amdgcn_readfirstlane(item_start[mi])), d.S, norm,
                                                                   d.snr, slab, bnd, kred);
        // one atomic per item, spread over the maps' keys
        if (threadIdx.x == 0 && key) atomicMax((unsigned long long *)(best + mi), (unsigned long long)key);
    }
}

// ---------------------------------------------------------------- FP16 map packing
// p = Y/sigma in FP32 (correctly rounded division). Its magnitude in FP64 (the
// FP32 components square exactly: one rounding of the sum, one of the square
// root) times 2^-e is rounded to binary16, round to nearest even straight from
// FP64; its argument atan2 / (2 pi) to the nearest 2^-16 turn (ties to even),
// modulo one turn. Word = argument | binary16 bits << 16. k_absmax_p finds the
// largest magnitude first (its FP64 bits: non-negative doubles order as
// integers), one atomic per workgroup of at most 1024: atomics on one address
// follow one another, 11 ns each, and one per wave of 2048 workgroups was 100 us.

__device__ __forceinline__ double p_mag64(float x, float y)
{
    const double dx = x, dy = y;
    return sqrt(fma(dx, dx, dy * dy));
}

// binary16 bits of a non-negative double below 65520, rounded to nearest, ties to even
__device__ __forceinline__ uint32_t f64_to_f16_rne(double d)
{
    const uint64_t b = (uint64_t)__double_as_longlong(d);
    if (b == 0) return 0;
    const int ex = (int)((b >> 52) & 0x7FF) - 1023;
    const uint64_t sig = (b & 0xFFFFFFFFFFFFFull) | (1ull << 52);  // d = sig * 2^(ex - 52)
    // normal results keep 11 significant bits (shift 42); subnormal ones count units of 2^-24
    const int shift = ex >= -14 ? 42 : 28 - ex;
    if (shift >= 64) return 0;  // below 2^-36: rounds to zero
    uint64_t q = sig >> shift;
    const uint64_t rem = sig & ((1ull << shift) - 1), half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (q & 1))) ++q;
    // a normal q in [2^10, 2^11]: exponent field plus fraction; the carry of q = 2^11 moves the exponent
    return ex >= -14 ? (uint32_t)(((uint32_t)(ex + 15) << 10) + (uint32_t)q - 1024u) : (uint32_t)q;
}

__global__ __launch_bounds__(256) void k_absmax_p(MapP m, unsigned long long *amax_bits)
{
    double mx = 0.0;
    const int64_t n = (int64_t)m.T * m.F;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t t = n >> 32 ? i / m.F : (int64_t)((uint32_t)i / (uint32_t)m.F), r = i - t * m.F;
        const int64_t e = t * m.ld + r;
        const float2 y = m.Y[e];
        const float sg = m.sig[e];
        mx = fmax(mx, p_mag64(y.x / sg, y.y / sg));
    }
    __shared__ double red[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        if (mx > 0.0) atomicMax(amax_bits, (unsigned long long)__double_as_longlong(mx));
    }
}

__global__ __launch_bounds__(256) void k_pack_p16(MapP m, double inv_scale, uint32_t *out, int64_t out_ld)
{
    const int64_t n = (int64_t)m.T * m.F;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t t = i / m.F, r = i - t * m.F;
        const int64_t e = t * m.ld + r;
        const float2 y = m.Y[e];
        const float sg = m.sig[e];
        const float px = y.x / sg, py = y.y / sg;
        const uint32_t mag = f64_to_f16_rne(p_mag64(px, py) * inv_scale);
        const double turns = atan2((double)py, (double)px) * 0.15915494309189535;  // 1 / (2 pi), rounded
        const uint32_t arg = (uint32_t)(int64_t)rint(turns * 65536.0) & 0xFFFFu;
        out[t * out_ld + r] = arg | (mag << 16);
    }
}

// ---------------------------------------------------------------- top-K
// Radix select over the 64-bit keys (score bits, ~index) -- all distinct -- by digits of 12 bits
// from the top, each pass a histogram of the keys that share the digits fixed so far. A pass may
// stop the select: once the keys at or above the chosen digit number at most kTopkCand they are
// gathered and ranked by comparison, each writing itself at its rank. Scores of real searches
// stop after the first pass (1/8 of an octave of the score), so the scores are read twice;
// degenerate arrays (all equal, all NaN) run every pass, and the index bits then leave exactly K.
// The later passes' launches return at once after a stop: nothing is read back by the host.
// Every workgroup of a pass finds the digit from the previous pass's histogram by itself, so no
// launch of its own chooses it. 2 x 10^7 scores, K = 1024: 8-bit digits with a scan launch each
// and a one-workgroup sort, 19 launches, took 221 us more than these 9. The gather takes 25 us (38
// with a cursor atomic and three barriers per batch of 8 elements a lane), the ranks 6 (11 by 4
// waves), a pass after the stop 2 to 5 us.
constexpr int kTopkBits = 12;
constexpr int kTopkBins = 1 << kTopkBits;
constexpr int kTopkPasses = 6;       // 5 x 12 + 4 bits
constexpr int kTopkCand = 16384;     // candidates ranked by comparison

// The select before pass p (p = kTopkPasses: its end).
struct TopkSel {
    uint64_t prefix;  // digits fixed so far, in place
    uint32_t shift;   // position of the lowest fixed digit (64: none)
    uint32_t need;    // how many of the K lie among the keys that share the prefix
    uint32_t above;   // keys above the prefix
    uint32_t done;    // the keys at or above the prefix are the candidates
};

struct TopkState {
    TopkSel sel[kTopkPasses + 1];
    uint32_t count;  // gather cursor
    uint32_t hist[kTopkPasses][kTopkBins];
};

__device__ __forceinline__ int topk_shift(int pass) { return max(0, 64 - kTopkBits * (pass + 1)); }

// Element i of a select's source as a key: a score array, or the scores of an array of best keys
// (an empty key counts as -inf).
struct TopkScores {
    const float *z;
    __device__ __forceinline__ float operator()(int64_t i) const { return z[i]; }
};
struct TopkKeys {
    const uint64_t *k;
    __device__ __forceinline__ float operator()(int64_t i) const
    {
        const uint32_t hi = (uint32_t)(k[i] >> 32);
        const uint32_t bits = (hi & 0x80000000u) ? (hi ^ 0x80000000u) : ~hi;  // undo the order-preserving map
        return hi == 0u ? -__builtin_inff() : __uint_as_float(bits);
    }
};

__global__ __launch_bounds__(1024) void k_topk_init(TopkState *st, uint32_t K)
{
    const int i = blockIdx.x * 1024 + threadIdx.x;
    if (i < kTopkPasses * kTopkBins) (&st->hist[0][0])[i] = 0;
    if (i == 0) {
        st->sel[0] = TopkSel{0, 64, K, 0, 0};
        st->count = 0;
    }
}

// The select before pass p >= 1 from the state and histogram before and of pass p - 1: the digit
// holding the need-th largest key. Called by the 256 threads of a workgroup; every workgroup
// computes the same, and the first stores it for the launches that follow.
__device__ __forceinline__ TopkSel topk_resolve(TopkState *st, int p)
{
    __shared__ uint32_t wsum[4];
    __shared__ TopkSel out;
    const TopkSel s = st->sel[p - 1];
    if (s.done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->sel[p] = s;
        return s;
    }
    // thread t takes bins from the top down: hi - 16 t .. hi - 16 t - 15
    constexpr int kPer = kTopkBins / 256;
    const uint32_t *h = st->hist[p - 1];
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        v[j] = h[kTopkBins - 1 - kPer * (int)threadIdx.x - j];
        sum += v[j];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t run = incl - sum;  // keys in bins above this thread's
    for (int w = 0; w < wv; ++w) run += wsum[w];
    if (run < s.need && run + sum >= s.need) {  // exactly one thread
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (run < s.need && run + v[j] >= s.need) {
                const uint32_t d = (uint32_t)(kTopkBins - 1 - kPer * (int)threadIdx.x - j);
                const int shift = topk_shift(p - 1);
                const uint32_t above = s.above + run;
                out = TopkSel{s.prefix | (uint64_t)d << shift, (uint32_t)shift, s.need - run, above,
                              above + v[j] <= (uint32_t)kTopkCand || p == kTopkPasses ? 1u : 0u};
            }
            run += v[j];
        }
    }
    __syncthreads();
    const TopkSel r = out;
    if (blockIdx.x == 0 && threadIdx.x == 0) st->sel[p] = r;
    return r;
}

template <typename SRC>
__global__ __launch_bounds__(256) void k_topk_hist(SRC src, int64_t n, uint64_t first, TopkState *st, int pass)
{
    __shared__ uint32_t h[kTopkBins];
    TopkSel s;
    if (pass > 0) s = topk_resolve(st, pass);
    else s = st->sel[0];
    if (s.done) return;  // uniform over the launch
    for (int i = threadIdx.x; i < kTopkBins; i += 256) h[i] = 0;
    __syncthreads();
    const int shift = topk_shift(pass);
    const uint32_t dmask = pass == kTopkPasses - 1 ? (1u << (64 - kTopkBits * (kTopkPasses - 1))) - 1u : kTopkBins - 1u;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < n; i0 += 4 * stride) {
        float z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) z[q] = i0 + q * stride < n ? src(i0 + q * stride) : 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = i0 + q * stride;
            if (i >= n) break;
            const uint64_t k = key_encode(z[q], (uint32_t)(first + (uint64_t)i));
            if (pass == 0 || k >> s.shift == s.prefix >> s.shift) atomicAdd(&h[(uint32_t)(k >> shift) & dmask], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kTopkBins; i += 256)
        if (h[i]) atomicAdd(&st->hist[pass][i], h[i]);
}

// The keys at or above the final prefix into cand (at most kTopkCand), by a list in LDS and one
// cursor atomic per workgroup; keys beyond the list take a cursor atomic each.
constexpr int kTopkList = 1024;

template <typename SRC>
__global__ __launch_bounds__(256) void k_topk_gather(SRC src, int64_t n, uint64_t first, TopkState *st, uint64_t *cand)
{
    __shared__ uint64_t list[kTopkList];
    __shared__ uint32_t cnt, base;
    if (threadIdx.x == 0) cnt = 0;
    const TopkSel s = topk_resolve(st, kTopkPasses);
    __syncthreads();
    const uint64_t thr = s.prefix >> s.shift;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < n; i0 += 8 * stride) {
        float z[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) z[q] = i0 + q * stride < n ? src(i0 + q * stride) : 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = i0 + q * stride;
            if (i >= n) break;
            const uint64_t k = key_encode(z[q], (uint32_t)(first + (uint64_t)i));
            if (k >> s.shift < thr) continue;
            const uint32_t at = atomicAdd(&cnt, 1u);
            if (at < (uint32_t)kTopkList) {
                list[at] = k;
            } else {
                const uint32_t o = atomicAdd(&st->count, 1u);
                if (o < (uint32_t)kTopkCand) cand[o] = k;  // the bound is a guard
            }
        }
    }
    __syncthreads();
    const uint32_t m = min(cnt, (uint32_t)kTopkList);
    if (threadIdx.x == 0 && m) base = atomicAdd(&st->count, m);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += 256)
        if (base + i < (uint32_t)kTopkCand) cand[base + i] = list[i];
}

// Rank of each candidate (64 per workgroup, a lane each; the 16 waves compare with a sixteenth of
// the candidates each): ranks below K are the answer, in order. last_only: val holds one score,
// that of rank K - 1.
__global__ __launch_bounds__(1024) void k_topk_rank(const TopkState *st, const uint64_t *cand, int K, int last_only,
                                                    int64_t *idx, float *val)
{
    constexpr int kTile = 4096;
    __shared__ uint64_t tile[kTile];
    __shared__ uint32_t rank[64];
    const int C = (int)min(st->count, (uint32_t)kTopkCand);
    const int e0 = blockIdx.x * 64;
    if (e0 >= C) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t k = e0 + lane < C ? cand[e0 + lane] : ~0ull;
    if (threadIdx.x < 64) rank[threadIdx.x] = 0;
    uint32_t r = 0;
    for (int t0 = 0; t0 < C; t0 += kTile) {
        const int tn = min(kTile, C - t0), per = (tn + 15) / 16;
        __syncthreads();
        for (int i = threadIdx.x; i < tn; i += 1024) tile[i] = cand[t0 + i];
        __syncthreads();
        const int q1 = min(wave * per + per, tn);
#pragma unroll 8
        for (int q = wave * per; q < q1; ++q) r += tile[q] > k;  // one LDS broadcast per key
    }
    atomicAdd(&rank[lane], r);
    __syncthreads();
    if (threadIdx.x >= 64 || e0 + lane >= C) return;
    r = rank[lane];
    if (r >= (uint32_t)K || (last_only && r != (uint32_t)K - 1)) return;
    const uint32_t o = (uint32_t)(k >> 32);
    const uint32_t b = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    if (idx) idx[r] = (int64_t)(0xFFFFFFFFu - (uint32_t)k);
    if (val) val[last_only ? 0 : r] = __uint_as_float(b);
}

// ---------------------------------------------------------------- FP64 re-score
// One wave per template: lanes stride over its columns; each pixel's row is
// the exact floor of Eq. 6 by 64-bit integer division, the phase the exact
// 2^-32-turn integer, the term and the sum in FP64 (fixed-order wave
// reduction, so the result is deterministic).

template <bool EXPL>
__global__ __launch_bounds__(256) void k_rescore_f64(MapP m, GenP g, const Trk *tr, int64_t ntr, uint64_t first,
                                                     const int64_t *idx, int32_t K, int32_t norm, double *out)
{
    const int w = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (w >= K) return;
    const int64_t j = idx[w];
    Trk t;
    bool ok;
    if (EXPL) {
        ok = j >= (int64_t)first && j - (int64_t)first < ntr;
        t = tr[ok ? j - (int64_t)first : 0];
        ok = ok && track_ok(t, m);
    } else {
        ok = j >= 0 && j < ((int64_t)1 << 32);
        t = draw_track(g, (uint64_t)j);
    }
    double s = 0.0;
    int32_t N = 1;
    if (ok) {
        const int64_t Dt = t.t2 - t.t0;
        N = (int32_t)Dt + 1;
        const uint64_t Q = (uint64_t)(Dt * Dt) << 8;
        for (int64_t k = lane; k <= Dt; k += 64) {
            const uint64_t a = (uint64_t)(Dt - k), b = (uint64_t)k;
            const uint64_t num = a * a * t.f0 + 2 * a * b * t.f1 + b * b * t.f2;
            const int64_t row = (int64_t)(num / Q);
            const int64_t e = (t.t0 + k) * m.ld + row;
            const double sg = m.sig[e];
            const double pr = (double)m.Y[e].x / sg, pim = (double)m.Y[e].y / sg;
            const uint32_t ph = (uint32_t)((int64_t)(m.fq4_lo + row * m.dfq4) * (int64_t)t.dtau);
            double sn, cs;
            sincos(6.283185307179586 * ((double)(int32_t)ph * 2.3283064365386963e-10), &sn, &cs);
            s += cs * pr - sn * pim;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) out[w] = ok ? (norm == 1 ? s / N : s / sqrt((double)N)) : __builtin_nan("");
}

// ---------------------------------------------------------------- smooth SNR and its gradient
// theta = (tau0, tau2, phi0, phi1, phi2, dtau_ms) per template, K samples
// xi_k = k/(K-1); sample (u, v) = (clamp(t_k, 0, T-1), clamp(f_k - 1/2, 0, F-1)),
// bilinear interpolation of G(t, r) = Re[exp(2 pi i f(r) dtau) p(t, r)] and
// of its dtau-derivative; z~ = K^-1/2 sum. One wave per template, lanes over
// samples; sums in FP64, reduced in a fixed order (deterministic).

// cos and sin of a row's phase and its frequency, shared by the row's nodes.
struct RowPhase {
    float c, s, w;  // w = -2 pi f
};

__device__ __forceinline__ RowPhase row_phase(const MapP &m, int r, double dtau_s)
{
    const double f_hz = (double)(m.fq4_lo + (int64_t)r * m.dfq4) * 0.0625;
    double turns = f_hz * dtau_s;
    turns -= floor(turns);
    const float x = (float)turns;
    return {__builtin_amdgcn_cosf(x), __builtin_amdgcn_sinf(x), -6.283185307179586f * (float)f_hz};
}

__device__ __forceinline__ void smooth_node(float2 p, const RowPhase &h, float &g, float &gd)
{
    g = h.c * p.x - h.s * p.y;
    gd = h.w * (h.s * p.x + h.c * p.y);
}

// p of rows r and r + 1 of two neighbouring columns, element e = (i, r) of the map: p[column][row].
// A lane's second column is its neighbour's first, and a wave's loads of one column fill up to 64
// cache lines of Y and 64 of sigma. The four loads of an FP32 map go out back to back, by array:
// with address arithmetic or the other array's load in between, the lines of the first column have
// left the L1 when the second one asks for them (20 000 templates on 1000 x 1000, 1000 samples each:
// 269 us, back to back 225; 500 samples 224 and 208).
template <int MAPT>
__device__ __forceinline__ void load_p22(const MapP &m, int64_t e, float2 (&p)[2][2])
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(8)));
    if constexpr (MAPT == kMapF32) {
        typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
        typedef const __attribute__((address_space(1))) f4 *g4;
        typedef const __attribute__((address_space(1))) f2 *g2;
        uint64_t s0 = (uint64_t)(m.sig + e), s1 = (uint64_t)(m.sig + e + m.ld);
        uint64_t y0 = (uint64_t)(m.Y + e), y1 = (uint64_t)(m.Y + e + m.ld);
        asm volatile("" : "+v"(s0), "+v"(s1), "+v"(y0), "+v"(y1));  // all addresses before the first load
        __builtin_amdgcn_sched_barrier(0);
        const f2 s[2] = {*(g2)s0, *(g2)s1};
        __builtin_amdgcn_sched_barrier(0);
        const f4 y[2] = {*(g4)y0, *(g4)y1};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float w0 = 1.0f / s[c].x, w1 = 1.0f / s[c].y;
            p[c][0] = make_float2(y[c].x * w0, y[c].y * w0);
            p[c][1] = make_float2(y[c].z * w1, y[c].w * w1);
        }
    } else if constexpr (MAPT == kMapPF) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const f4 v = *reinterpret_cast<const f4 *>(m.Y + e + c * m.ld);
            p[c][0] = make_float2(v.x, v.y);
            p[c][1] = make_float2(v.z, v.w);
        }
    } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            p[c][0] = load_p<MAPT>(m, e + c * m.ld);
            p[c][1] = load_p<MAPT>(m, e + c * m.ld + 1);
        }
    }
}

// Sums of 8 values over the wave, value q in the lanes with lane % 8 == q on return. The first three
// exchanges halve what each lane carries (10 exchanges for all 8; value by value they were 48).
__device__ __forceinline__ double wave_sum8(const double (&x)[8])
{
    const int lane = threadIdx.x & 63;
    double y[4], z[2];
    const bool h4 = lane & 4, h2 = lane & 2, h1 = lane & 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] = (h4 ? x[q + 4] : x[q]) + __shfl_xor(h4 ? x[q] : x[q + 4], 4);
#pragma unroll
    for (int q = 0; q < 2; ++q) z[q] = (h2 ? y[q + 2] : y[q]) + __shfl_xor(h2 ? y[q] : y[q + 2], 2);
    double v = (h1 ? z[1] : z[0]) + __shfl_xor(h1 ? z[0] : z[1], 1);
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// One workgroup of kSmoothWG lanes per template (lanes over the K samples):
// the bilinear gathers miss L2, so several waves per template keep more of
// them in flight than one wave could.
constexpr int kSmoothWG = 256;

// The smooth statistic of one template at th[0..5] (readable by every lane) and its gradient; all
// kSmoothWG lanes of the workgroup call it. Lane k sums samples k, k + kSmoothWG, ...; waves reduce
// by shuffles and the waves' sums are added in order, so the result does not depend on timing.
// Results (z, grad[0..5]) are valid in the lanes of wave 0. rK = 1 / (K - 1) in FP64, 0 for K <= 1.
// Bound by FP64 issue and, before it shared the phase of a row between its two nodes, took k / (K-1)
// by one correction of k rK (exactly the quotient: rK is the rounded reciprocal, and quotients of
// integers below 2^31 are not near a rounding boundary) and transposed the seven sums as they
// shrink, by twice the sines and 84 LDS exchanges per wave.
template <int MAPT>
__device__ __forceinline__ void smooth_block(const MapP &m, const float *th, int K, double rK, double (*red)[8],
                                             float &z_out, float (&grad)[6])
{
    const double tau0 = th[0], tau2 = th[1], ph0 = th[2], ph1 = th[3], ph2 = th[4];
    const double dtau_s = (double)th[5] * 1e-3;
    double sum[8] = {};  // z, then the gradient
    for (int k = threadIdx.x; k < K; k += kSmoothWG) {
        const double kd = (double)k, q0 = kd * rK;
        const double xi = fma(fma(-q0, (double)(K - 1), kd), rK, q0);
        const double b0 = (1 - xi) * (1 - xi), b1 = 2 * xi * (1 - xi), b2 = xi * xi;
        const double u0 = tau0 + xi * (tau2 - tau0), v0 = b0 * ph0 + b1 * ph1 + b2 * ph2 - 0.5;
        // clamp into the map (fmax/fmin also send a NaN coordinate to the lower edge)
        const double u = fmin(fmax(u0, 0.0), (double)(m.T - 1)), v = fmin(fmax(v0, 0.0), (double)(m.F - 1));
        const bool ut = u0 >= 0.0 && u0 <= (double)(m.T - 1), vt = v0 >= 0.0 && v0 <= (double)(m.F - 1);
        const int i = min((int)floor(u), m.T - 2), r = min((int)floor(v), m.F - 2);
        const double a = u - (double)i, b = v - (double)r;
        float2 p[2][2];
        load_p22<MAPT>(m, i * m.ld + r, p);
        const RowPhase h0 = row_phase(m, r, dtau_s), h1 = row_phase(m, r + 1, dtau_s);
        float G00, G10, G01, G11, D00, D10, D01, D11;
        smooth_node(p[0][0], h0, G00, D00);
        smooth_node(p[1][0], h0, G10, D10);
        smooth_node(p[0][1], h1, G01, D01);
        smooth_node(p[1][1], h1, G11, D11);
        const double w00 = (1 - a) * (1 - b), w10 = a * (1 - b), w01 = (1 - a) * b, w11 = a * b;
        sum[0] += w00 * G00 + w10 * G10 + w01 * G01 + w11 * G11;
        const double du = ut ? (1 - b) * (G10 - G00) + b * (G11 - G01) : 0.0;
        const double dv = vt ? (1 - a) * (G01 - G00) + a * (G11 - G10) : 0.0;
        sum[1] += (1 - xi) * du;
        sum[2] += xi * du;
        sum[3] += b0 * dv;
        sum[4] += b1 * dv;
        sum[5] += b2 * dv;
        sum[6] += (w00 * D00 + w10 * D10 + w01 * D01 + w11 * D11) * 1e-3;
    }
    const double v = wave_sum8(sum);
    if ((threadIdx.x & 63) < 8) red[threadIdx.x >> 6][threadIdx.x & 7] = v;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double sc = K > 0 ? 1.0 / sqrt((double)K) : 0.0;
        float out[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            double t = red[0][q];
#pragma unroll
            for (int w = 1; w < kSmoothWG / 64; ++w) t += red[w][q];
            out[q] = (float)(t * sc);
        }
        z_out = out[0];
#pragma unroll
        for (int q = 0; q < 6; ++q) grad[q] = out[q + 1];
    }
}

__device__ __forceinline__ double sample_step(int K) { return K > 1 ? 1.0 / (double)(K - 1) : 0.0; }

template <int MAPT>
__global__ __launch_bounds__(kSmoothWG, 4) void k_smooth_grad(MapP m, const float *theta, const int32_t *Ks, int32_t n,
                                                           float *z_out, float *grad_out)
{
    __shared__ double red[kSmoothWG / 64][8];
    const int w = blockIdx.x;
    if (w >= n) return;  // whole workgroup
    const int K = Ks[w];
    float z, g[6];
    smooth_block<MAPT>(m, theta + (int64_t)w * 6, K, sample_step(K), red, z, g);
    if (threadIdx.x == 0) {
        z_out[w] = z;
        if (grad_out) {
            for (int q = 0; q < 6; ++q) grad_out[(int64_t)w * 6 + q] = g[q];
        }
    }
}

// ---------------------------------------------------------------- refinement helpers

__global__ __launch_bounds__(256) void k_tracks_at(GenP g, const int64_t *idx, int64_t n, Trk *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = draw_track(g, (uint64_t)idx[i]);
}

// A plain template's parameters as a smooth-SNR point: times as columns,
// control frequencies in rows, delay in ms; K = its pixel count.
__global__ __launch_bounds__(256) void k_track_to_theta(const Trk *tr, int64_t n, float *theta, int32_t *Ks)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const Trk t = tr[i];
    float *th = theta + i * 6;
    th[0] = (float)t.t0;
    th[1] = (float)t.t2;
    th[2] = (float)t.f0 * (1.0f / 256.0f);
    th[3] = (float)t.f1 * (1.0f / 256.0f);
    th[4] = (float)t.f2 * (1.0f / 256.0f);
    th[5] = (float)((double)t.dtau * (1e3 / 268435456.0));
    Ks[i] = t.t2 - t.t0 + 1;
}

struct RefineP {
    int32_t T, F, L;
    double dmax_ms;
    double px0, px1, ms0, ms1;
    int32_t steps;
};

__device__ __forceinline__ void project_theta(double *th, const RefineP &p)
{
    double a = th[0], b = th[1];
    if (b - a < p.L - 1) {
        const double mid = 0.5 * (a + b);
        a = mid - 0.5 * (p.L - 1);
        b = mid + 0.5 * (p.L - 1);
    }
    if (a < 0) { b -= a; a = 0; }
    if (b > p.T - 1) { a -= b - (p.T - 1); b = p.T - 1; }
    if (a < 0) a = 0;
    th[0] = a;
    th[1] = b;
    const double fhi = (double)p.F - 1.0 / 512.0;
    for (int q = 2; q < 5; ++q) th[q] = fmin(fhi, fmax(0.0, th[q]));
    th[5] = fmin(p.dmax_ms, fmax(-p.dmax_ms, th[5]));
}

// Ascent step s of a template at th (FP32 parameters, updated in place) with
// gradient g: the five positions move by eta_px * g / |g|, the delay by
// eta_ms * sign(g), with the step sizes falling linearly over the steps; then
// projection onto the feasible set.
__device__ __forceinline__ void refine_move(float *th, const float *g, int32_t s, const RefineP &p)
{
    const double w = p.steps > 1 ? (double)s / (double)(p.steps - 1) : 0.0;
    const double epx = p.px0 + w * (p.px1 - p.px0), ems = p.ms0 + w * (p.ms1 - p.ms0);
    double t[6];
    for (int q = 0; q < 6; ++q) t[q] = th[q];
    double n2 = 0;
    for (int q = 0; q < 5; ++q) n2 += (double)g[q] * g[q];
    if (n2 > 0) {
        const double inv = 1.0 / sqrt(n2);
        for (int q = 0; q < 5; ++q) t[q] += epx * g[q] * inv;
    }
    if (g[5] > 0) t[5] += ems;
    else if (g[5] < 0) t[5] -= ems;
    project_theta(t, p);
    for (int q = 0; q < 6; ++q) th[q] = (float)t[q];
}

// The whole refinement of one template in one workgroup: project the start,
// then for s = 0..steps evaluate the smooth statistic and its gradient at the
// current point, keep the point if it is the best so far (s = 0 starts the
// best), and, while s < steps, take ascent step s. theta holds the start on
// entry and the best point on exit; best_z receives its smooth statistic.
template <int MAPT>
__global__ __launch_bounds__(kSmoothWG, 4) void k_refine(MapP m, float *theta, const int32_t *Ks, int32_t n,
                                                      float *best_z, RefineP p)
{
    __shared__ double red[kSmoothWG / 64][8];
    __shared__ float cur[6];
    const int w = blockIdx.x;
    if (w >= n) return;  // whole workgroup
    float *th_io = theta + (int64_t)w * 6;
    float th[6], best[6], bz = 0.0f, z, g[6];  // of wave 0, the same in all its lanes
    if (threadIdx.x < 64) {
        double t[6];
        for (int q = 0; q < 6; ++q) t[q] = th_io[q];
        project_theta(t, p);
        for (int q = 0; q < 6; ++q) th[q] = best[q] = (float)t[q];
        if (threadIdx.x == 0)
            for (int q = 0; q < 6; ++q) cur[q] = th[q];
    }
    __syncthreads();
    const int K = Ks[w];
    const double rK = sample_step(K);
    for (int32_t s = 0; s <= p.steps; ++s) {
        smooth_block<MAPT>(m, cur, K, rK, red, z, g);
        if (threadIdx.x < 64) {
            if (s == 0 || z > bz) {
                bz = z;
                for (int q = 0; q < 6; ++q) best[q] = th[q];
            }
            if (s < p.steps) {
                refine_move(th, g, s, p);
                if (threadIdx.x == 0)
                    for (int q = 0; q < 6; ++q) cur[q] = th[q];
            }
        }
        __syncthreads();  // the new point is visible; red may be reused
    }
    if (threadIdx.x == 0) {
        for (int q = 0; q < 6; ++q) th_io[q] = best[q];
        best_z[w] = bz;
    }
}

// Back to a plain template (times half up, widened to L pixels; frequencies
// floor(256 phi) inside the band; delay to the nearest 2^-28 s, clipped).
__global__ __launch_bounds__(256) void k_theta_to_track(const float *theta, int64_t n, int32_t T, int32_t F, int32_t L,
                                                        int32_t dtau_max, Trk *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float *th = theta + i * 6;
    // rounded and clamped in FP64 before converting, so any input stays inside the map
    int32_t t0 = (int32_t)fmin(fmax(floor((double)th[0] + 0.5), 0.0), (double)(T - 1));
    int32_t t2 = (int32_t)fmin(fmax(floor((double)th[1] + 0.5), 0.0), (double)(T - 1));
    if (t2 - t0 < L - 1) {
        t2 = t0 + L - 1;
        if (t2 > T - 1) { t0 -= t2 - (T - 1); t2 = T - 1; }
    }
    Trk t;
    t.t0 = t0;
    t.t2 = t2;
    uint32_t f[3];
    for (int q = 0; q < 3; ++q) {
        double v = floor((double)th[2 + q] * 256.0);
        v = fmin(fmax(v, 0.0), (double)F * 256 - 1);
        f[q] = (uint32_t)v;
    }
    t.f0 = f[0];
    t.f1 = f[1];
    t.f2 = f[2];
    double d = floor((double)th[5] * 1e-3 * 268435456.0 + 0.5);
    d = fmin(fmax(d, -(double)dtau_max), (double)dtau_max);
    t.dtau = (int32_t)d;
    out[i] = t;
}

}  // namespace stt
