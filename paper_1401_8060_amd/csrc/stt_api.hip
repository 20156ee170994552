// stt_api.hip -- host side of libstt: contexts, argument validation, scratch,
// launch configuration and the extern "C" entry points declared in stt.h.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include "stt.h"
#include "kernels.hpp"
#include "mapform.hpp"
#include "signif.hpp"

using namespace stt;

struct Rec {
    size_t base;  // first of the call's six events in the pool
    bool used[3];
};

constexpr int kLdsBytes = 160 * 1024;  // LDS of a CU, the default slab budget
constexpr int64_t kL2Bytes = 4 << 20;  // L2 of an XCD

struct stt_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    void *scratch = nullptr;
    size_t scratch_bytes = 0;
    void *aux = nullptr;  // top-K state and candidates, packing's maximum, follow-up ranks
    size_t aux_bytes = 0;
    void *pbuf = nullptr;  // folded p = Y/sigma maps for LDS-DMA staging
    size_t pbuf_bytes = 0;
    void *mdbuf = nullptr;  // running maxima of delay-grid scoring when the caller keeps none
    size_t mdbuf_bytes = 0;
    bool dma = true;       // fold + double-buffered LDS-DMA staging where a column fits
    int path = 0;  // 0 auto, 1 direct, 2 slab
    int lds_bytes = kLdsBytes;   // slab budget per workgroup
    int slab_wg = 1024;          // slab scorer shape: lanes per workgroup
    int slab_tpt = 4;            //                    templates per lane
    bool shape_set = false;      // by the caller or a tuner; else, and with the default budget, calls choose by size
    bool hw_trig = true;         // hardware sine/cosine (measured max error 1.3e-7) or the polynomial
    // Timing: every call takes six events from a pool (start/end of the scoring
    // kernel, of the binning kernels and of the whole call); queries sum them.
    bool timing = false;
    std::vector<hipEvent_t> pool;
    size_t next = 0;         // first free event of the pool
    size_t last = 0;         // first event of the last call
    bool used[3] = {false, false, false};
    // events that the next launch_ev records from its own dispatch (its start, its end)
    hipEvent_t kev_start = nullptr, kev_stop = nullptr;
    std::vector<Rec> recs;   // calls since the last total query
    // Batches: descriptor tables on the device, and the captured graph of the
    // last batch (replayed while the arguments stay the same).
    bool use_graph = true;
    hipStream_t cap_stream = nullptr;
    void *bdev = nullptr;
    size_t bdev_bytes = 0;
    std::vector<uint8_t> bkey;
    hipGraph_t graph = nullptr;
    hipGraphExec_t gexec = nullptr;
    int n_cu = 0;
    // map formation: FFT twiddles and window of the current column length
    void *fft_tab = nullptr;
    int fft_M = 0;
};

namespace {

stt_status fail(stt_ctx *c, stt_status s, const char *fmt, ...)
    __attribute__((format(printf, 3, 4)));

stt_status fail(stt_ctx *c, stt_status s, const char *fmt, ...)
{
    if (c) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        c->err = buf;
    }
    return s;
}

#define STT_HIP(c, call)                                                                      \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return fail((c), STT_EHIP, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

stt_status ensure_scratch(stt_ctx *c, size_t bytes)
{
    if (bytes <= c->scratch_bytes) return STT_OK;
    if (c->scratch) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return fail(c, STT_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
        (void)hipFree(c->scratch);
        c->scratch = nullptr;
        c->scratch_bytes = 0;
    }
    size_t want = std::max(bytes, (size_t)1 << 20);
    if (hipMalloc(&c->scratch, want) != hipSuccess) {
        (void)hipGetLastError();
        c->scratch = nullptr;
        return fail(c, STT_ENOMEM, "cannot allocate %zu bytes of scratch", want);
    }
    c->scratch_bytes = want;
    return STT_OK;
}

// What a top-K select needs of aux: its state and its candidates.
constexpr size_t kTopkStateBytes = (sizeof(TopkState) + 255) & ~(size_t)255;
constexpr size_t kTopkBytes = kTopkStateBytes + sizeof(uint64_t) * (size_t)kTopkCand;

// At least a select's need at once: after any call that uses aux a select allocates nothing (it may be
// recorded in a graph), and aux moves only for follow-ups of more maps than that holds ranks.
stt_status ensure_aux(stt_ctx *c, size_t bytes)
{
    if (bytes <= c->aux_bytes) return STT_OK;
    bytes = std::max(bytes, kTopkBytes);
    if (c->aux) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return fail(c, STT_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
        (void)hipFree(c->aux);
        c->aux = nullptr;
        c->aux_bytes = 0;
    }
    if (hipMalloc(&c->aux, bytes) != hipSuccess) {
        (void)hipGetLastError();
        c->aux = nullptr;
        return fail(c, STT_ENOMEM, "cannot allocate %zu bytes", bytes);
    }
    c->aux_bytes = bytes;
    return STT_OK;
}

stt_status ensure_pbuf(stt_ctx *c, size_t bytes)
{
    if (bytes <= c->pbuf_bytes) return STT_OK;
    if (c->pbuf) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return fail(c, STT_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
        (void)hipFree(c->pbuf);
        c->pbuf = nullptr;
        c->pbuf_bytes = 0;
    }
    if (hipMalloc(&c->pbuf, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, STT_ENOMEM, "cannot allocate %zu bytes for the folded map", bytes);
    }
    c->pbuf_bytes = bytes;
    return STT_OK;
}

stt_status ensure_mdbuf(stt_ctx *c, size_t bytes)
{
    if (bytes <= c->mdbuf_bytes) return STT_OK;
    if (c->mdbuf) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return fail(c, STT_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
        (void)hipFree(c->mdbuf);
        c->mdbuf = nullptr;
        c->mdbuf_bytes = 0;
    }
    if (hipMalloc(&c->mdbuf, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, STT_ENOMEM, "cannot allocate %zu bytes of delay-grid maxima", bytes);
    }
    c->mdbuf_bytes = bytes;
    return STT_OK;
}

// Column stride of a folded map and the slab depth that two buffers of it allow.
// Bytes per pixel of the folded map the scorers read: 8 for an FP32 map (polar FP32 pair), 4 for
// an FP16 map (its words).
int fold_esize(int dtype) { return dtype == STT_P16 ? 4 : 8; }
int64_t fold_ld(int F, int esize = 8)
{
    const int64_t per = kDmaBytes / esize;  // pixels per 1 KB piece
    return ((int64_t)F + per - 1) / per * per;
}
int dma_slab_cols(int lds_bytes, int64_t ldc, int esize = 8)
{
    return (int)std::min<int64_t>(64, (lds_bytes - 256) / (2 * ldc * esize));
}

stt_status check_map(stt_ctx *c, const stt_map *m)
{
    if (!m) return fail(c, STT_EINVAL, "map is NULL");
    if (m->dtype != STT_C64F32 && m->dtype != STT_P16)
        return fail(c, STT_EINVAL, "map dtype %d unknown", m->dtype);
    if (m->dtype == STT_P16 && m->sigma) return fail(c, STT_EINVAL, "an FP16 map has no sigma array (pass NULL)");
    if (m->dtype == STT_P16 && (m->scale_exp < -126 || m->scale_exp > 127))
        return fail(c, STT_ERANGE, "scale_exp=%d outside [-126, 127]", m->scale_exp);
    if (m->T < 2 || m->T > STT_MAX_T) return fail(c, STT_ERANGE, "T=%d outside [2, %d]", m->T, STT_MAX_T);
    if (m->F < 1 || m->F > STT_MAX_F) return fail(c, STT_ERANGE, "F=%d outside [1, %d]", m->F, STT_MAX_F);
    if (m->ld < m->F) return fail(c, STT_EINVAL, "ld=%lld < F=%d", (long long)m->ld, m->F);
    if (!m->Y || (m->dtype == STT_C64F32 && !m->sigma)) return fail(c, STT_EINVAL, "map Y or sigma is NULL");
    const int64_t fmax = std::llabs((int64_t)m->fq4_lo) + (int64_t)(m->F - 1) * std::llabs((int64_t)m->dfq4);
    if (fmax >= ((int64_t)1 << 31)) return fail(c, STT_ERANGE, "row frequencies overflow 32 bits");
    return STT_OK;
}

stt_status make_genp(stt_ctx *c, const stt_gen *g, int32_t T, int32_t F, GenP &p)
{
    if (!g) return fail(c, STT_EINVAL, "gen is NULL");
    if (T < 2 || T > STT_MAX_T) return fail(c, STT_ERANGE, "T=%d outside [2, %d]", T, STT_MAX_T);
    if (F < 1 || F > STT_MAX_F) return fail(c, STT_ERANGE, "F=%d outside [1, %d]", F, STT_MAX_F);
    if (g->min_len < 2 || g->min_len > T) return fail(c, STT_ERANGE, "min_len=%d outside [2, T=%d]", g->min_len, T);
    if (g->dtau_max < 0 || g->dtau_max >= (1 << 30)) return fail(c, STT_ERANGE, "dtau_max=%d outside [0, 2^30)", g->dtau_max);
    if (std::llabs((int64_t)g->dtau_center) + g->dtau_max >= ((int64_t)1 << 30))
        return fail(c, STT_ERANGE, "delay patch [%d - %d, %d + %d] leaves (-2^30, 2^30)", g->dtau_center, g->dtau_max,
                    g->dtau_center, g->dtau_max);
    const int64_t npos = (int64_t)T - g->min_len + 1;
    p.key0 = (uint32_t)g->seed;
    p.key1 = (uint32_t)(g->seed >> 32);
    p.stream = g->stream;
    p.npairs = (uint32_t)(npos * (npos + 1) / 2);
    p.L = g->min_len;
    p.frange = (uint32_t)F << 8;
    p.dmax = g->dtau_max - g->dtau_center;  // the draw subtracts this: delays on [center - D, center + D]
    p.dspan = 2u * (uint32_t)g->dtau_max + 1u;
    return STT_OK;
}

stt_status check_range(stt_ctx *c, int64_t first, int64_t n)
{
    if (first < 0 || n < 0) return fail(c, STT_EINVAL, "first=%lld, n=%lld must be >= 0", (long long)first, (long long)n);
    if (first + n > ((int64_t)1 << 32)) return fail(c, STT_ERANGE, "track indices must stay below 2^32");
    return STT_OK;
}

MapP to_mapp(const stt_map *m)
{
    MapP p;
    p.Y = (const float2 *)m->Y;
    p.sig = (const float *)m->sigma;
    p.T = m->T;
    p.F = m->F;
    p.ld = m->ld;
    p.fq4_lo = m->fq4_lo;
    p.dfq4 = m->dfq4;
    p.scale = m->dtype == STT_P16 ? std::ldexp(1.0f, m->scale_exp) : 1.0f;
    return p;
}

// Reserve six events for this call (growing the pool when needed).
stt_status ev_begin(stt_ctx *c)
{
    for (bool &u : c->used) u = false;
    c->kev_start = c->kev_stop = nullptr;
    if (!c->timing) return STT_OK;
    while (c->pool.size() < c->next + 6) {
        hipEvent_t e;
        STT_HIP(c, hipEventCreate(&e));
        c->pool.push_back(e);
    }
    c->last = c->next;
    c->next += 6;
    return STT_OK;
}

void ev_record(stt_ctx *c, int i)
{
    if (c->timing) (void)hipEventRecord(c->pool[c->last + i], c->stream);
}

// Events i (start) and j (end) of this call, -1 for none, taken by the next launch_ev from its
// kernel's own dispatch. (hipEventRecord enqueues a marker, which waits for the stream to drain:
// about 6 us between two kernels.)
void ev_attach(stt_ctx *c, int i, int j)
{
    c->kev_start = c->timing && i >= 0 ? c->pool[c->last + i] : nullptr;
    c->kev_stop = c->timing && j >= 0 ? c->pool[c->last + j] : nullptr;
}

// A kernel launch on the context's stream that records the attached events, if any.
template <typename K, typename... A>
void launch_ev(stt_ctx *c, K kern, dim3 grid, dim3 block, size_t shm, A... args)
{
    hipExtLaunchKernelGGL(kern, grid, block, (uint32_t)shm, c->stream, c->kev_start, c->kev_stop, 0u, args...);
    c->kev_start = c->kev_stop = nullptr;
}

void ev_end(stt_ctx *c)
{
    if (!c->timing) return;
    Rec r;
    r.base = c->last;
    for (int i = 0; i < 3; ++i) r.used[i] = c->used[i];
    c->recs.push_back(r);
}

// Bucket width 2^wb of the time-extent sort: the narrowest that keeps at most
// 128 buckets per axis and, on average, at least one wave's worth (256) of
// templates per (start, end) bucket -- narrow buckets make a wave's templates
// start and end together, so more of its columns need no mask.
int bucket_shift(int T, int64_t n)
{
    int wb = 0;
    for (;; ++wb) {
        const int64_t nb = ((T - 1) >> wb) + 1;
        if (nb > 128) continue;
        if (nb <= 1 || n / (nb * (nb + 1) / 2) >= 256) break;
    }
    return wb;
}

template <int WG, int TPT, bool HW, int MAPT, int SC>
stt_status launch_slab_t(stt_ctx *c, const MapP &m, const GenP &g, const Trk *tr, const uint32_t *order,
                         int64_t first, int64_t n, int S, size_t shm, int32_t norm, float *snr, uint64_t *wg_keys)
{
    auto kern = k_score_slab<WG, TPT, HW, MAPT, SC>;
    if (shm > 64 * 1024)
        STT_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    const unsigned grid = (unsigned)((n + WG * TPT - 1) / (WG * TPT));
    launch_ev(c, kern, dim3(grid), dim3(WG), shm, m, g, tr, order, (uint64_t)first, n, S, norm, snr, wg_keys);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

// The (workgroup size, templates per lane) shapes compiled into the library.
static const int kShapes[][2] = {{1024, 4}, {512, 4}, {256, 4}, {1024, 2}, {512, 2}};

template <bool HW, int MAPT, int SC>
stt_status launch_slab_h(stt_ctx *c, int wg, int tpt, const MapP &m, const GenP &g, const Trk *tr,
                         const uint32_t *order, int64_t first, int64_t n, int S, size_t shm, int32_t norm, float *snr,
                         uint64_t *wg_keys)
{
#define STT_SLAB_CASE(W, P)                                                                                     \
    if (wg == W && tpt == P)                                                                                    \
        return launch_slab_t<W, P, HW, MAPT, SC>(c, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    STT_SLAB_CASE(1024, 4)
    STT_SLAB_CASE(512, 4)
    STT_SLAB_CASE(256, 4)
    STT_SLAB_CASE(1024, 2)
    STT_SLAB_CASE(512, 2)
#undef STT_SLAB_CASE
    return fail(c, STT_EUNSUPPORTED, "no slab scorer compiled for workgroup %d x %d templates", wg, tpt);
}

template <int MAPT, int SC>
stt_status launch_slab_sc(stt_ctx *c, int wg, int tpt, const MapP &m, const GenP &g, const Trk *tr,
                          const uint32_t *order, int64_t first, int64_t n, int S, size_t shm, int32_t norm, float *snr,
                          uint64_t *wg_keys)
{
    if (c->hw_trig)
        return launch_slab_h<true, MAPT, SC>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    return launch_slab_h<false, MAPT, SC>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
}

// The widest aligned slab (a power of two dividing the 16-column flush grid) not wider than
// `cols`, the columns two buffers fit; 0 below 2 (then the slabs stage through registers).
int aligned_slab(int cols)
{
    int sc = 16;
    while (sc > cols) sc >>= 1;
    return sc >= 2 ? sc : 0;
}

// Shape of a slab scorer launch: lanes per workgroup, templates per lane, LDS budget.
struct SlabShape {
    int wg, tpt, lds;
};

// The shape of a call of n templates (all maps of a batch together) on folded columns of col_bytes,
// for callers that set none. Two templates per lane run 8 waves per SIMD; what is left is how many
// templates share a staged slab (fewer stagings) against how many workgroups there are to share the
// chip. Measured (us, per call):
//  - up to 400 000 templates there are not enough workgroups for every CU: the smallest, 512 x 2, with
//    the widest slabs (1000 x 1000, 10^5: 199; 512 x 2 of 80 KB 208, 1024 x 2 221, 1024 x 4 368);
//  - columns of 12 KB and more: two budgets of 80 KB hold 2-column slabs only, so one workgroup per
//    CU, of 1024 x 2 while there are few (2000 x 2000, 3 x 10^5: 519, 1024 x 4 746), then 1024 x 4
//    (10^7: 3021, 1024 x 2 3431, 512 x 4 3322);
//  - columns of 4 KB and more: 1024 x 2, one per CU up to 1.5 x 10^6 (10^6 on 1000 x 1000: 259; two
//    per CU 307), then two (10^7: 1311; one per CU 1501; 512 x 4 1327, 1024 x 4 1435; 64 maps x 10^6:
//    11.9 ms, 1024 x 4 12.1, 512 x 4 12.2);
//  - narrower columns: 512 x 2 in two per CU, then four (500 x 151, 10^6: 142, four 144; 2 x 10^7:
//    1336, two 1489, 1024 x 2 1389, 512 x 4 1379).
// With polynomial cosines the same shapes are the fastest, to 0.3 % in 15 sizes (1000 x 1000, 10^5 272, 1024 x
// 4 587; 10^7 2112, 1024 x 4 2232; 500 x 151, 2 x 10^7 2198, 512 x 4 2297; 2000 x 2000, 10^7 4736).
SlabShape slab_shape_for(int64_t n, int64_t col_bytes)
{
    constexpr int k160 = 160 * 1024, k80 = 80 * 1024, k40 = 40 * 1024;
    if (n < 400000) return {512, 2, k160};
    if (col_bytes >= 12 * 1024) return n < 600000 ? SlabShape{1024, 2, k160} : SlabShape{1024, 4, k160};
    if (col_bytes >= 4 * 1024) return {1024, 2, n < 1500000 ? k160 : k80};
    return {512, 2, n < 2000000 ? k80 : k40};
}

// sc > 0: LDS-DMA slabs of sc aligned columns (sc in 2, 4, 8, 16); sc = 0: register staging of
// S columns. Templates are drawn (tr == NULL) or given.
template <int MAPT>
stt_status launch_slab(stt_ctx *c, int sc, int wg, int tpt, const MapP &m, const GenP &g, const Trk *tr,
                       const uint32_t *order, int64_t first, int64_t n, int S, size_t shm, int32_t norm, float *snr,
                       uint64_t *wg_keys)
{
    switch (sc) {
    case 0: return launch_slab_sc<MAPT, 0>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    case 2: return launch_slab_sc<MAPT, 2>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    case 4: return launch_slab_sc<MAPT, 4>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    case 8: return launch_slab_sc<MAPT, 8>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    case 16: return launch_slab_sc<MAPT, 16>(c, wg, tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    default: return fail(c, STT_EUNSUPPORTED, "no slab scorer for %d-column slabs", sc);
    }
}

// Workgroups of a wave-per-template launch (four templates at a time each, striding over the rest):
// 16 waves per CU, and at most 1024 atomics on the best key, one per workgroup.
unsigned wave_grid(int64_t n) { return (unsigned)std::min<int64_t>((n + 3) / 4, 1024); }

// Mean template length: of generated templates by their least length, of given ones as for a small least one.
double mean_length(bool given, const GenP &g, int T) { return given ? T / 3.0 : g.L + (T - g.L) / 3.0; }

// Whether lanes that walk a template each gather one pixel at a time. 16 in flight pay while few lanes are
// active at a time; where more than some 40 000 are (templates, by their mean share of the columns), on a
// map beyond an L2, their lines push each other out of the caches. Measured (us, 16 and one): 70 000
// templates on 1000 x 1000 274, 347 of at least 10 columns, 413, 328 of 500; 3 x 10^5 624, 569 and 1021,
// 803; on 600 x 6000 821, 675 and, of at least 300 columns, 1376, 764. Delay grid, 3 x 10^5 on 600 x 6000:
// 840, 756 and 1301, 862. Maps within an L2 (10^6 on 300 x 100: 297, 324) keep 16.
bool lane_gathers_one(int64_t map_bytes, int T, int64_t n, double mean)
{
    return map_bytes > kL2Bytes && (double)n * mean > 40000.0 * T;
}

template <bool EXPL, bool HW, int MAPT>
void launch_direct(stt_ctx *c, bool per_wave, const MapP &m, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                   int32_t norm, float *snr, uint64_t *best)
{
    if (per_wave) {
        hipLaunchKernelGGL((k_score_wave<EXPL, HW, MAPT>), dim3(wave_grid(n)), dim3(256), 0, c->stream, m, g, tr,
                           (uint64_t)first, n, norm, snr, best);
        return;
    }
    const unsigned grid = (unsigned)((n + kWG - 1) / kWG);
    const bool one = lane_gathers_one(m.T * m.ld * (int64_t)sizeof(pol_t<MAPT>), m.T, n, mean_length(EXPL, g, m.T));
    auto kern = one ? k_score_direct<EXPL, HW, MAPT, 1> : k_score_direct<EXPL, HW, MAPT, kFlush>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWG), 0, c->stream, m, g, tr, (uint64_t)first, n, norm, snr, best);
}

// The direct scorers of one call on map m (format MAPT: kMapPol, kMapF32 or kMapP16), timed as the
// scoring stage.
template <bool EXPL, int MAPT>
stt_status score_direct(stt_ctx *c, bool per_wave, const MapP &m, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                        int32_t norm, float *snr, uint64_t *best)
{
    ev_record(c, 0);
    if (c->hw_trig)
        launch_direct<EXPL, true, MAPT>(c, per_wave, m, g, tr, first, n, norm, snr, best);
    else
        launch_direct<EXPL, false, MAPT>(c, per_wave, m, g, tr, first, n, norm, snr, best);
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    ev_record(c, 5);
    c->used[0] = true;
    return STT_OK;
}

// Work memory handed to a scoring call instead of the context's own (which grows
// on demand): the binning scratch and the folded map, both big enough for the
// call (checked by the caller).
struct FixedBufs {
    void *scratch;  // bucket tables, binned order, per-workgroup keys
    void *pbuf;     // folded map
};

// The map folded for the scorers into the context's folded-map buffer, or into fb's: an FP32 map
// as p in polar form (k_fold_polar, kMapPol), an FP16 map as its words in padded columns
// (k_fold_words, kMapPolH). Every scorer of Eq. 8 reads this copy; mf is its view (column stride
// fold_ld(F, element size)).
stt_status fold_polar(stt_ctx *c, const stt_map *map, const FixedBufs *fb, MapP &mf);
size_t folded_bytes(const stt_map *map);

// Scratch of a scoring call of n templates: bucket totals and cursors, the
// group starts and second-scatter chunk table, the binned order (padded to an
// even count; the count pass keeps each template's bucket there until the
// last scatter), one best-key slot per scorer workgroup (each takes at least
// 1024 templates, whatever the shape), the group regions of the first scatter
// (4 B index per template), the counts per group and sort chunk, then the
// bucket within the group of each entry of the group regions (1 B).
constexpr size_t score_scratch_bytes(int64_t n)
{
    const size_t n_order = ((size_t)n + 1) & ~(size_t)1;
    const size_t n_chunks = ((size_t)n + kBinChunk - 1) / kBinChunk;
    return sizeof(uint32_t) * (2 * (size_t)kMaxBins + 2 * (size_t)kGroupSlots + 2 * n_order + kMaxGroups * n_chunks) +
           n_order + sizeof(uint64_t) * (size_t)((n + 1023) / 1024);
}

}  // namespace

// ---------------------------------------------------------------- fixed scratch of stt_score_noalloc
// One static device array per GPU, for callers that cannot allocate: the
// folded map in its first kNaMapBytes, then the binning scratch of up to
// kNaMaxTracks templates. In host code `scratch` only names the symbol; its
// device address comes from hipGetSymbolAddress, taken once per device (with
// that device current) by stt_create and kept in g_na_ptr.
constexpr size_t kNaMapBytes = (size_t)32 << 20;
constexpr int64_t kNaMaxTracks = (int64_t)1 << 22;
constexpr size_t kNaScratchBytes = score_scratch_bytes(kNaMaxTracks);
constexpr size_t kNaBytes = kNaMapBytes + kNaScratchBytes;
static __device__ __align__(256) unsigned char scratch[kNaBytes];

namespace {

constexpr int kNaMaxDevices = 64;
void *g_na_ptr[kNaMaxDevices] = {};
std::mutex g_na_mu;

// Device address of this device's copy of `scratch` (device current); false when it is unavailable.
bool na_init(int device)
{
    if (device < 0 || device >= kNaMaxDevices) return false;
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (g_na_ptr[device]) return true;
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
        (void)hipGetLastError();
        return false;
    }
    g_na_ptr[device] = p;
    return true;
}

void *na_ptr(int device)
{
    if (device < 0 || device >= kNaMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_na_mu);
    return g_na_ptr[device];
}

bool slab_shape_ok(int wg, int tpt)
{
    for (const auto &s : kShapes)
        if (s[0] == wg && s[1] == tpt) return true;
    return false;
}

// Extents per class of the sort's order for nb buckets per axis. Slabs staged through registers and at most
// one workgroup per CU: by extent alone, a class each. Such a call lasts as long as its longest workgroup,
// and staging does not wait for an L2 that workgroups share (us for 3 x 10^5 and 10^6 templates on 600 x
// 6000: 869 and 868, in four classes 910 and 924; for 3 x 10^6, several workgroups per CU, 1945 and 1584).
uint32_t sort_class(bool dma, int64_t workgroups, int n_cu, int nb)
{
    return !dma && workgroups <= n_cu ? 1u : bucket_class((uint32_t)nb);
}

// Counting sort of templates first .. first+n-1 by time-extent bucket into the
// context's scratch (timed as the binning stage): returns the binned order and
// the per-workgroup key slots that follow it. per_wg: templates per workgroup of
// a scorer that stages through registers, 0 with DMA staging.
template <bool EXPL>
stt_status bin_templates(stt_ctx *c, const MapP &m, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                         const FixedBufs *fb, uint32_t *&order, uint64_t *&wg_keys, int per_wg = 0)
{
    const int wb = bucket_shift(m.T, n);
    const int nb = ((m.T - 1) >> wb) + 1;
    if (per_wg && !c->n_cu) STT_HIP(c, hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, c->device));
    const uint32_t cw = sort_class(!per_wg, per_wg ? (n + per_wg - 1) / per_wg : 0, c->n_cu, nb);
    const int nbins = nb * (nb + 1) / 2;
    const size_t n_order = ((size_t)n + 1) & ~(size_t)1;  // keeps the key slots 8-byte aligned
    if (!fb) {
        stt_status s = ensure_scratch(c, score_scratch_bytes(n));
        if (s != STT_OK) return s;
    }
    const int ngroups = (nbins + (1 << kGroupShift) - 1) >> kGroupShift;
    uint32_t *totals = (uint32_t *)(fb ? fb->scratch : c->scratch);
    uint32_t *cursor = totals + kMaxBins;
    const unsigned bgrid = (unsigned)((n + kBinChunk - 1) / kBinChunk);
    uint32_t *gstart = cursor + kMaxBins;
    uint32_t *fitem = gstart + kGroupSlots;
    order = fitem + kGroupSlots;
    wg_keys = (uint64_t *)(order + n_order);
    uint32_t *tmp = (uint32_t *)(wg_keys + (n + 1023) / 1024);
    uint32_t *ccnt = tmp + n_order;  // [group][chunk], ngroups rows of bgrid
    uint8_t *tsub = (uint8_t *)(ccnt + (size_t)kMaxGroups * bgrid);
    uint16_t *bins = (uint16_t *)order;
    ev_attach(c, 2, -1);
    launch_ev(c, k_fill_u32, dim3((nbins + 255) / 256), dim3(256), 0, totals, (int64_t)nbins, 0u);
    hipLaunchKernelGGL(k_bin_count<EXPL>, dim3(bgrid), dim3(256), 0, c->stream, m, g, tr, (uint64_t)first, n, wb, cw,
                       nbins, totals, bins, ccnt);
    hipLaunchKernelGGL(k_bin_scan, dim3(1 + (unsigned)ngroups), dim3(256), 0, c->stream, (const uint32_t *)totals, nbins,
                       cursor, gstart, fitem, ccnt, (int)bgrid);
    hipLaunchKernelGGL(k_bin_group, dim3(bgrid), dim3(kScatterWG), 0, c->stream, n, ngroups, (const uint16_t *)bins,
                       (const uint32_t *)gstart, (const uint32_t *)ccnt, tmp, tsub);
    // a group of c templates has ceil(c / kFineChunk) chunks: at most ceil(n / kFineChunk) + ngroups in all
    ev_attach(c, -1, 3);
    launch_ev(c, k_bin_fine, dim3((unsigned)((n + kFineChunk - 1) / kFineChunk) + (unsigned)ngroups), dim3(kScatterWG), 0,
              nbins, (const uint32_t *)gstart, (const uint32_t *)fitem, cursor, (const uint32_t *)tmp,
              (const uint8_t *)tsub, order);
    STT_HIP(c, hipGetLastError());
    c->used[1] = true;
    return STT_OK;
}

// The shape of this call: the context's, or by size while no shape is set, the budget is the default and
// the slabs stream in by DMA (registers stage into one buffer of the whole budget).
SlabShape call_shape(const stt_ctx *c, int64_t n, int64_t col_bytes)
{
    const SlabShape own{c->slab_wg, c->slab_tpt, c->lds_bytes};
    if (c->shape_set || c->lds_bytes != kLdsBytes || !c->dma) return own;
    const SlabShape sh = slab_shape_for(n, col_bytes);
    return aligned_slab(dma_slab_cols(sh.lds, col_bytes, 1)) >= 2 ? sh : own;
}

// The slab scorer of one call on the folded map m (format MAPT: kMapPol or kMapPolH).
template <bool EXPL, int MAPT>
stt_status score_slabs(stt_ctx *c, const MapP &m, const GenP &g, const Trk *tr, int64_t first, int64_t n, int32_t norm,
                       float *snr, uint64_t *best, const FixedBufs *fb)
{
    constexpr int esize = (int)sizeof(elem_t<MAPT>);
    stt_status s;
    const SlabShape sh = call_shape(c, n, m.ld * esize);
    const int64_t ldc = m.ld;
    const int sc = c->dma ? aligned_slab(dma_slab_cols(sh.lds, ldc, esize)) : 0;
    uint32_t *order = nullptr;
    uint64_t *wg_keys = nullptr;
    if ((s = bin_templates<EXPL>(c, m, g, tr, first, n, fb, order, wg_keys, sc > 0 ? 0 : sh.wg * sh.tpt)) != STT_OK) return s;
    if (sc > 0) {
        // aligned slabs of the folded map streamed into LDS with double-buffered DMA
        const size_t shm = 2 * (size_t)esize * (size_t)sc * ldc;
        ev_attach(c, 0, 1);
        s = launch_slab<MAPT>(c, sc, sh.wg, sh.tpt, m, g, tr, order, first, n, sc, shm, norm, snr, wg_keys);
    } else {
        // one slab buffer, staged through registers (maps too wide for two DMA slabs)
        const int S = std::min<int>(std::min<int>(64, (sh.lds - 256) / (esize * m.F)), m.T);
        const size_t shm = (size_t)esize * (size_t)S * m.F;
        ev_attach(c, 0, 1);
        s = launch_slab<MAPT>(c, 0, sh.wg, sh.tpt, m, g, tr, order, first, n, S, shm, norm, snr, wg_keys);
    }
    if (s != STT_OK) return s;
    c->used[0] = true;
    if (best) {
        const int64_t n_wg = (n + (int64_t)sh.wg * sh.tpt - 1) / ((int64_t)sh.wg * sh.tpt);
        ev_attach(c, -1, 5);
        launch_ev(c, k_reduce_keys, dim3(1), dim3(1024), 0, (const uint64_t *)wg_keys, n_wg, best);
        STT_HIP(c, hipGetLastError());
    } else {
        ev_record(c, 5);
    }
    return STT_OK;
}

// Wave-per-template calls that score fewer pixels than a large map holds gather from the caller's
// FP32 map and form the polar elements as they go; others fold the map first (10 us for 1000 x 1000;
// 4 us, a launch, for small ones). Measured, folded and not (us): below some 250 000 pixels folding
// is better at any n (9.1 and 18.5 for 128 templates on 100 x 128, 9.5 and 11.5 for 450 on
// 300 x 300); above, gathering is up to n T = 1.2e6 (20.7 and 16.2 for 1000 on 1000 x 1000, 13.2 and
// 11.2 for 600 on 300 x 1000; with templates of all T columns 24.9 and 20.8 at 1000, 26.6 and 28.8 at
// 1500). Fewer than 512 templates of fewer than 500 columns leave the chip to the few lanes that form the
// elements (100 templates: 13.7 and 17.2 on 300 x 1000, 14.3 and 19.2 on 200 x 4000, 13.8 and 13.9 on 500 x
// 800; 512 on 300 x 1000: 13.8 and 12.9) unless the fold is the longer part (400 x 30000: 51 and 15). A second
// launch of the delay grid would form them again (16 delays: 24 and 27 for 100 templates on 1000 x 1000, 26
// and 43 on 300 x 1000, 28 and 27 on 1000 x 2000). Past 64 flush groups a lane's second group waits for its first's polar forms: folding is
// better (500 templates on 2000 x 500: 24.1 and 27.5). One lane per template always folds: its polar
// forms would follow one another (326 us folded, 629 us not, for 1000 templates on 1000 x 1000). FP16
// maps are gathered as they are by every direct scorer: their words are the polar elements.
bool gather_unfolded(const stt_map *map, bool per_wave, int64_t n, int launches = 1)
{
    if (map->dtype == STT_P16) return true;
    const int64_t px = (int64_t)map->T * map->F;
    if (!per_wave || map->T > 64 * kFlush || n * map->T > 1200000 || px < 250000) return false;
    return px >= 4000000 * (int64_t)(launches - 1) && (map->T >= 500 || n >= 512 || px >= 1200000);
}

// Which scorer takes a call of n templates on T columns. The slab scorer sweeps the columns one slab
// after the other, so a small call costs it a floor that grows with T (58, 98, 203, 490 us at T = 100,
// 500, 1000, 2000 with F = 128, 151, 1000, 2000); the direct scorers' cost grows with the pixels.
// They cross near n T = 6e7 pixels' worth: at T = 300, 63 and 80 us for 10^5 templates, 140 and 79 for
// 3 x 10^5; at T = 1000, 100 and 203 us for 4 x 10^4, 223 and 203 for 10^5. Below that, one wave per
// template costs 1.1 + T/900 ns each, one lane per template at least the longest template's walk
// (0.11-0.16 us per column), which cross near n = 80000 T / (T + 600).
bool prefer_slabs(int T, int64_t n) { return n >= 4096 && n * (int64_t)T >= 60000000; }
bool prefer_wave(int T, int64_t n) { return n * (int64_t)(T + 600) < 80000 * (int64_t)T; }

// The same for the delay grid, per launch of 8 delays. A slab call costs at least 72, 162, 220, 432,
// 728 us at T = 100, 300, 500, 1000, 2000 (F = 128, 1000, 500, 1000, 500); the cheaper direct scorer
// reaches that at 4 x 10^5, 2 x 10^5, 1.65 x 10^5, 1.55 x 10^5, 1.7 x 10^5 templates (at 10^5: 37, 99,
// 161, 288, 454 us). One wave per template costs 2.35 ns each, one lane per template 0.16 T us and
// 0.00185 T ns each: they cross at 7 x 10^3, 2.7 x 10^4, 5.6 x 10^4 for T = 100, 300, 500, and for
// T > 1270 one wave per template is always better (10^5 at T = 1000: 288 and 360 us).
bool prefer_slabs_md(int T, int64_t n) { return n >= 130000 + 27000000 / T; }
bool prefer_wave_md(int T, int64_t n) { return n * (47000 - 37 * (int64_t)T) < 3200000 * (int64_t)T; }

// Where those two, measured with templates of 10 columns or more on maps up to 8 MB, choose a direct scorer,
// slabs are still the cheaper ones for longer templates, larger maps and more launches: by estimated times
// (us), mean the mean template length. A sweep per launch after one sort; a wave per template by its length,
// the more the further the folded map exceeds an L2; lane by lane by waves per SIMD (65 536 templates each).
// Measured (direct, slabs) with 1.5 x 10^5 templates: 1000 x 1000 of at least 500 columns 570, 443 for 8
// delays, 1692, 1237 for 17; 500 x 151 for 17 633, 543; 130 000 on 1900 x 1900 of at least 237 for 32 5558,
// 3630; 260 000 on 150 x 150 for 32 301, 269. Over 1420 sizes on 50 to 2800 columns the choice costs 0.6 %
// on average over the best scorer, 1.8 % without this.
bool slabs_beat_direct_md(int T, int64_t col_bytes, bool p16, int64_t n, double mean, int launches, bool per_wave)
{
    const double nd = (double)n, la = (double)launches;
    const double per_col = 0.31 + 8e-6 * (double)col_bytes + (p16 ? 0.04 : 0.0);
    const double slab = 50.0 + la * (5.0 + std::max(per_col * T, 2.2e-6 * nd * mean));
    if (per_wave) {
        const double mb = 1e-6 * (double)T * (double)col_bytes;
        const double per_px = std::clamp((mb - 2.0) * 0.55e-6, 0.3e-6, 10.5e-6);
        return slab < 0.95 * la * (10.0 + nd * (2e-3 + per_px * mean));
    }
    const double simd_waves = (double)((n + 65535) / 65536);
    return n > 2 * 65536 && slab < (T < 300 ? 0.9 : 1.0) * la * (6.0 + T * (0.2 + 0.105 * (simd_waves - 1.0)));
}

// And for n generated free-t_mid templates of mean length `mean` on columns of col_bytes, by estimated times
// (us): slabs take the sort and a sweep of the columns, which widen them; a wave per template takes 1.7 ns and
// 3 ps per column of its length, 0.45 more for each MB of folded map beyond 3 (13.5 at most). Measured (slabs,
// wave): 60 000 templates on 300 x 300 110, 119; 10^5 on 1000 x 1000 345, 306; on 2000 x 500 508, 572; on
// 1400 x 1400 584, 687 of at least 175 columns, 591, 1026 of 700; 125 000 on 1900 x 1900 970, 1411 of at least
// 237, on 2800 x 2000 1453, 5138 of 2798. Over 840 sizes (50 to 2800 columns, 40 to 2000 rows, 5000 to 2.5 x
// 10^5 templates) the choice costs 0.16 % on average over the better scorer, 4 % by the templates alone.
bool prefer_slabs_tm(int T, int64_t col_bytes, int64_t n, double mean)
{
    const double nd = (double)n, col = (double)col_bytes;
    const double slab = 40.0 + 6e-5 * nd + std::max(T * (0.24 + 1.2e-5 * col), 1.2e-6 * nd * mean);
    const double per_col = std::min(3e-6 + 0.45e-6 * std::max(0.0, 1e-6 * T * col - 3.0), 13.5e-6);
    return n >= 4096 && slab < 10.0 + nd * (1.7e-3 + mean * per_col);
}

template <bool EXPL>
stt_status score_impl(stt_ctx *c, const stt_map *map, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                      int32_t norm, float *snr, uint64_t *best, const FixedBufs *fb = nullptr)
{
    const int F = map->F, esize = fold_esize(map->dtype);
    // the slab plus the kernel's few static LDS words must fit the 160 KB of a CU
    bool slab = (c->lds_bytes - 256) / (esize * F) >= 1;
    if (c->path == 1 || c->path == 3) slab = false;
    if (c->path == 0 && !prefer_slabs(map->T, n)) slab = false;
    const bool per_wave = c->path == 3 || (c->path == 0 && prefer_wave(map->T, n));
    if (c->path == 2 && !slab)
        return fail(c, STT_EUNSUPPORTED, "F=%d too wide for an LDS slab of %d bytes", F, c->lds_bytes);

    stt_status s = ev_begin(c);
    if (s != STT_OK) return s;
    const bool p16 = map->dtype == STT_P16;
    // score_slabs and score_direct record event 5 at the end of their last kernel
    if (!slab && gather_unfolded(map, per_wave, n)) {
        ev_record(c, 4);
        const MapP m = to_mapp(map);
        s = p16 ? score_direct<EXPL, kMapP16>(c, per_wave, m, g, tr, first, n, norm, snr, best)
                : score_direct<EXPL, kMapF32>(c, per_wave, m, g, tr, first, n, norm, snr, best);
    } else {
        ev_attach(c, 4, -1);  // taken by the fold's launch
        MapP m;
        if ((s = fold_polar(c, map, fb, m)) != STT_OK) return s;
        s = !slab ? score_direct<EXPL, kMapPol>(c, per_wave, m, g, tr, first, n, norm, snr, best)
            : p16 ? score_slabs<EXPL, kMapPolH>(c, m, g, tr, first, n, norm, snr, best, fb)
                  : score_slabs<EXPL, kMapPol>(c, m, g, tr, first, n, norm, snr, best, fb);
    }
    if (s != STT_OK) return s;
    c->used[2] = true;
    ev_end(c);
    return STT_OK;
}

// Bytes of the folded copy of a map.
size_t folded_bytes(const stt_map *map)
{
    const int esize = fold_esize(map->dtype);
    return (size_t)esize * (size_t)map->T * (size_t)fold_ld(map->F, esize);
}

stt_status fold_polar(stt_ctx *c, const stt_map *map, const FixedBufs *fb, MapP &mf)
{
    const MapP m = to_mapp(map);
    const int esize = fold_esize(map->dtype);
    const int64_t ldc = fold_ld(m.F, esize);
    if (!fb) {
        const stt_status s = ensure_pbuf(c, folded_bytes(map));
        if (s != STT_OK) return s;
    }
    void *pbuf = fb ? fb->pbuf : c->pbuf;
    const dim3 fg((unsigned)m.T, (unsigned)((ldc + 256 * kFoldRows - 1) / (256 * kFoldRows)));  // one column per x, rows over y
    if (map->dtype == STT_P16)
        launch_ev(c, k_fold_words, fg, dim3(256), 0, m, (uint32_t *)pbuf, (int64_t)ldc);
    else
        launch_ev(c, k_fold_polar<kMapF32>, fg, dim3(256), 0, m, (float2 *)pbuf, (int64_t)ldc);
    STT_HIP(c, hipGetLastError());
    mf = m;  // an FP16 map keeps its scale 2^e
    mf.Y = (const float2 *)pbuf;
    mf.sig = nullptr;
    mf.ld = ldc;
    return STT_OK;
}

// The delay grid in launches of kMD delays by the direct scorers, one wave or one lane per template,
// on map m (format MAPT: kMapPol, kMapF32 or kMapP16).
template <bool EXPL, int MAPT>
stt_status maxdelay_direct(stt_ctx *c, bool per_wave, const MapP &m, const GenP &g, const Trk *tr, int64_t first,
                           int64_t n, int32_t d0, int32_t step, int32_t n_tau, int32_t norm, float *snr, int32_t *tidx,
                           uint64_t *best)
{
    const int n_launch = (n_tau + kMD - 1) / kMD;
    const unsigned grid = per_wave ? wave_grid(n) : (unsigned)((n + kWG - 1) / kWG);
    const bool one = lane_gathers_one(m.T * m.ld * (int64_t)sizeof(pol_t<MAPT>), m.T, n, mean_length(EXPL, g, m.T));
    auto kern = per_wave ? (c->hw_trig ? k_score_md_wave<EXPL, true, MAPT> : k_score_md_wave<EXPL, false, MAPT>)
                : one ? (c->hw_trig ? k_score_md_direct<EXPL, true, MAPT, 1> : k_score_md_direct<EXPL, false, MAPT, 1>)
                      : (c->hw_trig ? k_score_md_direct<EXPL, true, MAPT, kFlush> : k_score_md_direct<EXPL, false, MAPT, kFlush>);
    ev_record(c, 0);
    for (int l = 0; l < n_launch; ++l) {
        const int32_t m0 = l * kMD, cnt = std::min(kMD, n_tau - m0), last = l == n_launch - 1;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, c->stream, m, g, tr, (uint64_t)first, n, norm, d0, step, m0,
                           cnt, last, snr, tidx, best);
    }
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    c->used[0] = true;
    return STT_OK;
}

// The delay grid in launches of kMD delays from slabs (binned templates, folded map, LDS-DMA). The
// same bits as the direct scorers.
template <bool EXPL, int MAPT>
stt_status maxdelay_slabs(stt_ctx *c, const MapP &mf, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                          int32_t d0, int32_t step, int32_t n_tau, int32_t norm, float *snr, int32_t *tidx,
                          uint64_t *best, int lds)
{
    // 1024 lanes x 1 template, at most 80 KB of slabs (measured on the search map: 512 x 2, 1024 x 2,
    // 256 x 4 and smaller slabs were 15-75 % slower; one template per lane leaves room for more waves)
    constexpr int kMdWG = 1024, kMdTPT = 1;
    constexpr int esize = (int)sizeof(elem_t<MAPT>);
    const int64_t ldc = mf.ld;
    const int n_launch = (n_tau + kMD - 1) / kMD;
    stt_status s;
    uint32_t *order = nullptr;
    uint64_t *wg_keys = nullptr;
    if ((s = bin_templates<EXPL>(c, mf, g, tr, first, n, nullptr, order, wg_keys)) != STT_OK) return s;
    const int S = std::min(dma_slab_cols(lds, ldc, esize), mf.T);
    const size_t shm = 2 * (size_t)esize * (size_t)S * ldc;
    const unsigned grid = (unsigned)((n + kMdWG * kMdTPT - 1) / (kMdWG * kMdTPT));
    auto kh = k_score_md_slab<kMdWG, kMdTPT, EXPL, true, MAPT>;
    auto kp = k_score_md_slab<kMdWG, kMdTPT, EXPL, false, MAPT>;
    auto kern = c->hw_trig ? kh : kp;
    if (shm > 64 * 1024)
        STT_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    ev_record(c, 0);
    for (int l = 0; l < n_launch; ++l) {
        const int32_t m0 = l * kMD, cnt = std::min(kMD, n_tau - m0), last = l == n_launch - 1;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kMdWG), shm, c->stream, mf, g, tr, (const uint32_t *)order,
                           (uint64_t)first, n, S, norm, d0, step, m0, cnt, last, snr, tidx, wg_keys);
    }
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    c->used[0] = true;
    if (best) {
        hipLaunchKernelGGL(k_reduce_keys, dim3(1), dim3(1024), 0, c->stream, (const uint64_t *)wg_keys, (int64_t)grid,
                           best);
        STT_HIP(c, hipGetLastError());
    }
    return STT_OK;
}

template <bool EXPL>
stt_status maxdelay_impl(stt_ctx *c, const stt_map *map, const GenP &g, const Trk *tr, int64_t first, int64_t n,
                         int32_t d0, int32_t step, int32_t n_tau, int32_t norm, float *snr, int32_t *tidx,
                         uint64_t *best)
{
    const int lds = std::min(c->lds_bytes, 80 * 1024);
    const int esize = fold_esize(map->dtype);
    const int64_t ldc = fold_ld(map->F, esize);
    const bool p16 = map->dtype == STT_P16;
    const int n_launch = (n_tau + kMD - 1) / kMD;
    const bool per_wave = c->path == 3 || (c->path == 0 && prefer_wave_md(map->T, n));
    const double mean = mean_length(EXPL, g, map->T);
    const bool slab = c->dma && dma_slab_cols(lds, ldc, esize) >= 1 && c->path != 1 && c->path != 3 &&
                      (c->path == 2 || prefer_slabs_md(map->T, n) ||
                       slabs_beat_direct_md(map->T, ldc * esize, p16, n, mean, n_launch, per_wave));
    if (c->path == 2 && !slab)
        return fail(c, STT_EUNSUPPORTED, "F=%d too wide for two LDS slabs of %d bytes", map->F, lds);
    stt_status s;
    if (!snr || !tidx) {
        if ((s = ensure_mdbuf(c, (sizeof(float) + sizeof(int32_t)) * (size_t)n)) != STT_OK) return s;
        if (!snr) snr = (float *)c->mdbuf;
        if (!tidx) tidx = (int32_t *)((float *)c->mdbuf + n);
    }
    if ((s = ev_begin(c)) != STT_OK) return s;
    ev_record(c, 4);
    if (!slab && gather_unfolded(map, per_wave, n, n_launch)) {
        const MapP m = to_mapp(map);
        s = p16 ? maxdelay_direct<EXPL, kMapP16>(c, per_wave, m, g, tr, first, n, d0, step, n_tau, norm, snr, tidx, best)
                : maxdelay_direct<EXPL, kMapF32>(c, per_wave, m, g, tr, first, n, d0, step, n_tau, norm, snr, tidx, best);
    } else {
        MapP mf;
        if ((s = fold_polar(c, map, nullptr, mf)) != STT_OK) return s;
        s = !slab ? maxdelay_direct<EXPL, kMapPol>(c, per_wave, mf, g, tr, first, n, d0, step, n_tau, norm, snr, tidx, best)
            : p16 ? maxdelay_slabs<EXPL, kMapPolH>(c, mf, g, tr, first, n, d0, step, n_tau, norm, snr, tidx, best, lds)
                  : maxdelay_slabs<EXPL, kMapPol>(c, mf, g, tr, first, n, d0, step, n_tau, norm, snr, tidx, best, lds);
    }
    if (s != STT_OK) return s;
    ev_record(c, 5);
    c->used[2] = true;
    ev_end(c);
    return STT_OK;
}

// The free-t_mid slab scorer of one call on the folded map mf (format MAPT: kMapPol or kMapPolH).
template <int MAPT>
stt_status score_tm_slabs(stt_ctx *c, const MapP &mf, const GenP &g, int64_t first, int64_t n, int32_t norm,
                          float *snr_dev, uint64_t *best_key_dev, int lds)
{
    constexpr int kTmWG = 1024, kTmTPT = 1;
    constexpr int esize = (int)sizeof(elem_t<MAPT>);
    stt_status s;
    uint32_t *order = nullptr;
    uint64_t *wg_keys = nullptr;
    if ((s = bin_templates<false>(c, mf, g, nullptr, first, n, nullptr, order, wg_keys)) != STT_OK) return s;
    const int S = std::min(dma_slab_cols(lds, mf.ld, esize), mf.T);
    const size_t shm = 2 * (size_t)esize * (size_t)S * mf.ld;
    const unsigned grid = (unsigned)((n + kTmWG * kTmTPT - 1) / (kTmWG * kTmTPT));
    auto kern = c->hw_trig ? k_score_tm_slab<kTmWG, kTmTPT, true, MAPT> : k_score_tm_slab<kTmWG, kTmTPT, false, MAPT>;
    if (shm > 64 * 1024)
        STT_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    ev_record(c, 0);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kTmWG), shm, c->stream, mf, g, (const uint32_t *)order,
                       (uint64_t)first, n, S, norm, snr_dev, wg_keys);
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    c->used[0] = true;
    if (best_key_dev) {
        hipLaunchKernelGGL(k_reduce_keys, dim3(1), dim3(1024), 0, c->stream, (const uint64_t *)wg_keys,
                           (int64_t)grid, best_key_dev);
        STT_HIP(c, hipGetLastError());
    }
    return STT_OK;
}

// The free-t_mid wave scorer on map m (format MAPT: kMapPol, kMapF32 or kMapP16).
template <int MAPT>
stt_status score_tm_wave(stt_ctx *c, const MapP &m, const GenP &g, const TrkTm *tr, int64_t first, int64_t n, int32_t norm,
                         float *snr_dev, uint64_t *best_key_dev)
{
    auto kern = tr ? (c->hw_trig ? k_score_tm<true, true, MAPT> : k_score_tm<true, false, MAPT>)
                   : (c->hw_trig ? k_score_tm<false, true, MAPT> : k_score_tm<false, false, MAPT>);
    ev_record(c, 0);
    hipLaunchKernelGGL(kern, dim3(wave_grid(n)), dim3(256), 0, c->stream, m, g, tr, (uint64_t)first, n, norm, snr_dev,
                       best_key_dev);
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    c->used[0] = true;
    return STT_OK;
}

// Twiddles e^{-2 pi i j / M} (j < M/2) then the periodic Hann window sin^2(pi n / M) (n < M),
// evaluated in FP64 and rounded once; rewritten (after the stream drains) when M changes.
stt_status ensure_fft_tab(stt_ctx *c, int M)
{
    if (c->fft_tab && c->fft_M == M) return STT_OK;
    const int N = M / 2;
    std::vector<float> h((size_t)2 * N + M);
    for (int j = 0; j < N; ++j) {
        const double a = 2.0 * M_PI * (double)j / (double)M;
        h[2 * j] = (float)std::cos(a);
        h[2 * j + 1] = (float)-std::sin(a);
    }
    for (int n = 0; n < M; ++n) {
        const double v = std::sin(M_PI * (double)n / (double)M);
        h[(size_t)2 * N + n] = (float)(v * v);
    }
    if (!c->fft_tab) {
        const size_t most = sizeof(float) * (size_t)2 * kMaxFftM;  // room for the largest M
        if (hipMalloc(&c->fft_tab, most) != hipSuccess) {
            (void)hipGetLastError();
            c->fft_tab = nullptr;
            return fail(c, STT_ENOMEM, "cannot allocate the FFT table");
        }
    }
    STT_HIP(c, hipStreamSynchronize(c->stream));  // earlier transforms may still read the old table
    STT_HIP(c, hipMemcpy(c->fft_tab, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice));
    c->fft_M = M;
    return STT_OK;
}

stt_status check_spectro(stt_ctx *c, const stt_spectro *p)
{
    if (!p) return fail(c, STT_EINVAL, "null spectrogram parameters");
    if (!(p->fs > 0) || !std::isfinite(p->fs)) return fail(c, STT_EINVAL, "fs must be positive");
    if (p->M < 8 || p->M > kMaxFftM || (p->M & (p->M - 1)))
        return fail(c, STT_ERANGE, "M=%d: need a power of two in [8, %d]", p->M, kMaxFftM);
    if (p->k_lo < 0 || p->F < 1 || (int64_t)p->k_lo + p->F > p->M / 2)
        return fail(c, STT_ERANGE, "bins [%d, %d) outside [0, M/2)", p->k_lo, p->k_lo + p->F);
    if (p->nb < 1) return fail(c, STT_EINVAL, "nb=%d: need >= 1", p->nb);
    return STT_OK;
}

// 2 / Nrm with Nrm = M dt 3/8 (the Hann window's mean square)
float cross_scale(const stt_spectro *p) { return (float)(2.0 / ((double)p->M / p->fs * 0.375)); }

// The K best of src's n elements (stt_topk's launches), or with last_only the K-th best score alone.
template <typename SRC>
stt_status topk_launch(stt_ctx *c, SRC src, int64_t n, int64_t first, int32_t K, int last_only, int64_t *idx_dev,
                       float *val_dev)
{
    const stt_status s = ensure_aux(c, kTopkBytes);
    if (s != STT_OK) return s;
    TopkState *st = (TopkState *)c->aux;
    uint64_t *cand = (uint64_t *)((char *)c->aux + kTopkStateBytes);
    // 8 elements per lane where that still fills the chip; each workgroup flushes a histogram
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 2047) / 2048, 1024));
    hipLaunchKernelGGL(k_topk_init, dim3(kTopkPasses * kTopkBins / 1024), dim3(1024), 0, c->stream, st, (uint32_t)K);
    for (int pass = 0; pass < kTopkPasses; ++pass)
        hipLaunchKernelGGL(k_topk_hist<SRC>, dim3(grid), dim3(256), 0, c->stream, src, n, (uint64_t)first, st, pass);
    hipLaunchKernelGGL(k_topk_gather<SRC>, dim3(grid), dim3(256), 0, c->stream, src, n, (uint64_t)first, st, cand);
    const unsigned rgrid = (unsigned)((std::min<int64_t>(n, kTopkCand) + 63) / 64);
    hipLaunchKernelGGL(k_topk_rank, dim3(rgrid), dim3(1024), 0, c->stream, (const TopkState *)st, (const uint64_t *)cand, K,
                       last_only, idx_dev, val_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

// Whether the context's stream captures a graph, or cannot say (the null stream while another captures).
bool capturing(stt_ctx *c)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cs) == hipSuccess) return cs != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// Whether counts go by ranks. Directly they take 17 ns per reference, from 180 000 queries on more (25 ns
// for 3 x 10^5, 60 for 10^6); by ranks, a pass takes 12 us and, for the sort of its tiles, 11 ns per place
// of a tile (a power of two), and hardly depends on the references up to 10^4. Measured (us, direct and
// ranks): 513 references 10 and 12 for one query, 11 and 56 for 10^5; 1000 references 18 and 13 for one
// query, 19 and 25 for 1000, 19 and 55 for 4096; 2000 references 36 and 25 for 1000, 36 and 34 for 2048;
// 3000 references 53 and 58 for 4096; 5000 references 87 and 64 for 4096, 129 and 133 for 3 x 10^5.
bool prefer_ranks(int64_t n_ref, int64_t n_q)
{
    const int64_t per_pass = (int64_t)kRankTile * kRankTiles;
    const auto pass_ns = [](int64_t queries) {
        int P = 64;
        while (P < queries && P < kRankTile) P <<= 1;
        return 11500.0 + 11.0 * P;
    };
    const int64_t full = n_q / per_pass, rest = n_q - full * per_pass;
    return (double)n_ref * std::max(17.0, 8.0 + (double)n_q / 20000) >
           (double)full * pass_ns(per_pass) + (rest ? pass_ns(rest) : 0.0);
}

// Counts (and FAP = count / n_ref) of n_q query keys against n_ref reference keys: directly, or by ranks
// in passes of kRankTiles tiles of queries where those are faster. The ranks need
// scratch. A call that finds no memory for it counts directly too, and so does one on a capturing stream: its
// graph would keep the scratch's address, and the scratch moves when a later call needs more of it.
stt_status count_louder(stt_ctx *c, const uint64_t *ref, int64_t n_ref, const uint64_t *q, int64_t n_q, int64_t *count,
                        float *fap)
{
    const int64_t per_pass = (int64_t)kRankTile * kRankTiles;
    const size_t need = sizeof(RankTile) * (size_t)std::min<int64_t>(kRankTiles, (n_q + kRankTile - 1) / kRankTile);
    bool ranks = prefer_ranks(n_ref, n_q) && !capturing(c);
    if (ranks) {
        const std::string before = c->err;
        const stt_status s = ensure_mdbuf(c, need);
        if (s != STT_OK && s != STT_ENOMEM) return s;
        if (s == STT_ENOMEM) {
            ranks = false;
            c->err = before;
        }
    }
    if (!ranks) {
        hipLaunchKernelGGL(k_count_louder, dim3((unsigned)((n_q + 255) / 256)), dim3(256), 0, c->stream, ref, n_ref, q, n_q,
                           count, fap, (double)n_ref);
        STT_HIP(c, hipGetLastError());
        return STT_OK;
    }
    RankTile *tiles = (RankTile *)c->mdbuf;
    for (int64_t q0 = 0; q0 < n_q; q0 += per_pass) {
        const int64_t m = std::min(per_pass, n_q - q0);
        const unsigned nt = (unsigned)((m + kRankTile - 1) / kRankTile);
        // 8 references per lane, at most four workgroups per CU over all tiles
        const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n_ref + 8191) / 8192, 1024 / nt));
        hipLaunchKernelGGL(k_rank_sort, dim3(nt), dim3(1024), 0, c->stream, q + q0, m, tiles);
        hipLaunchKernelGGL(k_rank_count, dim3(nb, nt), dim3(1024), 0, c->stream, ref, n_ref, m, tiles);
        hipLaunchKernelGGL(k_rank_finish, dim3(nt), dim3(1024), 0, c->stream, (const RankTile *)tiles, m,
                           count ? count + q0 : nullptr, fap ? fap + q0 : nullptr, (double)n_ref);
    }
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

}  // namespace

extern "C" {

const char *stt_strerror(stt_status s)
{
    switch (s) {
    case STT_OK: return "ok";
    case STT_EINVAL: return "invalid argument";
    case STT_ERANGE: return "size out of supported range";
    case STT_ENOMEM: return "out of device memory";
    case STT_EHIP: return "HIP runtime error";
    case STT_EUNSUPPORTED: return "unsupported";
    default: return "unknown status";
    }
}

const char *stt_last_error(const stt_ctx *c) { return c ? c->err.c_str() : "no context"; }

stt_status stt_create(int device, void *hip_stream, stt_ctx **out)
{
    if (!out) return STT_EINVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return STT_EHIP;
    if (hipSetDevice(device) != hipSuccess) return STT_EHIP;
    stt_ctx *c = new stt_ctx;
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    // the fixed scratch of stt_score_noalloc on this device (that call fails cleanly without it)
    (void)na_init(device);
    *out = c;
    return STT_OK;
}

stt_status stt_destroy(stt_ctx *c)
{
    if (!c) return STT_EINVAL;
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->stream);
    if (c->scratch) (void)hipFree(c->scratch);
    if (c->aux) (void)hipFree(c->aux);
    if (c->pbuf) (void)hipFree(c->pbuf);
    if (c->mdbuf) (void)hipFree(c->mdbuf);
    if (c->bdev) (void)hipFree(c->bdev);
    if (c->fft_tab) (void)hipFree(c->fft_tab);
    if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
    if (c->graph) (void)hipGraphDestroy(c->graph);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    for (auto &e : c->pool) (void)hipEventDestroy(e);
    delete c;
    return STT_OK;
}

stt_status stt_set_stream(stt_ctx *c, void *hip_stream)
{
    if (!c) return STT_EINVAL;
    c->stream = (hipStream_t)hip_stream;
    return STT_OK;
}

stt_status stt_sync(stt_ctx *c)
{
    if (!c) return STT_EINVAL;
    STT_HIP(c, hipStreamSynchronize(c->stream));
    return STT_OK;
}

stt_status stt_reserve(stt_ctx *c, int64_t max_tracks)
{
    if (!c || max_tracks < 0) return fail(c, STT_EINVAL, "bad reserve request");
    return ensure_scratch(c, score_scratch_bytes(max_tracks));
}

stt_status stt_set_timing(stt_ctx *c, int32_t on)
{
    if (!c) return STT_EINVAL;
    c->timing = on != 0;
    c->recs.clear();
    c->next = c->last = 0;
    return STT_OK;
}

static const int kEvPair[3] = {0, 2, 4};  // start event of each stage within a call's six

stt_status stt_kernel_ms(stt_ctx *c, int32_t which, float *ms)
{
    if (!c || !ms || which < 0 || which > 2) return fail(c, STT_EINVAL, "bad timing query");
    if (!c->timing || c->recs.empty() || !c->recs.back().used[which])
        return fail(c, STT_EINVAL, "no timed stage %d in the last call", which);
    STT_HIP(c, hipStreamSynchronize(c->stream));
    const size_t a = c->recs.back().base + kEvPair[which];
    STT_HIP(c, hipEventElapsedTime(ms, c->pool[a], c->pool[a + 1]));
    return STT_OK;
}

stt_status stt_kernel_ms_total(stt_ctx *c, int32_t which, double *total_ms, int32_t *count)
{
    if (!c || !total_ms || !count || which < 0 || which > 2) return fail(c, STT_EINVAL, "bad timing query");
    if (!c->timing) return fail(c, STT_EINVAL, "timing is off");
    STT_HIP(c, hipStreamSynchronize(c->stream));
    double tot = 0.0;
    int32_t n = 0;
    for (const auto &r : c->recs) {
        if (!r.used[which]) continue;
        float ms = 0.0f;
        const size_t a = r.base + kEvPair[which];
        STT_HIP(c, hipEventElapsedTime(&ms, c->pool[a], c->pool[a + 1]));
        tot += ms;
        ++n;
    }
    *total_ms = tot;
    *count = n;
    c->recs.clear();
    c->next = c->last = 0;
    return STT_OK;
}

// Internal knob used by tests and tuning: 0 auto, 1 direct gathers, 2 LDS slabs.
stt_status stt_set_path(stt_ctx *c, int32_t path, int32_t lds_bytes)
{
    if (!c || path < 0 || path > 3) return STT_EINVAL;
    if (lds_bytes != 0 && (lds_bytes < 1024 || lds_bytes > 160 * 1024))
        return fail(c, STT_ERANGE, "lds_bytes=%d outside [1024, 163840]", lds_bytes);
    c->path = path;
    if (lds_bytes) c->lds_bytes = lds_bytes;
    return STT_OK;
}

stt_status stt_set_slab_shape(stt_ctx *c, int32_t wg, int32_t tpt)
{
    if (!c) return STT_EINVAL;
    if (!slab_shape_ok(wg, tpt)) return fail(c, STT_EUNSUPPORTED, "no slab scorer for %d x %d", wg, tpt);
    c->slab_wg = wg;
    c->slab_tpt = tpt;
    c->shape_set = true;
    return STT_OK;
}

stt_status stt_set_staging(stt_ctx *c, int32_t dma)
{
    if (!c || dma < 0 || dma > 1) return STT_EINVAL;
    c->dma = dma == 1;
    return STT_OK;
}

stt_status stt_set_trig(stt_ctx *c, int32_t hw)
{
    if (!c || hw < 0 || hw > 1) return STT_EINVAL;
    c->hw_trig = hw == 1;
    return STT_OK;
}

stt_status stt_make_tracks(stt_ctx *c, const stt_gen *gen, int32_t T, int32_t F, int64_t first, int64_t n,
                           stt_track *out_dev)
{
    if (!c) return STT_EINVAL;
    GenP g;
    stt_status s = make_genp(c, gen, T, F, g);
    if (s != STT_OK) return s;
    if ((s = check_range(c, first, n)) != STT_OK) return s;
    if (n == 0) return STT_OK;
    if (!out_dev) return fail(c, STT_EINVAL, "out_dev is NULL");
    STT_HIP(c, hipSetDevice(c->device));
    const unsigned grid = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_make_tracks, dim3(grid), dim3(256), 0, c->stream, g, (uint64_t)first, n, (Trk *)out_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

stt_status stt_score(stt_ctx *c, const stt_map *map, const stt_gen *gen, const stt_track *tracks_dev, int64_t first,
                     int64_t n, int32_t norm, float *snr_dev, uint64_t *best_key_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if ((s = check_range(c, first, n)) != STT_OK) return s;
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    GenP g{};
    if (!tracks_dev) {
        if ((s = make_genp(c, gen, map->T, map->F, g)) != STT_OK) return s;
    }
    if (n == 0) return STT_OK;
    STT_HIP(c, hipSetDevice(c->device));
    if (tracks_dev)
        return score_impl<true>(c, map, g, (const Trk *)tracks_dev, first, n, norm, snr_dev, best_key_dev);
    return score_impl<false>(c, map, g, nullptr, first, n, norm, snr_dev, best_key_dev);
}

stt_status stt_score_noalloc(stt_ctx *c, const stt_map *map, const stt_gen *gen, const stt_track *tracks_dev,
                             int64_t first, int64_t n, int32_t norm, float *snr_dev, uint64_t *best_key_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if ((s = check_range(c, first, n)) != STT_OK) return s;
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    if (n > kNaMaxTracks)
        return fail(c, STT_ERANGE, "n=%lld exceeds the %lld templates of the fixed scratch", (long long)n,
                    (long long)kNaMaxTracks);
    const size_t map_bytes = folded_bytes(map);
    if (map_bytes > kNaMapBytes)
        return fail(c, STT_ERANGE, "the folded %dx%d map needs %zu bytes; the fixed scratch holds %zu", map->T,
                    map->F, map_bytes, kNaMapBytes);
    GenP g{};
    if (!tracks_dev) {
        if ((s = make_genp(c, gen, map->T, map->F, g)) != STT_OK) return s;
    }
    if (n == 0) return STT_OK;
    STT_HIP(c, hipSetDevice(c->device));
    void *base = na_ptr(c->device);
    if (!base) return fail(c, STT_EHIP, "no fixed scratch on device %d (hipGetSymbolAddress failed)", c->device);
    const FixedBufs fb{(unsigned char *)base + kNaMapBytes, base};
    // no timing events either: the event pool grows by allocation
    const bool timing = c->timing;
    c->timing = false;
    if (tracks_dev)
        s = score_impl<true>(c, map, g, (const Trk *)tracks_dev, first, n, norm, snr_dev, best_key_dev, &fb);
    else
        s = score_impl<false>(c, map, g, nullptr, first, n, norm, snr_dev, best_key_dev, &fb);
    c->timing = timing;
    return s;
}

stt_status stt_score_maxdelay(stt_ctx *c, const stt_map *map, const stt_gen *gen, const stt_track *tracks_dev,
                              int64_t first, int64_t n, int32_t dtau0, int32_t dtau_step, int32_t n_tau, int32_t norm,
                              float *snr_dev, int32_t *tau_idx_dev, uint64_t *best_key_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if ((s = check_range(c, first, n)) != STT_OK) return s;
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    if (n_tau < 1 || n_tau > 65536) return fail(c, STT_ERANGE, "n_tau=%d outside [1, 65536]", n_tau);
    const int64_t dlast = (int64_t)dtau0 + (int64_t)(n_tau - 1) * dtau_step;
    const int64_t dlim = ((int64_t)1 << 30) - 1;
    if (dtau0 < -dlim || dtau0 > dlim || dlast < -dlim || dlast > dlim)
        return fail(c, STT_ERANGE, "delay grid %d + m*%d (m < %d) leaves (-2^30, 2^30)", dtau0, dtau_step, n_tau);
    GenP g{};
    if (!tracks_dev) {
        if ((s = make_genp(c, gen, map->T, map->F, g)) != STT_OK) return s;
    }
    if (n == 0) return STT_OK;
    STT_HIP(c, hipSetDevice(c->device));
    const Trk *tr = (const Trk *)tracks_dev;
    if (tracks_dev)
        return maxdelay_impl<true>(c, map, g, tr, first, n, dtau0, dtau_step, n_tau, norm, snr_dev, tau_idx_dev,
                                   best_key_dev);
    return maxdelay_impl<false>(c, map, g, nullptr, first, n, dtau0, dtau_step, n_tau, norm, snr_dev, tau_idx_dev,
                                best_key_dev);
}

stt_status stt_make_tracks_tm(stt_ctx *c, const stt_gen *gen, int32_t T, int32_t F, int64_t first, int64_t n,
                              stt_track_tm *out_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_range(c, first, n);
    if (s != STT_OK) return s;
    GenP g;
    if ((s = make_genp(c, gen, T, F, g)) != STT_OK) return s;
    if (n == 0) return STT_OK;
    if (!out_dev) return fail(c, STT_EINVAL, "out_dev is NULL");
    STT_HIP(c, hipSetDevice(c->device));
    hipLaunchKernelGGL(k_make_tracks_tm, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, g,
                       (uint64_t)first, n, (TrkTm *)out_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

stt_status stt_score_tm(stt_ctx *c, const stt_map *map, const stt_gen *gen, const stt_track_tm *tracks_dev,
                        int64_t first, int64_t n, int32_t norm, float *snr_dev, uint64_t *best_key_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if ((s = check_range(c, first, n)) != STT_OK) return s;
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    GenP g{};
    if (!tracks_dev) {
        if ((s = make_genp(c, gen, map->T, map->F, g)) != STT_OK) return s;
    }
    if (n == 0) return STT_OK;
    STT_HIP(c, hipSetDevice(c->device));
    // generated templates: binned by time extent (a free t_mid keeps it) and scored from LDS slabs
    // (1024 lanes x 1 template, at most 80 KB of slabs) when a column fits; otherwise one wave each
    const int lds = std::min(c->lds_bytes, 80 * 1024);
    const int esize = fold_esize(map->dtype);
    const int64_t ldc = fold_ld(map->F, esize);
    const bool slab = !tracks_dev && c->dma && dma_slab_cols(lds, ldc, esize) >= 1 && c->path != 1 && c->path != 3 &&
                      (c->path == 2 || prefer_slabs_tm(map->T, ldc * esize, n, mean_length(false, g, map->T)));
    if ((s = ev_begin(c)) != STT_OK) return s;
    ev_record(c, 4);
    const bool p16 = map->dtype == STT_P16;
    const TrkTm *tr = (const TrkTm *)tracks_dev;
    if (!slab && gather_unfolded(map, true, n)) {
        const MapP m = to_mapp(map);
        s = p16 ? score_tm_wave<kMapP16>(c, m, g, tr, first, n, norm, snr_dev, best_key_dev)
                : score_tm_wave<kMapF32>(c, m, g, tr, first, n, norm, snr_dev, best_key_dev);
    } else {
        MapP mf;
        if ((s = fold_polar(c, map, nullptr, mf)) != STT_OK) return s;
        s = !slab ? score_tm_wave<kMapPol>(c, mf, g, tr, first, n, norm, snr_dev, best_key_dev)
            : p16 ? score_tm_slabs<kMapPolH>(c, mf, g, first, n, norm, snr_dev, best_key_dev, lds)
                  : score_tm_slabs<kMapPol>(c, mf, g, first, n, norm, snr_dev, best_key_dev, lds);
    }
    if (s != STT_OK) return s;
    ev_record(c, 5);
    c->used[2] = true;
    ev_end(c);
    return STT_OK;
}

stt_status stt_argmax(stt_ctx *c, const float *snr_dev, int64_t n, int64_t first, uint64_t *best_key_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_range(c, first, n);
    if (s != STT_OK) return s;
    if (n == 0) return STT_OK;
    if (!snr_dev || !best_key_dev) return fail(c, STT_EINVAL, "snr_dev and best_key_dev must be non-NULL");
    STT_HIP(c, hipSetDevice(c->device));
    const int64_t blocks = std::min<int64_t>((n + 1023) / 1024, 1024);  // one atomic each
    hipLaunchKernelGGL(k_argmax, dim3((unsigned)blocks), dim3(256), 0, c->stream, snr_dev, n, (uint64_t)first,
                       best_key_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

stt_status stt_map_pack_p16(stt_ctx *c, const stt_map *map, void *out_dev, int64_t out_ld, int32_t *scale_exp)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if (map->dtype != STT_C64F32) return fail(c, STT_EINVAL, "stt_map_pack_p16 packs an FP32 (Y, sigma) map");
    if (!out_dev || !scale_exp) return fail(c, STT_EINVAL, "out_dev and scale_exp must be non-NULL");
    if (out_ld < map->F) return fail(c, STT_EINVAL, "out_ld=%lld < F=%d", (long long)out_ld, map->F);
    STT_HIP(c, hipSetDevice(c->device));
    if ((s = ensure_aux(c, sizeof(unsigned long long))) != STT_OK) return s;
    unsigned long long *amax = (unsigned long long *)c->aux;
    const MapP m = to_mapp(map);
    const int64_t n = (int64_t)map->T * map->F;
    const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, c->stream, (uint32_t *)amax, (int64_t)2, 0u);
    hipLaunchKernelGGL(k_absmax_p, dim3(std::min(grid, 1024u)), dim3(256), 0, c->stream, m, amax);
    STT_HIP(c, hipGetLastError());
    unsigned long long bits = 0;
    STT_HIP(c, hipMemcpyAsync(&bits, amax, sizeof bits, hipMemcpyDeviceToHost, c->stream));
    STT_HIP(c, hipStreamSynchronize(c->stream));
    double amaxd;
    std::memcpy(&amaxd, &bits, sizeof amaxd);
    if (!std::isfinite(amaxd)) return fail(c, STT_EINVAL, "map holds a non-finite Y/sigma");
    // e = ceil(log2(max |p|)) - 15, exactly: with max = fr 2^k, fr in [1/2, 1), the ceiling is k
    // unless fr = 1/2 (a power of two, its own ceiling k - 1)
    int e = 0;
    if (amaxd > 0.0) {
        int k = 0;
        const double fr = std::frexp(amaxd, &k);
        e = (fr > 0.5 ? k : k - 1) - 15;
    }
    hipLaunchKernelGGL(k_pack_p16, dim3(grid), dim3(256), 0, c->stream, m, std::ldexp(1.0, -e), (uint32_t *)out_dev,
                       out_ld);
    STT_HIP(c, hipGetLastError());
    *scale_exp = e;
    return STT_OK;
}

stt_status stt_topk(stt_ctx *c, const float *snr_dev, int64_t n, int64_t first, int32_t K, int64_t *idx_dev,
                    float *val_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_range(c, first, n);
    if (s != STT_OK) return s;
    if (K < 0 || K > n || K > 8192) return fail(c, STT_ERANGE, "K=%d must be in [0, min(n, 8192)]", K);
    if (K == 0) return STT_OK;
    if (!snr_dev || (!idx_dev && !val_dev)) return fail(c, STT_EINVAL, "snr_dev and an output must be non-NULL");
    STT_HIP(c, hipSetDevice(c->device));
    return topk_launch(c, TopkScores{snr_dev}, n, first, K, 0, idx_dev, val_dev);
}

stt_status stt_rescore_f64(stt_ctx *c, const stt_map *map, const stt_gen *gen, const stt_track *tracks_dev,
                           int64_t n_tracks, int64_t first, const int64_t *idx_dev, int32_t K, int32_t norm,
                           double *z_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if (map->dtype != STT_C64F32) return fail(c, STT_EINVAL, "the FP64 re-score reads an FP32 (Y, sigma) map");
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    if (K < 0) return fail(c, STT_EINVAL, "K=%d", K);
    if (first < 0) return fail(c, STT_EINVAL, "first=%lld", (long long)first);
    if (tracks_dev && n_tracks < 0) return fail(c, STT_EINVAL, "n_tracks=%lld", (long long)n_tracks);
    GenP g{};
    if (!tracks_dev && (s = make_genp(c, gen, map->T, map->F, g)) != STT_OK) return s;
    if (K == 0) return STT_OK;
    if (!idx_dev || !z_dev) return fail(c, STT_EINVAL, "idx_dev and z_dev must be non-NULL");
    STT_HIP(c, hipSetDevice(c->device));
    const MapP m = to_mapp(map);
    const unsigned grid = (unsigned)(((int64_t)K * 64 + 255) / 256);
    if (tracks_dev)
        hipLaunchKernelGGL(k_rescore_f64<true>, dim3(grid), dim3(256), 0, c->stream, m, g, (const Trk *)tracks_dev,
                           n_tracks, (uint64_t)first, idx_dev, K, norm, z_dev);
    else
        hipLaunchKernelGGL(k_rescore_f64<false>, dim3(grid), dim3(256), 0, c->stream, m, g, (const Trk *)nullptr,
                           (int64_t)0, (uint64_t)first, idx_dev, K, norm, z_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

// ----------------------------------------------------------------------------- batches

stt_status stt_significance(stt_ctx *c, const uint64_t *bg_keys_dev, int64_t n_bg, const uint64_t *fg_keys_dev,
                            int64_t n_fg, double alpha, int64_t *n_louder_dev, float *fap_dev, float *z_alpha_dev)
{
    if (!c) return STT_EINVAL;
    if (n_bg < 1) return fail(c, STT_EINVAL, "need at least one background map");
    if (n_fg < 0) return fail(c, STT_EINVAL, "n_fg=%lld", (long long)n_fg);
    if (!bg_keys_dev) return fail(c, STT_EINVAL, "null background keys");
    if (n_fg > 0 && !fg_keys_dev && (n_louder_dev || fap_dev)) return fail(c, STT_EINVAL, "null foreground keys");
    if (n_bg > ((int64_t)1 << 38) || n_fg > ((int64_t)1 << 38))
        return fail(c, STT_ERANGE, "more than 2^38 keys");  // keeps the 1-D grids below 2^31 workgroups
    int32_t m = 0;
    if (z_alpha_dev) {
        if (!(alpha > 0.0 && alpha <= 1.0)) return fail(c, STT_EINVAL, "alpha must be in (0, 1]");
        const double mm = std::max(1.0, std::ceil(alpha * (double)n_bg));
        if (mm > 8192) return fail(c, STT_ERANGE, "ceil(alpha n_bg) = %.0f exceeds 8192", mm);
        m = (int32_t)mm;
    }
    STT_HIP(c, hipSetDevice(c->device));
    stt_status s;
    if (n_fg > 0 && (n_louder_dev || fap_dev)) {
        if ((s = count_louder(c, bg_keys_dev, n_bg, fg_keys_dev, n_fg, n_louder_dev, fap_dev)) != STT_OK) return s;
    }
    if (z_alpha_dev) {  // the m-th largest background score
        if ((s = check_range(c, 0, n_bg)) != STT_OK) return s;
        return topk_launch(c, TopkKeys{bg_keys_dev}, n_bg, 0, m, 1, nullptr, z_alpha_dev);
    }
    return STT_OK;
}

stt_status stt_follow_up(stt_ctx *c, const stt_map *maps_host, int32_t n_maps, uint64_t *keys_dev, const stt_gen *gen,
                         int64_t n_deep, int32_t k, int32_t norm, int32_t *chosen_host, int32_t *n_chosen)
{
    if (!c) return STT_EINVAL;
    if (n_chosen) *n_chosen = 0;
    if (n_maps < 1 || !maps_host || !keys_dev) return fail(c, STT_EINVAL, "need at least one map and its key");
    if (k < 1) return fail(c, STT_EINVAL, "k=%d must be >= 1", k);
    if (!gen) return fail(c, STT_EINVAL, "gen is NULL");
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    stt_status s;
    if ((s = check_range(c, 0, n_deep)) != STT_OK) return s;
    if ((uint64_t)gen->stream + (uint64_t)(n_maps - 1) > 0xFFFFFFFFull)
        return fail(c, STT_ERANGE, "Philox streams gen->stream + m overflow 32 bits");
    for (int32_t m = 0; m < n_maps; ++m) {
        if ((s = check_map(c, &maps_host[m])) != STT_OK) return s;
        GenP g;
        if ((s = make_genp(c, gen, maps_host[m].T, maps_host[m].F, g)) != STT_OK) return s;
    }
    STT_HIP(c, hipSetDevice(c->device));
    // rank of map m = the number of maps at least as loud, itself included (as stt_significance counts)
    if ((s = ensure_aux(c, sizeof(int64_t) * (size_t)n_maps)) != STT_OK) return s;
    int64_t *rank_dev = (int64_t *)c->aux;
    if ((s = count_louder(c, keys_dev, n_maps, keys_dev, n_maps, rank_dev, nullptr)) != STT_OK) return s;
    std::vector<int64_t> rank((size_t)n_maps);
    STT_HIP(c, hipMemcpyAsync(rank.data(), rank_dev, sizeof(int64_t) * (size_t)n_maps, hipMemcpyDeviceToHost,
                              c->stream));
    STT_HIP(c, hipStreamSynchronize(c->stream));
    int32_t done = 0;
    for (int32_t m = 0; m < n_maps; ++m) {
        if (rank[(size_t)m] > k) continue;
        if (n_deep > 0) {
            stt_gen gm = *gen;
            gm.stream = gen->stream + (uint32_t)m;
            if ((s = stt_score(c, &maps_host[m], &gm, nullptr, 0, n_deep, norm, nullptr, keys_dev + m)) != STT_OK)
                return s;
        }
        if (chosen_host) chosen_host[done] = m;
        ++done;
        if (n_chosen) *n_chosen = done;
    }
    return STT_OK;
}

stt_status stt_spectra(stt_ctx *c, const stt_spectro *p, const float *strain_dev, int64_t n_samples, int32_t T,
                       float *spec_dev, float *psd_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_spectro(c, p);
    if (s != STT_OK) return s;
    if (!strain_dev || !spec_dev || !psd_dev) return fail(c, STT_EINVAL, "null buffer");
    if (((uintptr_t)strain_dev & 7) || ((uintptr_t)spec_dev & 7) || ((uintptr_t)psd_dev & 3))
        return fail(c, STT_EINVAL, "strain and spec must be 8-byte aligned, psd 4-byte aligned");
    if (T < 4 || T > 65535) return fail(c, STT_ERANGE, "T=%d: need 4 <= T <= 65535", T);
    if (n_samples < 0 || (int64_t)(T + 1) * (p->M / 2) > n_samples)
        return fail(c, STT_ERANGE, "%d columns of %d samples need %lld samples, have %lld", T, p->M,
                    (long long)(T + 1) * (p->M / 2), (long long)n_samples);
    STT_HIP(c, hipSetDevice(c->device));
    if ((s = ensure_fft_tab(c, p->M)) != STT_OK) return s;
    if ((s = ev_begin(c)) != STT_OK) return s;
    const int N = p->M / 2;
    int lg = 0;
    while ((1 << lg) < N) ++lg;
    ev_record(c, 4);
    // a lane holds 8 points at a time. 1000 columns of 4096 samples: 28 us a stage at a time through LDS,
    // 15 us with three stages in registers.
    const int fft_wg = std::min(kFftThreads, std::max(64, N / 8));
    hipLaunchKernelGGL(k_col_fft, dim3(T), dim3(fft_wg), sizeof(float2) * fft_slot(N), c->stream, strain_dev, p->M, lg,
                       p->k_lo, p->F, (float)(1.0 / p->fs), (const float2 *)c->fft_tab, (float2 *)spec_dev);
    STT_HIP(c, hipGetLastError());
    const int psd_cols = (int64_t)T * p->F >= kPsdPixels ? 4 : 1;
    const dim3 psd_grid((p->F + 255) / 256, (T + psd_cols - 1) / psd_cols);
    if (psd_cols == 4)
        hipLaunchKernelGGL(k_psd<4>, psd_grid, dim3(256), 0, c->stream, (const float2 *)spec_dev, T, p->F,
                           std::min(p->nb, T), cross_scale(p), psd_dev);
    else
        hipLaunchKernelGGL(k_psd<1>, psd_grid, dim3(256), 0, c->stream, (const float2 *)spec_dev, T, p->F,
                           std::min(p->nb, T), cross_scale(p), psd_dev);
    STT_HIP(c, hipGetLastError());
    ev_record(c, 5);
    c->used[2] = true;
    ev_end(c);
    return STT_OK;
}

stt_status stt_form_maps(stt_ctx *c, const stt_spectro *p, int32_t T, const float *spec_i_dev, const float *psd_i_dev,
                         const float *spec_j_dev, const float *psd_j_dev, int32_t n_slides, const int32_t *shifts,
                         int64_t ld, float *const *Y_dev, float *const *sigma_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_spectro(c, p);
    if (s != STT_OK) return s;
    if (!spec_i_dev || !psd_i_dev || !spec_j_dev || !psd_j_dev) return fail(c, STT_EINVAL, "null spectrum");
    if (((uintptr_t)spec_i_dev & 7) || ((uintptr_t)spec_j_dev & 7)) return fail(c, STT_EINVAL, "spectra must be 8-byte aligned");
    if (T < 4 || T > 65535) return fail(c, STT_ERANGE, "T=%d: need 4 <= T <= 65535", T);
    if (n_slides < 0) return fail(c, STT_EINVAL, "n_slides=%d", n_slides);
    if (ld < p->F) return fail(c, STT_EINVAL, "ld=%lld < F=%d", (long long)ld, p->F);
    if (n_slides == 0) return STT_OK;
    if (!shifts || !Y_dev || !sigma_dev) return fail(c, STT_EINVAL, "null slide table");
    for (int k = 0; k < n_slides; ++k) {
        if (!Y_dev[k] || !sigma_dev[k]) return fail(c, STT_EINVAL, "slide %d: null output", k);
        if (((uintptr_t)Y_dev[k] & 7) || ((uintptr_t)sigma_dev[k] & 3))
            return fail(c, STT_EINVAL, "slide %d: misaligned output", k);
    }
    // two bins per lane where every row segment stays 16-byte aligned
    bool pair = (p->F % 2 == 0) && (ld % 2 == 0) && !((uintptr_t)spec_i_dev & 15) && !((uintptr_t)spec_j_dev & 15) &&
                !((uintptr_t)psd_i_dev & 7) && !((uintptr_t)psd_j_dev & 7);
    for (int k = 0; k < n_slides && pair; ++k)
        pair = !((uintptr_t)Y_dev[k] & 15) && !((uintptr_t)sigma_dev[k] & 7);
    const int per_lane = pair ? 2 : 1;
    const int64_t nchunk = ((int64_t)T * p->F + 256 * per_lane - 1) / (256 * per_lane);
    STT_HIP(c, hipSetDevice(c->device));
    if ((s = ev_begin(c)) != STT_OK) return s;
    ev_record(c, 4);
    ev_record(c, 0);
    // a launch holds below 2^32 lanes: at least 15 slides of the largest map
    const int64_t slide_wgs = 8 * ((nchunk + 7) / 8);
    const int per_launch = (int)std::min<int64_t>(kSlidesPerLaunch, (((int64_t)1 << 24) - 1) / slide_wgs);
    const bool runs = slide_wgs / 8 > kFormRun / (256 * per_lane);
    auto kern = pair ? (runs ? k_form_maps<2, true> : k_form_maps<2, false>)
                     : (runs ? k_form_maps<1, true> : k_form_maps<1, false>);
    // a launch writes its slides in no order: a buffer that comes again starts the next launch, so that
    // the last slide into it stands
    const auto taken = [](const SlideArgs &a, const float *Y, const float *sigma) {
        for (int k = 0; k < a.n; ++k)
            if ((const float *)a.Y[k] == Y || a.sigma[k] == sigma) return true;
        return false;
    };
    for (int k0 = 0; k0 < n_slides;) {
        SlideArgs a{};
        for (; k0 < n_slides && a.n < per_launch && !taken(a, Y_dev[k0], sigma_dev[k0]); ++k0, ++a.n) {
            a.Y[a.n] = (float2 *)Y_dev[k0];
            a.sigma[a.n] = sigma_dev[k0];
            const int64_t sh = shifts[k0] % T;
            a.shift[a.n] = (int32_t)(sh < 0 ? sh + T : sh);
        }
        const dim3 grid((unsigned)(slide_wgs * a.n));
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, c->stream, (const float2 *)spec_i_dev, psd_i_dev,
                           (const float2 *)spec_j_dev, psd_j_dev, T, p->F, cross_scale(p), ld, a);
        STT_HIP(c, hipGetLastError());
    }
    ev_record(c, 1);
    ev_record(c, 5);
    c->used[0] = true;
    c->used[2] = true;
    ev_end(c);
    return STT_OK;
}

}  // extern "C"

namespace {

template <int WG, int TPT, bool HW, int MAPT, int SC>
stt_status launch_batch_t(stt_ctx *c, hipStream_t st, const BatchMap *maps, int n_maps, const uint32_t *item_start,
                          uint32_t total_items, uint32_t *queue, const uint32_t *order, int32_t norm, uint64_t *best,
                          size_t shm)
{
    auto kern = k_score_batch<WG, TPT, HW, MAPT, SC>;
    if (shm > 64 * 1024)
        STT_HIP(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    int per_cu = 0;
    STT_HIP(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, WG, shm));
    if (per_cu < 1) return fail(c, STT_EUNSUPPORTED, "batch scorer %dx%d does not fit with %zu B of LDS", WG, TPT, shm);
    const unsigned grid = (unsigned)std::min<int64_t>((int64_t)per_cu * c->n_cu, total_items);
    if (grid == 0) return STT_OK;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WG), shm, st, maps, n_maps, item_start, queue, order, norm, best);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

template <bool HW, int MAPT, int SC>
stt_status launch_batch_h(stt_ctx *c, const SlabShape &sh, hipStream_t st, const BatchMap *maps, int n_maps, const uint32_t *item_start,
                          uint32_t total_items, uint32_t *queue, const uint32_t *order, int32_t norm, uint64_t *best,
                          size_t shm)
{
#define STT_BATCH_CASE(W, P)                                                                                        \
    if (sh.wg == W && sh.tpt == P)                                                                                  \
        return launch_batch_t<W, P, HW, MAPT, SC>(c, st, maps, n_maps, item_start, total_items, queue, order, norm, \
                                                  best, shm);
    STT_BATCH_CASE(1024, 4)
    STT_BATCH_CASE(512, 4)
    STT_BATCH_CASE(256, 4)
    STT_BATCH_CASE(1024, 2)
    STT_BATCH_CASE(512, 2)
#undef STT_BATCH_CASE
    return fail(c, STT_EUNSUPPORTED, "no batch scorer for %dx%d", sh.wg, sh.tpt);
}

template <typename T>
void key_add(std::vector<uint8_t> &k, const T &v)
{
    const uint8_t *b = (const uint8_t *)&v;
    k.insert(k.end(), b, b + sizeof(T));
}

}  // namespace

extern "C" {

stt_status stt_set_graph(stt_ctx *c, int32_t on)
{
    if (!c || on < 0 || on > 1) return STT_EINVAL;
    c->use_graph = on == 1;
    return STT_OK;
}

stt_status stt_score_batch(stt_ctx *c, const stt_map *maps_host, int32_t n_maps, const stt_gen *gen,
                           const int64_t *n_trk_host, int32_t norm, uint64_t *best_key_per_map_dev,
                           float *const *snr_dev_host)
{
    if (!c) return STT_EINVAL;
    if (n_maps < 0 || n_maps > 65536) return fail(c, STT_ERANGE, "n_maps=%d outside [0, 65536]", n_maps);
    if (n_maps == 0) return STT_OK;
    if (!maps_host || !n_trk_host || !gen) return fail(c, STT_EINVAL, "maps, gen and n_trk must be non-NULL");
    if (!best_key_per_map_dev) return fail(c, STT_EINVAL, "best_key_per_map_dev must be non-NULL");
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    const int dtype = maps_host[0].dtype;
    const int esize = fold_esize(dtype);
    std::vector<BatchMap> bm(n_maps);
    std::vector<uint32_t> chunk_start(n_maps + 1), item_start(n_maps + 1), fine_start(n_maps + 1);
    // one shape for the batch, by its total templates and widest column (what is out of range is refused below)
    int64_t n_total = 0, widest = 0;
    for (int i = 0; i < n_maps; ++i) {
        n_total += std::clamp<int64_t>(n_trk_host[i], 0, (int64_t)1 << 32);
        widest = std::max(widest, fold_ld(std::max(1, maps_host[i].F), esize) * esize);
    }
    const SlabShape sh = call_shape(c, n_total, widest);
    const int per_item = sh.wg * sh.tpt;
    uint64_t norder = 0, nchunks = 0, nitems = 0, nfine = 0;
    size_t ncc = 0;     // counts per group and sort chunk, all maps
    int max_groups = 1;  // most groups of any map
    size_t shm = 0;
    bool dma_ok = c->dma;  // every map's column fits two DMA slabs
    uint64_t fold_px = 0, fold_cols = 0;
    std::vector<uint64_t> fold_off(n_maps, 0), fold_col(n_maps, 0);
    int64_t max_ldc = 0;
    for (int i = 0; i < n_maps; ++i) {
        const stt_map *mp = &maps_host[i];
        stt_status s = check_map(c, mp);
        if (s != STT_OK) return fail(c, s, "map %d: %s", i, c->err.c_str());
        if (mp->dtype != dtype) return fail(c, STT_EINVAL, "all maps of a batch share one dtype");
        const int64_t n = n_trk_host[i];
        if (n < 0 || n > ((int64_t)1 << 32)) return fail(c, STT_ERANGE, "map %d: n_trk=%lld", i, (long long)n);
        stt_gen g = *gen;
        g.stream = gen->stream + (uint32_t)i;
        BatchMap &d = bm[i];
        if ((s = make_genp(c, &g, mp->T, mp->F, d.g)) != STT_OK) return fail(c, s, "map %d: %s", i, c->err.c_str());
        d.m = to_mapp(mp);
        d.n = n;
        d.order0 = norder;
        d.bin0 = (uint64_t)i * kMaxBins;
        d.wb = bucket_shift(mp->T, n);
        const int nb = ((mp->T - 1) >> d.wb) + 1;
        d.nbins = nb * (nb + 1) / 2;
        d.S = std::min(std::min<int>(64, (sh.lds - 256) / (esize * mp->F)), mp->T);
        if (d.S < 1) return fail(c, STT_EUNSUPPORTED, "map %d: F=%d too wide for the LDS slab", i, mp->F);
        {
            const int64_t ldc = fold_ld(mp->F, esize);
            dma_ok = dma_ok && aligned_slab(dma_slab_cols(sh.lds, ldc, esize)) >= 2;
            fold_off[i] = fold_px;
            fold_px += (uint64_t)mp->T * (uint64_t)ldc;
            fold_col[i] = fold_cols;
            fold_cols += (uint64_t)mp->T;
        }
        d.snr = snr_dev_host ? snr_dev_host[i] : nullptr;
        chunk_start[i] = (uint32_t)nchunks;
        fine_start[i] = (uint32_t)nfine;
        item_start[i] = (uint32_t)nitems;
        d.chunk0 = (int32_t)nchunks;
        norder += (uint64_t)n;
        nchunks += (uint64_t)((n + kBinChunk - 1) / kBinChunk);
        {
            const int ng = (d.nbins + kGroupMask) >> kGroupShift;
            nfine += (uint64_t)((n + kFineChunk - 1) / kFineChunk) + (uint64_t)ng;
            d.cc0 = ncc;
            ncc += (size_t)ng * (size_t)((n + kBinChunk - 1) / kBinChunk);
            max_groups = std::max(max_groups, ng);
        }
        nitems += (uint64_t)((n + per_item - 1) / per_item);
        if (norder >= ((uint64_t)1 << 32) || nitems >= ((uint64_t)1 << 31))
            return fail(c, STT_ERANGE, "a batch holds fewer than 2^32 templates");
    }
    chunk_start[n_maps] = (uint32_t)nchunks;
    fine_start[n_maps] = (uint32_t)nfine;
    item_start[n_maps] = (uint32_t)nitems;
    STT_HIP(c, hipSetDevice(c->device));
    // every map is scored from its polar fold (one launch folds them all); slabs stream in by DMA
    // when every map's column fits two of them, else through registers
    std::vector<MapP> orig(n_maps);
    for (int i = 0; i < n_maps; ++i) orig[i] = bm[i].m;
    {
        stt_status sf = ensure_pbuf(c, (size_t)esize * (size_t)fold_px);
        if (sf != STT_OK) return sf;
    }
    std::vector<FoldJob> jobs(n_maps + 1);
    shm = 0;
    // one aligned slab width for the whole batch: the narrowest any map's columns allow
    int sc_all = 16;
    if (dma_ok)
        for (int i = 0; i < n_maps; ++i)
            sc_all = std::min(sc_all, aligned_slab(dma_slab_cols(sh.lds, fold_ld(bm[i].m.F, esize), esize)));
    for (int i = 0; i < n_maps; ++i) {
        BatchMap &d = bm[i];
        const int64_t ldc = fold_ld(d.m.F, esize);
        void *dst = (char *)c->pbuf + (size_t)esize * fold_off[i];
        jobs[i] = FoldJob{orig[i], dst, ldc, (uint32_t)fold_col[i]};
        max_ldc = std::max(max_ldc, ldc);
        d.m.Y = (const float2 *)dst;  // an FP16 map keeps its scale 2^e
        d.m.sig = nullptr;
        d.m.ld = ldc;
        if (dma_ok) {
            d.S = sc_all;
            shm = std::max(shm, 2 * (size_t)esize * (size_t)d.S * (size_t)ldc);
        } else {
            shm = std::max(shm, (size_t)esize * (size_t)d.S * (size_t)d.m.F);
        }
    }
    jobs[n_maps] = FoldJob{MapP{}, nullptr, 0, (uint32_t)fold_cols};
    if (!c->n_cu) STT_HIP(c, hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, c->device));

    // scratch: [totals | cursor | queue | order (first the buckets of the count) | group starts | second-
    // scatter chunk tables | group regions | counts per group and sort chunk | buckets within the group]
    const size_t nb_all = (size_t)n_maps * kMaxBins;
    const size_t ng_all = (size_t)n_maps * kGroupSlots;
    const size_t need = sizeof(uint32_t) * (2 * nb_all + 64 + 2 * norder + 2 * ng_all + ncc) + norder;
    stt_status s = ensure_scratch(c, need);
    if (s != STT_OK) return s;
    uint32_t *totals = (uint32_t *)c->scratch;
    uint32_t *cursor = totals + nb_all;
    uint32_t *queue = cursor + nb_all;
    uint32_t *order = queue + 64;
    uint32_t *gstart = order + norder;
    uint32_t *fitem = gstart + ng_all;
    uint32_t *tmp = fitem + ng_all;
    uint32_t *ccnt = tmp + norder;
    uint8_t *tsub = (uint8_t *)(ccnt + ncc);
    uint16_t *bins = (uint16_t *)order;

    // the argument key: a repeat of the last batch replays its graph
    std::vector<uint8_t> key;
    key_add(key, n_maps);
    key_add(key, norm);
    key_add(key, best_key_per_map_dev);
    key_add(key, c->scratch);
    key_add(key, sh);
    key_add(key, c->hw_trig);
    key_add(key, dma_ok);
    key_add(key, sc_all);
    key_add(key, c->pbuf);
    for (const auto &d : bm) key_add(key, d);
    for (const auto &o : orig) key_add(key, o);
    const bool same = c->use_graph && c->gexec && key == c->bkey;

    if (!same) {
        // descriptor tables to the device (synchronous: they must outlive the call)
        const size_t tbl = sizeof(BatchMap) * n_maps + sizeof(FoldJob) * (n_maps + 1) + sizeof(uint32_t) * 3 * (n_maps + 1);
        if (tbl > c->bdev_bytes) {
            STT_HIP(c, hipStreamSynchronize(c->stream));
            if (c->bdev) (void)hipFree(c->bdev);
            c->bdev = nullptr;
            c->bdev_bytes = 0;
            if (hipMalloc(&c->bdev, tbl) != hipSuccess) {
                (void)hipGetLastError();
                return fail(c, STT_ENOMEM, "cannot allocate %zu bytes of batch tables", tbl);
            }
            c->bdev_bytes = tbl;
        }
        STT_HIP(c, hipStreamSynchronize(c->stream));  // the previous batch may still read the tables
        BatchMap *dmaps = (BatchMap *)c->bdev;
        FoldJob *djobs = (FoldJob *)(dmaps + n_maps);
        uint32_t *dchunk = (uint32_t *)(djobs + (n_maps + 1));
        uint32_t *ditem = dchunk + (n_maps + 1);
        uint32_t *dfine = ditem + (n_maps + 1);
        STT_HIP(c, hipMemcpy(dmaps, bm.data(), sizeof(BatchMap) * n_maps, hipMemcpyHostToDevice));
        STT_HIP(c, hipMemcpy(djobs, jobs.data(), sizeof(FoldJob) * (n_maps + 1), hipMemcpyHostToDevice));
        STT_HIP(c, hipMemcpy(dchunk, chunk_start.data(), sizeof(uint32_t) * (n_maps + 1), hipMemcpyHostToDevice));
        STT_HIP(c, hipMemcpy(ditem, item_start.data(), sizeof(uint32_t) * (n_maps + 1), hipMemcpyHostToDevice));
        STT_HIP(c, hipMemcpy(dfine, fine_start.data(), sizeof(uint32_t) * (n_maps + 1), hipMemcpyHostToDevice));
        if (c->gexec) { (void)hipGraphExecDestroy(c->gexec); c->gexec = nullptr; }
        if (c->graph) { (void)hipGraphDestroy(c->graph); c->graph = nullptr; }
        c->bkey.clear();

        auto enqueue = [&](hipStream_t st) -> stt_status {
            const bool timed = st == c->stream;  // events only outside graph capture
            if (timed) ev_record(c, 2);
            {
                const dim3 fg((unsigned)fold_cols, (unsigned)((max_ldc + 256 * kFoldRows - 1) / (256 * kFoldRows)));  // columns over x, rows over y
                if (dtype == STT_P16)
                    hipLaunchKernelGGL(k_fold_batch<kMapP16>, dim3(fg), dim3(256), 0, st, (const FoldJob *)djobs,
                                       n_maps);
                else
                    hipLaunchKernelGGL(k_fold_batch<kMapF32>, dim3(fg), dim3(256), 0, st, (const FoldJob *)djobs,
                                       n_maps);
            }
            hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((nb_all + 64 + 255) / 256)), dim3(256), 0, st, totals,
                               (int64_t)(nb_all), 0u);
            hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, queue, (int64_t)1, 0u);
            if (nchunks) {
                hipLaunchKernelGGL(k_bin_count_batch, dim3((unsigned)nchunks), dim3(256), 0, st,
                                   (const BatchMap *)dmaps, n_maps, (const uint32_t *)dchunk, totals, bins, ccnt);
                hipLaunchKernelGGL(k_bin_scan_batch, dim3((unsigned)(max_groups + 1) * (unsigned)n_maps), dim3(256), 0,
                                   st, (const BatchMap *)dmaps, (const uint32_t *)dchunk, max_groups,
                                   (const uint32_t *)totals, cursor, gstart, fitem, ccnt);
                hipLaunchKernelGGL(k_bin_group_batch, dim3((unsigned)nchunks), dim3(kScatterWG), 0, st,
                                   (const BatchMap *)dmaps, n_maps, (const uint32_t *)dchunk, (const uint16_t *)bins,
                                   (const uint32_t *)gstart, (const uint32_t *)ccnt, tmp, tsub);
                hipLaunchKernelGGL(k_bin_fine_batch, dim3((unsigned)nfine), dim3(kScatterWG), 0, st,
                                   (const BatchMap *)dmaps, n_maps, (const uint32_t *)dfine,
                                   (const uint32_t *)gstart, (const uint32_t *)fitem, cursor, (const uint32_t *)tmp,
                                   (const uint8_t *)tsub, order);
            }
            STT_HIP(c, hipGetLastError());
            if (timed) {
                ev_record(c, 3);
                ev_record(c, 0);
                c->used[0] = c->used[1] = true;
            }
            stt_status r;
            const uint32_t ni = (uint32_t)nitems;
            const int sc = dma_ok ? sc_all : 0;
#define STT_BATCH_SC(MT, SCV)                                                                                  \
    r = c->hw_trig ? launch_batch_h<true, MT, SCV>(c, sh, st, dmaps, n_maps, ditem, ni, queue, order, norm,        \
                                                   best_key_per_map_dev, shm)                                 \
                   : launch_batch_h<false, MT, SCV>(c, sh, st, dmaps, n_maps, ditem, ni, queue, order, norm,       \
                                                    best_key_per_map_dev, shm)
#define STT_BATCH_MT(MT)                                                                                       \
    switch (sc) {                                                                                              \
    case 0: STT_BATCH_SC(MT, 0); break;                                                                        \
    case 2: STT_BATCH_SC(MT, 2); break;                                                                        \
    case 4: STT_BATCH_SC(MT, 4); break;                                                                        \
    case 8: STT_BATCH_SC(MT, 8); break;                                                                        \
    case 16: STT_BATCH_SC(MT, 16); break;                                                                      \
    default: r = fail(c, STT_EUNSUPPORTED, "no batch scorer for %d-column slabs", sc);                        \
    }
            if (dtype == STT_P16) { STT_BATCH_MT(kMapPolH) } else { STT_BATCH_MT(kMapPol) }
#undef STT_BATCH_MT
#undef STT_BATCH_SC
            if (timed) ev_record(c, 1);
            return r;
        };

        if (!c->use_graph) {
            if ((s = ev_begin(c)) != STT_OK) return s;
            ev_record(c, 4);
            s = enqueue(c->stream);
            ev_record(c, 5);
            c->used[2] = true;
            ev_end(c);
            return s;
        }
        if (!c->cap_stream) STT_HIP(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
        STT_HIP(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed));
        s = enqueue(c->cap_stream);
        hipGraph_t g = nullptr;
        const hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
        if (s != STT_OK) {
            if (g) (void)hipGraphDestroy(g);
            return s;
        }
        if (e != hipSuccess) return fail(c, STT_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
        c->graph = g;
        STT_HIP(c, hipGraphInstantiate(&c->gexec, c->graph, nullptr, nullptr, 0));
        c->bkey = key;
    }
    if ((s = ev_begin(c)) != STT_OK) return s;
    ev_record(c, 4);
    STT_HIP(c, hipGraphLaunch(c->gexec, c->stream));
    ev_record(c, 5);
    c->used[2] = true;  // a replayed graph is timed as a whole
    ev_end(c);
    return STT_OK;
}

// ----------------------------------------------------------------------------- differentiation

stt_status stt_tracks_at(stt_ctx *c, const stt_gen *gen, int32_t T, int32_t F, const int64_t *idx_dev, int64_t n,
                         stt_track *out_dev)
{
    if (!c) return STT_EINVAL;
    GenP g;
    stt_status s = make_genp(c, gen, T, F, g);
    if (s != STT_OK) return s;
    if (n < 0) return fail(c, STT_EINVAL, "n=%lld", (long long)n);
    if (n == 0) return STT_OK;
    if (!idx_dev || !out_dev) return fail(c, STT_EINVAL, "idx_dev and out_dev must be non-NULL");
    STT_HIP(c, hipSetDevice(c->device));
    hipLaunchKernelGGL(k_tracks_at, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, g, idx_dev, n,
                       (Trk *)out_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

stt_status stt_tracks_to_theta(stt_ctx *c, const stt_track *tracks_dev, int64_t n, float *theta_dev, int32_t *K_dev)
{
    if (!c) return STT_EINVAL;
    if (n < 0) return fail(c, STT_EINVAL, "n=%lld", (long long)n);
    if (n == 0) return STT_OK;
    if (!tracks_dev || !theta_dev || !K_dev) return fail(c, STT_EINVAL, "NULL buffer");
    STT_HIP(c, hipSetDevice(c->device));
    hipLaunchKernelGGL(k_track_to_theta, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream,
                       (const Trk *)tracks_dev, n, theta_dev, K_dev);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

}  // extern "C"

namespace {

stt_status smooth_launch(stt_ctx *c, const stt_map *map, const float *theta, const int32_t *K, int32_t n, float *z,
                         float *grad, hipStream_t st)
{
    const MapP m = to_mapp(map);
    const unsigned grid = (unsigned)n;  // one workgroup per template
    if (map->dtype == STT_P16)
        hipLaunchKernelGGL(k_smooth_grad<kMapP16>, dim3(grid), dim3(kSmoothWG), 0, st, m, theta, K, n, z, grad);
    else
        hipLaunchKernelGGL(k_smooth_grad<kMapF32>, dim3(grid), dim3(kSmoothWG), 0, st, m, theta, K, n, z, grad);
    STT_HIP(c, hipGetLastError());
    return STT_OK;
}

stt_status check_smooth(stt_ctx *c, const stt_map *map, const float *theta, const int32_t *K, int32_t n, float *z)
{
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if (map->F < 2) return fail(c, STT_ERANGE, "the smooth statistic needs F >= 2");
    if (n < 0) return fail(c, STT_EINVAL, "n=%d", n);
    if (n > 0 && (!theta || !K || !z)) return fail(c, STT_EINVAL, "NULL buffer");
    return STT_OK;
}

}  // namespace

extern "C" {

stt_status stt_smooth(stt_ctx *c, const stt_map *map, const float *theta_dev, const int32_t *K_dev, int32_t n,
                      float *z_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_smooth(c, map, theta_dev, K_dev, n, z_dev);
    if (s != STT_OK || n == 0) return s;
    STT_HIP(c, hipSetDevice(c->device));
    return smooth_launch(c, map, theta_dev, K_dev, n, z_dev, nullptr, c->stream);
}

stt_status stt_grad(stt_ctx *c, const stt_map *map, const float *theta_dev, const int32_t *K_dev, int32_t n,
                    float *z_dev, float *grad_dev)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_smooth(c, map, theta_dev, K_dev, n, z_dev);
    if (s != STT_OK || n == 0) return s;
    if (!grad_dev) return fail(c, STT_EINVAL, "grad_dev is NULL");
    STT_HIP(c, hipSetDevice(c->device));
    return smooth_launch(c, map, theta_dev, K_dev, n, z_dev, grad_dev, c->stream);
}

stt_status stt_refine(stt_ctx *c, const stt_map *map, int32_t min_len, int32_t dtau_max, float *theta_dev,
                      const int32_t *K_dev, int32_t n, int32_t steps, const float *sched_host, float *z_smooth_dev,
                      stt_track *plain_dev, float *z_plain_dev, int32_t norm)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_smooth(c, map, theta_dev, K_dev, n, z_smooth_dev);
    if (s != STT_OK) return s;
    if (steps < 0 || steps > 100000) return fail(c, STT_ERANGE, "steps=%d", steps);
    if (min_len < 2 || min_len > map->T) return fail(c, STT_ERANGE, "min_len=%d outside [2, T]", min_len);
    if (dtau_max < 0 || dtau_max >= (1 << 30)) return fail(c, STT_ERANGE, "dtau_max=%d", dtau_max);
    if (norm != STT_NORM_SQRT_N && norm != STT_NORM_N) return fail(c, STT_EINVAL, "norm=%d", norm);
    if (z_plain_dev && !plain_dev) return fail(c, STT_EINVAL, "z_plain_dev needs plain_dev");
    if (n == 0) return STT_OK;
    STT_HIP(c, hipSetDevice(c->device));
    RefineP p;
    p.T = map->T;
    p.F = map->F;
    p.L = min_len;
    p.dmax_ms = (double)dtau_max * (1e3 / 268435456.0);
    p.px0 = sched_host ? sched_host[0] : 1.0;
    p.px1 = sched_host ? sched_host[1] : 0.02;
    p.ms0 = sched_host ? sched_host[2] : 0.5;
    p.ms1 = sched_host ? sched_host[3] : 0.01;
    p.steps = steps;
    const MapP m = to_mapp(map);
    // The steps gather p = Y/sigma from the folded copy the scorers use (bit-identical to forming
    // it at each gather: one division per pixel instead of one per gather, 8 bytes instead of 12).
    const int64_t ldc = fold_ld(m.F);
    if ((s = ensure_pbuf(c, sizeof(float2) * (size_t)m.T * (size_t)ldc)) != STT_OK) return s;
    // timing: the refinement kernel is this call's stage 0 (the plain re-score below records its own)
    if ((s = ev_begin(c)) != STT_OK) return s;
    ev_record(c, 4);
    const unsigned fg = (unsigned)std::min<int64_t>(((int64_t)m.T * ldc + 255) / 256, 4096);
    if (map->dtype == STT_P16)
        hipLaunchKernelGGL(k_fold_p<kMapP16>, dim3(fg), dim3(256), 0, c->stream, m, (float2 *)c->pbuf, ldc);
    else
        hipLaunchKernelGGL(k_fold_p<kMapF32>, dim3(fg), dim3(256), 0, c->stream, m, (float2 *)c->pbuf, ldc);
    MapP mf = m;
    mf.Y = (const float2 *)c->pbuf;
    mf.sig = nullptr;
    mf.ld = ldc;
    ev_record(c, 0);
    // 1024 templates x 51 evaluations on 1000 x 1000: 335 us with a phase per node, an FP64 division per
    // sample and 84 exchanges per wave; 283 us without; 245 us with its registers held to 128, so that 4
    // instead of 3 workgroups share a CU and 1024 templates run in one round.
    hipLaunchKernelGGL(k_refine<kMapPF>, dim3((unsigned)n), dim3(kSmoothWG), 0, c->stream, mf, theta_dev, K_dev, n,
                       z_smooth_dev, p);
    STT_HIP(c, hipGetLastError());
    ev_record(c, 1);
    ev_record(c, 5);
    c->used[0] = true;
    c->used[2] = true;
    ev_end(c);
    if (plain_dev) {
        hipLaunchKernelGGL(k_theta_to_track, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream,
                           (const float *)theta_dev, (int64_t)n,
                           map->T, map->F, min_len, dtau_max, (Trk *)plain_dev);
        STT_HIP(c, hipGetLastError());
        if (z_plain_dev) {
            const int old = c->path;
            c->path = 0;  // automatic: a short explicit list takes one wave per template
            s = stt_score(c, map, nullptr, plain_dev, 0, n, norm, z_plain_dev, nullptr);
            c->path = old;
            if (s != STT_OK) return s;
        }
    }
    return STT_OK;
}

// ----------------------------------------------------------------------------- autotuning

}  // extern "C"

namespace {

struct TuneChoice {
    int wg, tpt, lds;
    double ms;
};

std::string gpu_arch(const stt_ctx *c)
{
    hipDeviceProp_t prop;
    std::string arch = "gpu";
    if (hipGetDeviceProperties(&prop, c->device) == hipSuccess) arch = prop.gcnArchName;
    return arch.substr(0, arch.find(':'));
}

int log2_floor(int64_t v)
{
    int b = 0;
    while (((int64_t)1 << (b + 1)) <= v) ++b;
    return b;
}

// Generation of the scorers' inner loop: part of every cache key, so that choices timed on an
// earlier loop are searched again. "pol3": polar folded map, one cosine per pixel, rows carried by one
// FP64 add (lazy rows), slabs streamed by scalar-addressed DMA, two templates per lane at 64 VGPRs.
constexpr const char *kCoreTag = "pol3";

// maps of similar duration (power-of-two bucket) and call size share a choice
std::string tune_key(const stt_ctx *c, const stt_map *m, int64_t n)
{
    char buf[192];
    snprintf(buf, sizeof buf, "%s/%s/F=%d/dtype=%d/T=2^%d/n=2^%d/trig=%d", gpu_arch(c).c_str(), kCoreTag, m->F,
             m->dtype, log2_floor(m->T), log2_floor(n), c->hw_trig ? 1 : 0);
    return buf;
}

std::string tune_key_batch(const stt_ctx *c, int F, int dtype, int T, int n_maps, int64_t n_total)
{
    char buf[224];
    snprintf(buf, sizeof buf, "%s/%s/batch/F=%d/dtype=%d/T=2^%d/maps=2^%d/n=2^%d/trig=%d", gpu_arch(c).c_str(),
             kCoreTag, F, dtype, log2_floor(T), log2_floor(n_maps), log2_floor(n_total), c->hw_trig ? 1 : 0);
    return buf;
}

// Times `call` (which must leave a timed scoring stage) for every compiled
// shape and LDS budget that fits columns of F pixels: `reps` timed runs after
// one warm-up, mean of the scoring kernel's HIP-event time. The context's
// shape, budget, timing and graph settings and the caller's pending timing
// records are restored afterwards.
stt_status tune_search(stt_ctx *c, int F, int reps, const std::function<stt_status()> &call, TuneChoice &best)
{
    const int old_path = c->path, old_wg = c->slab_wg, old_tpt = c->slab_tpt, old_lds = c->lds_bytes;
    const bool old_timing = c->timing, old_graph = c->use_graph, old_set = c->shape_set;
    c->shape_set = true;
    std::vector<Rec> saved;
    saved.swap(c->recs);
    const size_t saved_next = c->next;
    c->timing = true;
    c->use_graph = false;
    c->recs.clear();
    c->next = saved_next;  // tuning events come after any the caller has not read yet
    static const int ldss[] = {160 * 1024, 112 * 1024, 80 * 1024, 48 * 1024, 40 * 1024};
    stt_status s = STT_OK;
    for (const auto &sh : kShapes) {
        for (int lds : ldss) {
            if ((lds - 256) / (8 * F) < 1) continue;
            c->path = 2;
            c->slab_wg = sh[0];
            c->slab_tpt = sh[1];
            c->lds_bytes = lds;
            double tot = 0;
            int cnt = 0;
            for (int rep = 0; rep <= reps && s == STT_OK; ++rep) {
                if ((s = call()) != STT_OK) break;
                float ms = 0;
                if ((s = stt_kernel_ms(c, 0, &ms)) != STT_OK) break;
                if (rep > 0) { tot += ms; ++cnt; }  // the first run warms up
            }
            c->recs.clear();
            c->next = saved_next;
            if (s != STT_OK) break;
            if (cnt && tot / cnt < best.ms) best = TuneChoice{sh[0], sh[1], lds, tot / cnt};
        }
        if (s != STT_OK) break;
    }
    c->path = old_path;
    c->slab_wg = old_wg;
    c->slab_tpt = old_tpt;
    c->lds_bytes = old_lds;
    c->timing = old_timing;
    c->use_graph = old_graph;
    c->shape_set = old_set;
    c->recs.swap(saved);
    c->next = saved_next;
    if (s != STT_OK) return s;
    if (best.wg == 0) return fail(c, STT_EUNSUPPORTED, "no slab configuration fits F=%d", F);
    return STT_OK;
}

stt_status apply_choice(stt_ctx *c, const std::string &key, const TuneChoice &best, int32_t *choice_out)
{
    if (!slab_shape_ok(best.wg, best.tpt) || best.lds < 1024 || best.lds > 160 * 1024)
        return fail(c, STT_EINVAL, "cache entry for %s is not a valid configuration", key.c_str());
    c->slab_wg = best.wg;
    c->slab_tpt = best.tpt;
    c->lds_bytes = best.lds;
    c->shape_set = true;
    if (choice_out) {
        choice_out[0] = best.wg;
        choice_out[1] = best.tpt;
        choice_out[2] = best.lds;
    }
    return STT_OK;
}

// The cache file holds one line per key:  "<key>": {"wg": W, "tpt": P, "lds": B, "ms": T}
bool cache_lookup(const char *path, const std::string &key, TuneChoice &out)
{
    if (!path) return false;
    FILE *f = fopen(path, "r");
    if (!f) return false;
    char line[512];
    bool found = false;
    const std::string pat = "\"" + key + "\":";
    while (fgets(line, sizeof line, f)) {
        const char *p = strstr(line, pat.c_str());
        if (!p) continue;
        TuneChoice t;
        if (sscanf(p + pat.size(), " {\"wg\": %d, \"tpt\": %d, \"lds\": %d, \"ms\": %lf}", &t.wg, &t.tpt, &t.lds,
                   &t.ms) == 4) {
            out = t;
            found = true;
        }
    }
    fclose(f);
    return found;
}

void cache_store(const char *path, const std::string &key, const TuneChoice &t)
{
    if (!path) return;
    std::vector<std::string> lines;
    if (FILE *f = fopen(path, "r")) {
        char line[512];
        const std::string pat = "\"" + key + "\":";
        while (fgets(line, sizeof line, f)) {
            std::string l(line);
            while (!l.empty() && (l.back() == '\n' || l.back() == ',')) l.pop_back();
            // keep the other entries only: braces (also "{}" of an empty cache) are written anew
            const size_t q = l.find_first_not_of(" \t");
            if (q == std::string::npos || l[q] != '"' || l.find(pat) != std::string::npos) continue;
            lines.push_back(l);
        }
        fclose(f);
    }
    char buf[512];
    snprintf(buf, sizeof buf, "  \"%s\": {\"wg\": %d, \"tpt\": %d, \"lds\": %d, \"ms\": %.6f}", key.c_str(), t.wg,
             t.tpt, t.lds, t.ms);
    lines.push_back(buf);
    const std::string tmp = std::string(path) + ".tmp";
    if (FILE *f = fopen(tmp.c_str(), "w")) {
        fprintf(f, "{\n");
        for (size_t i = 0; i < lines.size(); ++i) fprintf(f, "%s%s\n", lines[i].c_str(), i + 1 < lines.size() ? "," : "");
        fprintf(f, "}\n");
        fclose(f);
        rename(tmp.c_str(), path);
    }
}

}  // namespace

extern "C" {

stt_status stt_autotune(stt_ctx *c, const stt_map *map, const stt_gen *gen, int64_t n, const char *cache_path,
                        int32_t *choice_out)
{
    if (!c) return STT_EINVAL;
    stt_status s = check_map(c, map);
    if (s != STT_OK) return s;
    if (n < 1 || n > ((int64_t)1 << 32)) return fail(c, STT_ERANGE, "n=%lld", (long long)n);
    GenP gp;
    if ((s = make_genp(c, gen, map->T, map->F, gp)) != STT_OK) return s;
    const std::string key = tune_key(c, map, n);
    TuneChoice best{0, 0, 0, 1e30};
    if (!cache_lookup(cache_path, key, best)) {
        s = tune_search(c, map->F, 3, [&] { return stt_score(c, map, gen, nullptr, 0, n, STT_NORM_SQRT_N, nullptr, nullptr); },
                        best);
        if (s != STT_OK) return s;
        cache_store(cache_path, key, best);
    }
    return apply_choice(c, key, best, choice_out);
}

stt_status stt_autotune_batch(stt_ctx *c, const stt_map *maps_host, int32_t n_maps, const stt_gen *gen,
                              const int64_t *n_trk_host, const char *cache_path, int32_t *choice_out)
{
    if (!c) return STT_EINVAL;
    if (n_maps < 1 || n_maps > 65536) return fail(c, STT_ERANGE, "n_maps=%d outside [1, 65536]", n_maps);
    if (!maps_host || !gen || !n_trk_host) return fail(c, STT_EINVAL, "maps, gen and n_trk must be non-NULL");
    int Fmax = 0, Tmax = 0;
    int64_t ntot = 0;
    for (int i = 0; i < n_maps; ++i) {
        stt_status s = check_map(c, &maps_host[i]);
        if (s != STT_OK) return s;
        if (n_trk_host[i] < 0) return fail(c, STT_ERANGE, "n_trk[%d] < 0", i);
        Fmax = std::max(Fmax, maps_host[i].F);
        Tmax = std::max(Tmax, maps_host[i].T);
        ntot += n_trk_host[i];
    }
    if (ntot < 1) return fail(c, STT_ERANGE, "no templates to time");
    const std::string key = tune_key_batch(c, Fmax, maps_host[0].dtype, Tmax, n_maps, ntot);
    TuneChoice best{0, 0, 0, 1e30};
    if (!cache_lookup(cache_path, key, best)) {
        void *keys = nullptr;
        STT_HIP(c, hipSetDevice(c->device));
        if (hipMalloc(&keys, sizeof(uint64_t) * (size_t)n_maps) != hipSuccess) {
            (void)hipGetLastError();
            return fail(c, STT_ENOMEM, "cannot allocate the tuner's %d keys", n_maps);
        }
        stt_status s = tune_search(c, Fmax, 2, [&] {
            return stt_score_batch(c, maps_host, n_maps, gen, n_trk_host, STT_NORM_SQRT_N, (uint64_t *)keys, nullptr);
        }, best);
        (void)hipStreamSynchronize(c->stream);
        (void)hipFree(keys);
        if (s != STT_OK) return s;
        cache_store(cache_path, key, best);
    }
    return apply_choice(c, key, best, choice_out);
}

uint64_t stt_key_encode(float z, uint32_t j) { return key_encode(z, j); }

void stt_key_decode(uint64_t key, float *z, uint32_t *j)
{
    const uint32_t o = (uint32_t)(key >> 32);
    const uint32_t b = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    if (z) std::memcpy(z, &b, sizeof b);
    if (j) *j = 0xFFFFFFFFu - (uint32_t)key;
}

}  // extern "C"
