// Host harness around the library's host side (stt_api.hip) with the HIP runtime replaced by a
// recorder: no GPU is touched. Reads commands from stdin, prints one line for each.
//   louder n_ref n_q have cap malloc sync -> the counts' status, allocations, launched kernels and "message" if an
//       error message is left, with
//       `have` bytes of scratch, a stream that captures (cap 1) or whose query fails (cap 2), and these
//       statuses of hipMalloc and hipStreamSynchronize
//   slides T F n (y s) x n -> status of stt_form_maps of n slides into buffers number y (Y) and s (sigma),
//       F even, and the slides of each launch
//   topk bytes n K cap -> after another call took `bytes` of the auxiliary scratch: status of stt_topk
//       and its allocations, which fail while the stream captures (cap 1)
//   shape wg tpt lds ... - n col_bytes -> the slab shape of a call of n templates on columns of col_bytes, after
//       stt_set_slab_shape(wg, tpt) (0 0: not called) and a stt_set_path for each lds (0: budget kept)
//   batch n0 n1 -> status of stt_score_batch for two maps of these many templates
//   items per n run -> (slide, place) of the per n workgroups that an XCD takes of a slide launch, in order
//   md T F esize n L n_tau -> the delay grid's scorer (lane, slab or wave) for n generated templates of L
//       columns or more
//   tm T F esize n L -> the free-t_mid scorer (slab or wave) for n generated templates of L columns or more
//   gather T F p16 wave n launches -> 1 if that direct call reads the caller's map unfolded
//   class dma workgroups n_cu nb -> extents per class of the sort
//   one bytes T n mean -> 1 if lanes gather one pixel at a time
//   plain T n -> the plain search's scorer by size
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

namespace fake {
std::string launches;
std::vector<unsigned> grids;
int n_malloc = 0;
hipError_t malloc_status = hipSuccess, sync_status = hipSuccess, capture_query = hipSuccess;
hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;

hipError_t Malloc(void **p, size_t bytes)
{
    ++n_malloc;
    if (malloc_status != hipSuccess) return malloc_status;
    if (capture != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    *p = std::malloc(bytes);
    return hipSuccess;
}
hipError_t Free(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t IsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capture;
    return capture_query;
}
void launch(const char *kernel, dim3 grid)
{
    launches += " " + std::string(kernel) + ":" + std::to_string(grid.x);
    grids.push_back(grid.x);
}
void reset()
{
    launches.clear();
    grids.clear();
    n_malloc = 0;
    malloc_status = sync_status = capture_query = hipSuccess;
    capture = hipStreamCaptureStatusNone;
}
}  // namespace fake

#define hipMalloc(p, n) fake::Malloc((void **)(p), n)
#define hipFree(p) fake::Free(p)
#define hipSetDevice(d) hipSuccess
#define hipGetLastError() hipSuccess
#define hipStreamSynchronize(s) fake::sync_status
#define hipStreamIsCapturing(s, p) fake::IsCapturing(s, p)
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kern, grid, ...) fake::launch(#kern, grid)

#include "stt_api.hip"

static int louder()
{
    long long n_ref, n_q, have;
    int cap, m, s;
    if (std::scanf("%lld %lld %lld %d %d %d", &n_ref, &n_q, &have, &cap, &m, &s) != 6) return 2;
    fake::reset();
    stt_ctx c;
    if (have && ensure_mdbuf(&c, (size_t)have) != STT_OK) return 2;
    fake::n_malloc = 0;
    fake::capture = cap == 1 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    fake::capture_query = cap == 2 ? hipErrorStreamCaptureImplicit : hipSuccess;
    fake::malloc_status = (hipError_t)m;
    fake::sync_status = (hipError_t)s;
    const stt_status st = count_louder(&c, nullptr, n_ref, nullptr, n_q, nullptr, nullptr);
    std::printf("%d %d%s%s\n", st, fake::n_malloc, fake::launches.c_str(), c.err.empty() ? "" : " message");
    return 0;
}

static int slides()
{
    int T, F, n, y, sg;
    if (std::scanf("%d %d %d", &T, &F, &n) != 3) return 2;
    fake::reset();
    stt_ctx c;
    alignas(16) static float in[4];
    std::vector<float *> Y, S;
    std::vector<int32_t> shifts(n, 0);
    for (int k = 0; k < n; ++k) {
        if (std::scanf("%d %d", &y, &sg) != 2) return 2;
        Y.push_back((float *)((uintptr_t)1 << 40) + ((size_t)y << 32));
        S.push_back((float *)((uintptr_t)1 << 48) + ((size_t)sg << 32));
    }
    stt_spectro p{4096.0, 8192, 0, F, 4};
    const stt_status st = stt_form_maps(&c, &p, T, in, in, in, in, n, shifts.data(), F, Y.data(), S.data());
    const int per = 8 * ((T * F + 4095) / 4096);  // workgroups a slide takes, two bins per lane
    std::printf("%d", st);
    for (unsigned g : fake::grids) std::printf(" %u", g % per ? 0u : g / per);
    std::printf("\n");
    return 0;
}

static int topk()
{
    long long bytes, n;
    int K, cap;
    if (std::scanf("%lld %lld %d %d", &bytes, &n, &K, &cap) != 4) return 2;
    fake::reset();
    stt_ctx c;
    if (bytes && ensure_aux(&c, (size_t)bytes) != STT_OK) return 2;
    fake::n_malloc = 0;
    fake::capture = cap ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    float z = 0.0f;
    int64_t idx = 0;
    const stt_status st = stt_topk(&c, &z, n, 0, K, &idx, &z);
    std::printf("%d %d\n", st, fake::n_malloc);
    return 0;
}

static int shape()
{
    int wg, tpt;
    char w[32];
    long long n, col;
    if (std::scanf("%d %d", &wg, &tpt) != 2) return 2;
    stt_ctx c;
    if (wg && stt_set_slab_shape(&c, wg, tpt) != STT_OK) return 2;
    while (std::scanf("%31s", w) == 1 && std::strcmp(w, "-"))
        if (stt_set_path(&c, 0, std::atoi(w)) != STT_OK) return 2;
    if (std::scanf("%lld %lld", &n, &col) != 2) return 2;
    const SlabShape sh = call_shape(&c, n, col);
    std::printf("%d %d %d\n", sh.wg, sh.tpt, sh.lds);
    return 0;
}

static int batch()
{
    long long n0, n1;
    if (std::scanf("%lld %lld", &n0, &n1) != 2) return 2;
    fake::reset();
    stt_ctx c;
    float y[2], sg = 1.0f;
    stt_map m{};
    m.Y = y;
    m.sigma = &sg;
    m.T = 100;
    m.F = 64;
    m.ld = 64;
    m.dtype = STT_C64F32;
    const stt_map maps[2] = {m, m};
    const int64_t n[2] = {n0, n1};
    stt_gen g{};
    g.min_len = 10;
    uint64_t best[2] = {};
    std::printf("%d\n", stt_score_batch(&c, maps, 2, &g, n, STT_NORM_N, best, nullptr));
    return 0;
}

static int items()
{
    unsigned per, n, run;
    if (std::scanf("%u %u %u", &per, &n, &run) != 3) return 2;
    for (unsigned b = 0; b < per * n; ++b) {
        const SlideItem w = slide_item(b, per, n, run);
        std::printf("%u %u ", w.k, w.at);
    }
    std::printf("\n");
    return 0;
}

static int md()
{
    int T, F, e, L, n_tau;
    long long n;
    if (std::scanf("%d %d %d %lld %d %d", &T, &F, &e, &n, &L, &n_tau) != 6) return 2;
    const bool wave = prefer_wave_md(T, n);
    const bool slab = prefer_slabs_md(T, n) || slabs_beat_direct_md(T, fold_ld(F, e) * e, e == 4, n, L + (T - L) / 3.0,
                                                                    (n_tau + kMD - 1) / kMD, wave);
    std::printf("%s\n", slab ? "slab" : wave ? "wave" : "lane");
    return 0;
}

static int tm()
{
    int T, F, e, L;
    long long n;
    if (std::scanf("%d %d %d %lld %d", &T, &F, &e, &n, &L) != 5) return 2;
    std::printf("%s\n", prefer_slabs_tm(T, fold_ld(F, e) * e, n, L + (T - L) / 3.0) ? "slab" : "wave");
    return 0;
}

static int gather()
{
    int T, F, p16, wave, launches;
    long long n;
    if (std::scanf("%d %d %d %d %lld %d", &T, &F, &p16, &wave, &n, &launches) != 6) return 2;
    stt_map m{};
    m.T = T;
    m.F = F;
    m.dtype = p16 ? STT_P16 : STT_C64F32;
    std::printf("%d\n", gather_unfolded(&m, wave != 0, n, launches));
    return 0;
}

static int sclass()
{
    int dma, n_cu, nb;
    long long wgs;
    if (std::scanf("%d %lld %d %d", &dma, &wgs, &n_cu, &nb) != 4) return 2;
    std::printf("%u\n", sort_class(dma != 0, wgs, n_cu, nb));
    return 0;
}

static int one()
{
    long long bytes, n;
    int T;
    double mean;
    if (std::scanf("%lld %d %lld %lf", &bytes, &T, &n, &mean) != 4) return 2;
    std::printf("%d\n", lane_gathers_one(bytes, T, n, mean));
    return 0;
}

static int plain()
{
    int T;
    long long n;
    if (std::scanf("%d %lld", &T, &n) != 2) return 2;
    std::printf("%s\n", prefer_slabs(T, n) ? "k_score_slab" : prefer_wave(T, n) ? "k_score_wave" : "k_score_direct");
    return 0;
}

int main()
{
    char cmd[16];
    while (std::scanf("%15s", cmd) == 1) {
        const int bad = !std::strcmp(cmd, "louder") ? louder() : !std::strcmp(cmd, "slides") ? slides()
                        : !std::strcmp(cmd, "topk") ? topk()
                        : !std::strcmp(cmd, "shape") ? shape()
                        : !std::strcmp(cmd, "batch") ? batch()
                        : !std::strcmp(cmd, "items") ? items()
                        : !std::strcmp(cmd, "md") ? md()
                        : !std::strcmp(cmd, "tm") ? tm()
                        : !std::strcmp(cmd, "gather") ? gather()
                        : !std::strcmp(cmd, "class") ? sclass()
                        : !std::strcmp(cmd, "one") ? one()
                        : !std::strcmp(cmd, "plain") ? plain() : 2;
        if (bad) return bad;
    }
    return 0;
}

// The device code's registration, which would reach for a GPU.
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h = nullptr; return &h; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
