// Significance of per-map maxima (the step after the search): Sec. V records each map's
// maximum statistic; background maps (time slides) give its distribution in noise, and a map
// is significant at false-alarm probability FAP < alpha (Sec. IV: 0.1 %).
//
//   k_count_louder  for each query key, the number of reference keys at least as loud,
//                   compared on the keys' high words (the order-preserving image of the FP32
//                   score; an empty key, 0, is quieter than every score)
//   k_rank_*        the same counts over many references: sorted queries, bisection, suffix sums
// The threshold is the last of a top-K select over the keys' scores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stt {

constexpr int kLouderTile = 4096;  // reference high words staged in LDS per pass (16 KB)

// Grid: ceil(n_q / 256) workgroups of 256 lanes, one query per lane.
__global__ __launch_bounds__(256) void k_count_louder(const uint64_t *__restrict__ ref, int64_t n_ref,
                                                      const uint64_t *__restrict__ q, int64_t n_q,
                                                      int64_t *__restrict__ count, float *__restrict__ fap,
                                                      double n_div)
{
    __shared__ __attribute__((aligned(16))) uint32_t tile[kLouderTile];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t hq = i < n_q ? (uint32_t)(q[i] >> 32) : 0u;
    int64_t c = 0;
    for (int64_t r0 = 0; r0 < n_ref; r0 += kLouderTile) {
        const int m = (int)(n_ref - r0 < kLouderTile ? n_ref - r0 : kLouderTile);
        __syncthreads();
        for (int k = threadIdx.x; k < m; k += 256) tile[k] = (uint32_t)(ref[r0 + k] >> 32);
        __syncthreads();
        int cc = 0;
        const int m4 = m & ~3;
        for (int k = 0; k < m4; k += 4) {  // one broadcast 16-byte LDS read per four references
            const uint4 v = *reinterpret_cast<const uint4 *>(tile + k);
            cc += (v.x >= hq) + (v.y >= hq) + (v.z >= hq) + (v.w >= hq);
        }
        for (int k = m4; k < m; ++k) cc += tile[k] >= hq;
        c += cc;
    }
    if (i < n_q) {
        if (count) count[i] = c;
        if (fap) fap[i] = (float)((double)c / n_div);
    }
}

// Counts over many reference keys. The direct count above walks them in one workgroup per 256
// queries (17 ns per reference whatever the number of queries up to 10^5: 17.5 ms for 10^6), so where
// that takes longer (prefer_ranks) the queries are sorted in tiles (k_rank_sort), every reference finds
// its place among a tile's queries by bisection in LDS (k_rank_count), and the place histogram's
// suffix sums are the counts (k_rank_finish): 10^6 references and 1000 queries in 36 us (sort 16, count 15,
// sums 5).
constexpr int kRankTile = 4096;       // queries per tile
constexpr int kRankTiles = 64;        // tiles per pass

struct RankTile {
    uint32_t hi[kRankTile];                // sorted high words
    uint32_t pos[kRankTile];               // the query each belongs to, within the tile
    unsigned long long hist[kRankTile + 1];  // references with exactly i queries at or below them
};

// Sort of tile blockIdx.x: queries q[q0 + tile * kRankTile ..) by high word (bitonic in LDS).
__global__ __launch_bounds__(1024) void k_rank_sort(const uint64_t *__restrict__ q, int64_t n_q, RankTile *tiles)
{
    __shared__ uint64_t kk[kRankTile];
    const int64_t base = (int64_t)blockIdx.x * kRankTile;
    const int m = (int)(n_q - base < kRankTile ? n_q - base : kRankTile);
    RankTile &t = tiles[blockIdx.x];
    int P = 64;
    while (P < m) P <<= 1;
    for (int i = threadIdx.x; i < P; i += 1024)
        kk[i] = i < m ? (q[base + i] & 0xFFFFFFFF00000000ull) | (uint32_t)i : ~0ull;
    for (int i = threadIdx.x; i <= m; i += 1024) t.hist[i] = 0;
    __syncthreads();
    for (int size = 2; size <= P; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int p = threadIdx.x; p < P / 2; p += 1024) {
                const int i = ((p & ~(stride - 1)) << 1) | (p & (stride - 1)), j = i + stride;
                const uint64_t a = kk[i], b = kk[j];
                if ((i & size) == 0 ? a > b : a < b) { kk[i] = b; kk[j] = a; }
            }
            __syncthreads();
        }
    for (int i = threadIdx.x; i < m; i += 1024) {
        t.hi[i] = (uint32_t)(kk[i] >> 32);
        t.pos[i] = (uint32_t)kk[i];
    }
}

// Grid: (blocks over the references, tiles). hist[i] += the references at or above exactly i of
// the tile's queries (i = 0 counts for none and is left out).
__global__ __launch_bounds__(1024) void k_rank_count(const uint64_t *__restrict__ ref, int64_t n_ref, int64_t n_q,
                                                     RankTile *tiles)
{
    __shared__ uint32_t hi[kRankTile];
    __shared__ uint32_t hist[kRankTile + 1];
    RankTile &t = tiles[blockIdx.y];
    const int64_t base = (int64_t)blockIdx.y * kRankTile;
    const int m = (int)(n_q - base < kRankTile ? n_q - base : kRankTile);
    for (int i = threadIdx.x; i < m; i += 1024) hi[i] = t.hi[i];
    for (int i = threadIdx.x; i <= m; i += 1024) hist[i] = 0;
    __syncthreads();
    int top = 1;  // largest power of two <= m
    while (2 * top <= m) top <<= 1;
    const int64_t stride = (int64_t)gridDim.x * 1024;
    for (int64_t i0 = (int64_t)blockIdx.x * 1024 + threadIdx.x; i0 < n_ref; i0 += 4 * stride) {
        uint32_t r[4];
        int p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            r[u] = i0 + u * stride < n_ref ? (uint32_t)(ref[i0 + u * stride] >> 32) : 0u;
            p[u] = 0;  // queries hi[0 .. p-1] are at or below the reference
        }
        for (int s = top; s > 0; s >>= 1)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p[u] + s <= m && hi[p[u] + s - 1] <= r[u]) p[u] += s;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * stride < n_ref && p[u]) atomicAdd(&hist[p[u]], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= m; i += 1024)
        if (hist[i]) atomicAdd(&t.hist[i], (unsigned long long)hist[i]);
}

// count of the query at sorted place i = references with more than i queries at or below them.
__global__ __launch_bounds__(1024) void k_rank_finish(const RankTile *tiles, int64_t n_q, int64_t *__restrict__ count,
                                                      float *__restrict__ fap, double n_div)
{
    constexpr int kPer = kRankTile / 1024;
    __shared__ unsigned long long wsum[16];
    const RankTile &t = tiles[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * kRankTile;
    const int m = (int)(n_q - base < kRankTile ? n_q - base : kRankTile);
    // thread x takes places from the top down: m - 1 - kPer x - j
    unsigned long long v[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = m - 1 - kPer * (int)threadIdx.x - j;
        v[j] = i >= 0 ? t.hist[i + 1] : 0;
        sum += v[j];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    unsigned long long incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    unsigned long long run = incl - sum;
    for (int w = 0; w < wv; ++w) run += wsum[w];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = m - 1 - kPer * (int)threadIdx.x - j;
        if (i < 0) break;
        run += v[j];
        const int64_t e = base + t.pos[i];
        if (count) count[e] = (int64_t)run;
        if (fap) fap[e] = (float)((double)(int64_t)run / n_div);
    }
}

}  // namespace stt
