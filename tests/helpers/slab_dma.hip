// Kernels with the LDS-DMA staging of the slab scorers, compiled to gfx950 assembly by
// test_slab_dma_isa.py: the staging loop alone, from a scalar base address and from one that
// arrives in a vector register, and a whole scorer.
#include <hip/hip_runtime.h>

#include "stt.h"

#include "kernels.hpp"

using namespace stt;

__global__ void stage(MapP m, int c0, int ncol)
{
    extern __shared__ float2 slab[];
    SlabDma<4>(m, 8).issue(c0, ncol, lds_addr(slab));
    slab_sync();
}

__global__ void stage_loaded(const MapP *maps, const int *cols)
{
    extern __shared__ float2 slab[];
    const int i = blockIdx.x & cols[0];
    SlabDma<4>(maps[i], 8).issue(cols[i + 1], cols[i + 2], lds_addr(slab));
    slab_sync();
}

template __global__ void stt::k_score_slab<1024, 2, true, kMapPol, 4>(MapP, GenP, const Trk *, const uint32_t *, uint64_t,
                                                                      int64_t, int, int32_t, float *, uint64_t *);
