// The wave-per-template delay-grid scorer, compiled to gfx950 LLVM IR by test_wave_exchange_ir.py.
#include <hip/hip_runtime.h>

#include "stt.h"

#include "kernels.hpp"

template __global__ void stt::k_score_md_wave<false, true, stt::kMapPol>(MapP, GenP, const Trk *, uint64_t, int64_t,
                                                                        int32_t, int32_t, int32_t, int32_t, int32_t,
                                                                        int32_t, float *, int32_t *, uint64_t *);
