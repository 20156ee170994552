// The smooth statistic of an FP32 map, compiled to gfx950 assembly by test_smooth_isa.py.
#include <hip/hip_runtime.h>

#include "stt.h"

#include "kernels.hpp"

template __global__ void stt::k_smooth_grad<stt::kMapF32>(MapP, const float *, const int32_t *, int32_t, float *, float *);
