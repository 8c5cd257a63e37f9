// Device helpers shared by the network's kernels (mlp.hip, mlp_train.hip).
#pragma once
#include "common.h"

// FP32 to half, the FP32 value rounded first: the empty asm keeps the
// compiler from fusing the multiply or add that produced x and the
// conversion into one mixed-precision FMA (a single rounding from the exact
// result), so every half is the nearest half to an FP32 number, in the
// training kernels and in fused inference alike.
__device__ __forceinline__ _Float16 half_of(float x)
{
    asm volatile("" : "+v"(x));
    return (_Float16)x;
}
