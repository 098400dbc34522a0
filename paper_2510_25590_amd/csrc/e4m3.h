// E4M3 codes of float32 values: clamp(x * mult, +-448), round to nearest even (v_cvt_pk_fp8_f32).
#pragma once
#include "common.h"

constexpr float kE4M3Max = 448.0f;

__device__ __forceinline__ unsigned fp8_codes4(const float* x, float mult) {
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = __builtin_fminf(__builtin_fmaxf(x[e] * mult, -kE4M3Max), kE4M3Max);
    unsigned codes = 0;
    codes = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], codes, false);
    return __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], codes, true);
}
__device__ __forceinline__ uint2 fp8_codes(const float (&x)[8], float mult) { return make_uint2(fp8_codes4(x, mult), fp8_codes4(x + 4, mult)); }
