// LayerNorm over one row (no affine, biased variance, eps 1e-6) with the modulation y*(1+scale)+shift, by one wave: the row is
// read once with 16-byte loads and kept in registers (at most 64 lanes * 8 * MAXV elements, a multiple of 8), two-pass mean/variance.
#pragma once
#include "common.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 ln_bf16x8;
typedef __attribute__((ext_vector_type(4))) float ln_f32x4;

template <typename T> __device__ __forceinline__ void ld8(const T* p, float (&v)[8]);
template <> __device__ __forceinline__ void ld8<bf16_t>(const bf16_t* p, float (&v)[8]) {
    const ln_bf16x8 x = *reinterpret_cast<const ln_bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<float>(x[e]);
}
template <> __device__ __forceinline__ void ld8<float>(const float* p, float (&v)[8]) {
    const ln_f32x4 a = *reinterpret_cast<const ln_f32x4*>(p), b = *reinterpret_cast<const ln_f32x4*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}

// put(group, values): takes the eight results, as float32, of columns 8*group..8*group+7
template <typename T, int MAXV, typename Put>
__device__ __forceinline__ void layernorm_row(const T* hr, int hidden, const float* shift, const float* scale, Put put) {
    const int lane = threadIdx.x & 63;
    const int groups = hidden >> 3;          // 8-element groups in a row; lane owns groups lane, lane + 64, ...
    float x[MAXV][8];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int g = lane + 64 * i;
        if (g < groups) {
            ld8<T>(hr + g * 8, x[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += x[i][e];
        }
    }
    // the modulation vectors are requested now, so that they arrive while the two reductions run
    float sc[MAXV][8], sh[MAXV][8];
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int g = lane + 64 * i;
        if (g < groups) {
            if (scale) ld8<float>(scale + g * 8, sc[i]);
            if (shift) ld8<float>(shift + g * 8, sh[i]);
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
    const float mean = sum / hidden;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        if (lane + 64 * i < groups) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float d = x[i][e] - mean; sq += d * d; }
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sq += __shfl_xor(sq, m, 64);
    const float rstd = rsqrtf(sq / hidden + 1e-6f);
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int g = lane + 64 * i;
        if (g < groups) {
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float y = (x[i][e] - mean) * rstd;
                y = y * (1.f + (scale ? sc[i][e] : 0.f)) + (shift ? sh[i][e] : 0.f);
                o[e] = y;
            }
            put(g, o);
        }
    }
}

template <typename T> __device__ __forceinline__ void st8(T* p, const float (&v)[8]);
template <> __device__ __forceinline__ void st8<bf16_t>(bf16_t* p, const float (&v)[8]) {
    ln_bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(v[e]);
    *reinterpret_cast<ln_bf16x8*>(p) = o;
}
template <> __device__ __forceinline__ void st8<float>(float* p, const float (&v)[8]) {
    *reinterpret_cast<ln_f32x4*>(p) = ln_f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<ln_f32x4*>(p + 4) = ln_f32x4{v[4], v[5], v[6], v[7]};
}

}  // namespace
