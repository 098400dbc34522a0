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

template <int CTRL, int BANKS> __device__ __forceinline__ unsigned ln_dpp(unsigned old, unsigned x) { return __builtin_amdgcn_update_dpp(old, x, CTRL, 0xf, BANKS, false); }
// op over the wave, the same bits in every lane: partners l ^ 32, 16, 8, 4, 2, 1 in this order, as a butterfly of shuffles takes them, but through the vector ALU instead of LDS
// (gfx950's half and row swaps: two copies of x become the value of the one and of the other half everywhere, elements copied out before the casts; then DPP:
// row_ror 8, lanes + 4 and - 4 by banks of four, and two permutations of quads).  The codes of an E4M3 block hang on every bit of these sums.
template <typename Op> __device__ __forceinline__ float wave_reduce(float x, Op op) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const unsigned a0 = a[0], a1 = a[1];
    x = op(__uint_as_float(a0), __uint_as_float(a1));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const unsigned b0 = b[0], b1 = b[1];
    x = op(__uint_as_float(b0), __uint_as_float(b1));
    unsigned u = __float_as_uint(x);
    x = op(x, __uint_as_float(ln_dpp<0x128, 0xf>(u, u)));
    u = __float_as_uint(x);
    x = op(x, __uint_as_float(ln_dpp<0x114, 0xa>(ln_dpp<0x104, 0x5>(u, u), u)));
    u = __float_as_uint(x);
    x = op(x, __uint_as_float(ln_dpp<0x4e, 0xf>(u, u)));
    u = __float_as_uint(x);
    return op(x, __uint_as_float(ln_dpp<0xb1, 0xf>(u, u)));
}
__device__ __forceinline__ float wave_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return __builtin_fmaxf(a, b); }); }

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
    sum = wave_sum(sum);
    const float mean = sum / hidden;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        if (lane + 64 * i < groups) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float d = x[i][e] - mean; sq += d * d; }
        }
    }
    sq = wave_sum(sq);
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

// ---- a row by several waves
// eight elements as loaded, converted when they are used
template <typename T> struct LnRaw;
template <> struct LnRaw<bf16_t> {
    ln_bf16x8 v;
    __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const ln_bf16x8*>(p); }
    __device__ __forceinline__ void store(bf16_t* p) const { *reinterpret_cast<ln_bf16x8*>(p) = v; }
    __device__ __forceinline__ void values(float (&x)[8]) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = static_cast<float>(v[e]);
    }
};
template <> struct LnRaw<float> {
    ln_f32x4 a, b;
    __device__ __forceinline__ void load(const float* p) { a = *reinterpret_cast<const ln_f32x4*>(p); b = *reinterpret_cast<const ln_f32x4*>(p + 4); }
    __device__ __forceinline__ void store(float* p) const { *reinterpret_cast<ln_f32x4*>(p) = a; *reinterpret_cast<ln_f32x4*>(p + 4) = b; }
    __device__ __forceinline__ void values(float (&x)[8]) const {
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
    }
};

// Rows of more than 1024 and at most 64 * 8 * W values by workgroups of W waves, a group of eight values per lane; a workgroup goes through rows blockIdx.x,
// + gridDim.x, ... with the modulation vectors in registers and the next row on its way.  Each wave forms the mean and the squared deviations of its own part
// (two passes over registers), the parts meet in LDS once: M2 = sum of M2_w + n_w (mean_w - mean)^2.
// A wave for a whole row, as for shorter ones, is a long chain of its own (six rounds of loads, twelve shuffles through LDS) and reads the modulation vectors again for
// every row, twice the bytes of the row itself.
// us, a wave per row -> here, bf16 / float32 rows: 820 x 3072 7.0 / 6.7 -> 5.4 / 5.9, 8704 x 3072 42.5 / 42.4 -> 27.7 / 30.1 (3.9 and 5.3 TB/s; a copy reaches 5.9), 8704 x 1536 23.3 / 24.3 -> 13.8 / 17.4,
// 2048 x 3072 the same.
// put(row, group, values): takes eight results of a live lane; each(row, lane's raw values) before them.
template <typename T, int W, typename Each, typename Put>
__device__ __forceinline__ void layernorm_rows_wide(const T* h, int n, int hidden, const float* shift, const float* scale, float2 (&part)[2][W], Each source, Put put) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = threadIdx.x, groups = hidden >> 3;
    const bool live = g < groups;
    int mine = groups - 64 * wave;                       // groups of this wave
    mine = mine < 0 ? 0 : (mine < 64 ? mine : 64);
    const float count = 8.0f * mine, inv_count = mine > 0 ? 1.0f / count : 0.f;
    float sc[8], sh[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { sc[e] = 0.f; sh[e] = 0.f; }
    LnRaw<T> next;
    int row = blockIdx.x;
    if (live && row < n) next.load(h + source(row) * hidden + g * 8);
    if (live && scale) ld8<float>(scale + g * 8, sc);
    if (live && shift) ld8<float>(shift + g * 8, sh);
#pragma unroll
    for (int e = 0; e < 8; ++e) sc[e] = 1.f + sc[e];
    for (int turn = 0; row < n; row += gridDim.x, turn ^= 1) {
        const LnRaw<T> raw = next;
        const int after = row + static_cast<int>(gridDim.x);
        if (live && after < n) next.load(h + source(after) * hidden + g * 8);
        float x[8];
        raw.values(x);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) { x[e] = live ? x[e] : 0.f; s += x[e]; }
        s = wave_sum(s);
        const float own = s * inv_count;
        float sq = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float d = x[e] - own; sq += d * d; }
        sq = wave_sum(live ? sq : 0.f);
        if (lane == 0) part[turn][wave] = make_float2(s, sq);
        __syncthreads();                                 // the other buffer is written next, and this one only after the next barrier
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) sum += part[turn][w].x;
        const float mean = sum / hidden;
        float m2 = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            int in = groups - 64 * w;
            in = in < 0 ? 0 : (in < 64 ? in : 64);
            const float cnt = 8.0f * in, d = in > 0 ? part[turn][w].x / cnt - mean : 0.f;
            m2 += part[turn][w].y + cnt * d * d;
        }
        const float rstd = rsqrtf(m2 / hidden + 1e-6f);
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (x[e] - mean) * rstd * sc[e] + sh[e];
        put(row, g, live, raw, o);
    }
}
// workgroups of W waves that the chip holds at a time
constexpr int ln_wide_grid(int waves) { return 256 * (32 / waves); }

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
