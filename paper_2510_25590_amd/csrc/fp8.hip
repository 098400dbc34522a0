// 8-bit floating point (OCP E4M3) variant of the dense projections on the edited rows (section "Region-Aware
// Generation"); an extension, the paper itself computes in the model's precision.  This file: per-row quantisation
// and the entry points; the matrix-core kernel is the 8-bit form of the LDS GEMM in gemm.hip.
#include "common.h"
#include "e4m3.h"
#include "layernorm_row.h"
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

// TPR threads per row (64: four rows per workgroup, 256: one); the row stays in registers between the maximum and the
// conversion (up to 8 16-byte pieces per thread, so 4096 columns per wave and 16384 per workgroup).
//   amax = max |x|;  scale = amax / 448;  code = e4m3(clamp(x * (448 / amax), +-448)), round to nearest even
// (v_cvt_pk_fp8_f32).  The divisions are IEEE float32 divisions, the product a float32 product.
template <int TPR>
__global__ void __launch_bounds__(256)
quantize_rows_fp8_kernel(const bf16_t* __restrict__ x, int64_t rows, int cols, uint8_t* __restrict__ q, float* __restrict__ scale) {
    constexpr int MAXV = 8, RPB = 256 / TPR;
    __shared__ float most[4];
    const int t = threadIdx.x % TPR;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * RPB + threadIdx.x / TPR;
    const bool live_row = row < rows;      // (a workgroup of TPR = 256 has one row, so the barrier below is uniform)
    const int pieces = cols >> 3;
    const bf16x8* src = reinterpret_cast<const bf16x8*>(x + (live_row ? row : 0) * cols);
    bf16x8 v[MAXV];
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int p = i * TPR + t;
        if (live_row && p < pieces) {
            v[i] = src[p];
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = __builtin_fmaxf(amax, __builtin_fabsf(static_cast<float>(v[i][e])));
        }
    }
    amax = wave_max(amax);
    if (TPR == 256) {
        if ((threadIdx.x & 63) == 0) most[threadIdx.x >> 6] = amax;
        __syncthreads();
        amax = __builtin_fmaxf(__builtin_fmaxf(most[0], most[1]), __builtin_fmaxf(most[2], most[3]));
    }
    if (!live_row) return;
    const bool live = amax > 0.f;
    const float mult = live ? kE4M3Max / amax : 1.0f;
    if (t == 0) scale[row] = live ? amax / kE4M3Max : 1.0f;
    uint2* dst = reinterpret_cast<uint2*>(q + row * cols);
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int p = i * TPR + t;
        if (p < pieces) {
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = static_cast<float>(v[i][e]);
            dst[p] = fp8_codes(y, mult);
        }
    }
}

// LayerNorm + modulation (as layernorm_mod_vec_kernel in rows.hip: no affine, biased variance, eps 1e-6, two passes in
// float32, u = y * (1 + scale) + shift) with the row quantisation above applied to its float32 result while the row is
// still in registers: the bf16 rounding of u, its store and the quantiser's load of it fall away.  One wave per row, whatever its
// length: sums in another order, as of several waves, would move an E4M3 block's output by up to 1.3 %, more than the 1e-2 that it is held to from one version to the next (a few
// scales differ in their last bit, then queries by one bf16 rounding, and the quantisations that follow turn that into whole code steps).  A kernel for as many rounds of 512 values
// as the row has, with the modulation vectors requested ahead of the sums; us before -> after, kernel trace, bf16 / float32 rows: 820 x 3072 9.3 / 10.6 -> 6.8 / 8.0.
template <typename T, int MAXV>
__global__ void __launch_bounds__(256)
layernorm_mod_fp8_kernel(const T* __restrict__ h, int n, int hidden, const float* __restrict__ shift, const float* __restrict__ scale,
                         uint8_t* __restrict__ q, float* __restrict__ row_scale) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n) return;
    const T* hr = h + static_cast<int64_t>(row) * hidden;
    const int groups = hidden >> 3;
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
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int g = lane + 64 * i;
        if (g < groups) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float y = (x[i][e] - mean) * rstd;
                y = y * (1.f + (scale ? sc[i][e] : 0.f)) + (shift ? sh[i][e] : 0.f);
                x[i][e] = y;
                amax = __builtin_fmaxf(amax, __builtin_fabsf(y));
            }
        }
    }
    amax = wave_max(amax);
    const bool live = amax > 0.f;
    const float mult = live ? kE4M3Max / amax : 1.0f;
    if (lane == 0) row_scale[row] = live ? amax / kE4M3Max : 1.0f;
    uint2* dst = reinterpret_cast<uint2*>(q + static_cast<int64_t>(row) * hidden);
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int g = lane + 64 * i;
        if (g < groups) {
            dst[g] = fp8_codes(x[i], mult);
        }
    }
}

}  // namespace

int rg_layernorm_mod_fp8(regione_ctx* ctx, const void* h, int h_f32, int n, int hidden, const float* shift, const float* scale,
                         uint8_t* q, float* row_scale) {
    if (n <= 0) return REGIONE_OK;
    if ((hidden & 7) || hidden > 4096 || hidden <= 0) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "layernorm_fp8: hidden=%d (a multiple of 8, at most 4096)", hidden);
    if (!rg_aligned16(h) || !rg_aligned16(q) || (shift && !rg_aligned16(shift)) || (scale && !rg_aligned16(scale)))
        RG_FAIL(REGIONE_ERR_INVALID_ARG, "layernorm_fp8: tensors must be 16-byte aligned");
    ProfScope prof(ctx, REGIONE_PROF_LAYERNORM);
    auto launch = [&](auto* rows) {
        typedef std::remove_const_t<std::remove_pointer_t<decltype(rows)>> T;
#define RG_LN(R) hipLaunchKernelGGL((layernorm_mod_fp8_kernel<T, R>), dim3((n + 3) / 4), dim3(256), 0, ctx->stream, rows, n, hidden, shift, scale, q, row_scale)
        if (hidden <= 1024) RG_LN(2); else if (hidden <= 2048) RG_LN(4); else if (hidden <= 3072) RG_LN(6); else RG_LN(8);
#undef RG_LN
    };
    if (h_f32) launch(static_cast<const float*>(h)); else launch(static_cast<const bf16_t*>(h));
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

extern "C" int regione_quantize_rows_fp8(regione_ctx* ctx, const void* x, int64_t rows, int32_t cols, void* q, float* scale) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "quantize_rows_fp8: null context");
    if (rows < 0 || cols <= 0 || (cols & 7) || cols > 16384) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "quantize_rows_fp8: rows=%lld, cols=%d (a multiple of 8, at most 16384)", (long long)rows, cols);
    if (rows == 0) return REGIONE_OK;
    if (rows > (int64_t(1) << 31)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "quantize_rows_fp8: rows=%lld too many", (long long)rows);
    if (!x || !q || !scale || !rg_aligned16(x) || !rg_aligned16(q)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "quantize_rows_fp8: null or unaligned tensor");
    ProfScope prof(ctx, REGIONE_PROF_ROWS);
    const bf16_t* xs = static_cast<const bf16_t*>(x);
    uint8_t* qs = static_cast<uint8_t*>(q);
    // short rows: a wave per row; long rows (or few of them): a workgroup per row, so that the launch fills the chip
    if (cols <= 2048 || (cols <= 4096 && rows >= 4096))
        hipLaunchKernelGGL(quantize_rows_fp8_kernel<64>, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, ctx->stream, xs, rows, cols, qs, scale);
    else
        hipLaunchKernelGGL(quantize_rows_fp8_kernel<256>, dim3(static_cast<unsigned>(rows)), dim3(256), 0, ctx->stream, xs, rows, cols, qs, scale);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

extern "C" int regione_pack_weight_fp8(regione_ctx* ctx, const void* wq, int32_t n, int32_t k, void* wq_packed) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "pack_weight_fp8: null context");
    if (ctx->f32) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "pack_weight_fp8: the 8-bit projections belong to bf16 contexts");
    if (n <= 0 || k <= 0 || (k % 128)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "pack_weight_fp8: n=%d, k=%d (k must be a multiple of 128)", n, k);
    // the 8-bit layout is the 16-bit one with every pair of codes taken as one element
    return regione_pack_weight(ctx, wq, n, k / 2, wq_packed);
}

extern "C" int regione_linear_fp8(regione_ctx* ctx, const void* xq, const float* x_scale, const void* wq_packed, const float* w_scale,
                                  const float* b_opt, int32_t m, int32_t n, int32_t k, int32_t act, int32_t out_dtype, void* y) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear_fp8: null context");
    if (ctx->f32) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "linear_fp8: the 8-bit projections belong to bf16 contexts");
    if (m < 0 || n <= 0 || k <= 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear_fp8: m=%d n=%d k=%d", m, n, k);
    if (act != REGIONE_ACT_NONE && act != REGIONE_ACT_GELU_TANH) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear_fp8: bad act %d", act);
    if (out_dtype != REGIONE_BF16 && out_dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear_fp8: bad out_dtype %d", out_dtype);
    if (k % 128) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "linear_fp8: k=%d must be a multiple of 128", k);
    if (m == 0) return REGIONE_OK;
    if (!xq || !x_scale || !wq_packed || !w_scale || !y) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear_fp8: null tensor");
    GemmEpilogue ep = {};
    ep.kind = EPI_PLAIN; ep.bias = b_opt; ep.act = act; ep.act_from = 0;
    ep.y = y; ep.ldy = n; ep.y_f32 = out_dtype == REGIONE_FP32;
    ep.row_scale = x_scale; ep.col_scale = w_scale;
    return rg_gemm_fp8(ctx, static_cast<const uint8_t*>(xq), k, static_cast<const uint8_t*>(wq_packed), m, n, k, ep);
}
