// Launch of one instantiation of the two-group GEMM kernels.
#pragma once
#include "gemm_pp.h"
#include "gemm_tiles.h"

namespace {

template <typename T, typename Kernel>
int launch_tile(regione_ctx* ctx, Kernel kernel, std::atomic<uint64_t>& granted, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    const int m_tiles = (m + T::ROWS - 1) / T::ROWS, n_tiles = (n + T::COLS - 1) / T::COLS;
    const int tiles = m_tiles * n_tiles;
    const int steps = k / 64, per = (steps + splits - 1) / splits;
    const int used_splits = (steps + per - 1) / per;
    if (used_splits > 1 && (static_cast<size_t>(used_splits) * tiles * T::PART_FLOATS * sizeof(float) > ctx->gemm_part_bytes || tiles > kMaxSplitTiles))
        RG_FAIL(REGIONE_ERR_WORKSPACE, "gemm: %d K-splits of a %d x %d result exceed the workspace", used_splits, m, n);
    // many row tiles: groups of four (the workgroups that run at a time on an XCD then share weight and activation lines in
    // its L2: 2-7 % on the 8704-row GEMMs against all row tiles of a column tile in a row); few row tiles: one group
    const int group_rows = m_tiles > 8 ? 4 : m_tiles;
    if (int rc = rg_grant_lds(ctx, reinterpret_cast<const void*>(kernel), granted, T::LDS_BYTES)) return rc;
    const int units_per_xcd = (tiles * used_splits + 7) / 8;
    hipLaunchKernelGGL(kernel, dim3(units_per_xcd * 8), dim3(T::THREADS), T::LDS_BYTES, ctx->stream,
                       a, lda, wp, m, n, k, m_tiles, n_tiles, units_per_xcd, group_rows, used_splits, per, ctx->gemm_part, ctx->gemm_arrived, ep);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
template <int RF, int CF, int KIND, bool FP8>
int launch_pp_any(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    static std::atomic<uint64_t> granted{0};
    return launch_tile<PpTile<RF, CF>>(ctx, gemm_pp_kernel<RF, CF, KIND, FP8>, granted, a, lda, wp, m, n, k, splits, ep);
}
template <int RF, int CF, int KIND>
int launch_pp(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    return launch_pp_any<RF, CF, KIND, false>(ctx, a, lda, wp, m, n, k, splits, ep);
}
template <int RF, int CF, int KIND>
int launch_pp_fp8(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    return launch_pp_any<RF, CF, KIND, true>(ctx, a, lda, wp, m, n, k, splits, ep);
}
template <int RF, int CF, int WM, int KIND>
int launch_kg(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    static std::atomic<uint64_t> granted{0};
    return launch_tile<KgTile<RF, CF, WM>>(ctx, gemm_kg_kernel<RF, CF, WM, KIND>, granted, a, lda, wp, m, n, k, splits, ep);
}

template <int RF, int CF, int WM, int KIND>
int launch_kg8(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    static std::atomic<uint64_t> granted{0};
    return launch_tile<Kg8Tile<RF, CF, WM>>(ctx, gemm_kg8_kernel<RF, CF, WM, KIND>, granted, a, lda, wp, m, n, k, splits, ep);
}
template <int RF, int KIND>
int launch_pp8(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    static std::atomic<uint64_t> granted{0};
    return launch_tile<Pp8Tile<RF>>(ctx, gemm_pp8_kernel<RF, KIND>, granted, a, lda, wp, m, n, k, splits, ep);
}

}  // namespace

// One entry of a list of tiles: the launch of tile CODE through LAUNCH<tile parameters, epilogue kind>.  The bf16 tiles also finish the
// velocity head.
#define RG_TILE_FP8(CODE, LAUNCH, ...)                                                                          \
    if (tile == CODE) {                                                                                         \
        if (ep.kind == EPI_QKV) return LAUNCH<__VA_ARGS__, EPI_QKV>(ctx, a, lda, wp, m, n, k, splits, ep);      \
        if (ep.kind == EPI_RESID) return LAUNCH<__VA_ARGS__, EPI_RESID>(ctx, a, lda, wp, m, n, k, splits, ep);  \
        return LAUNCH<__VA_ARGS__, EPI_PLAIN>(ctx, a, lda, wp, m, n, k, splits, ep);                            \
    }
#define RG_TILE(CODE, LAUNCH, ...)                                                                              \
    if (tile == CODE && ep.kind == EPI_VELOCITY) return LAUNCH<__VA_ARGS__, EPI_VELOCITY>(ctx, a, lda, wp, m, n, k, splits, ep); \
    RG_TILE_FP8(CODE, LAUNCH, __VA_ARGS__)
