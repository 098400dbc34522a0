// The 64- and 128-column tiles of the two-group GEMM.
#include "gemm_launch.h"

int rg_gemm_tile_128(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
#define RG_TILE(CODE, ...)                                                                                                  \
    if (tile == CODE) {                                                                                                     \
        if (ep.kind == EPI_QKV) return launch_kg<__VA_ARGS__, EPI_QKV>(ctx, a, lda, wp, m, n, k, splits, ep);     \
        if (ep.kind == EPI_RESID) return launch_kg<__VA_ARGS__, EPI_RESID>(ctx, a, lda, wp, m, n, k, splits, ep); \
        return launch_kg<__VA_ARGS__, EPI_PLAIN>(ctx, a, lda, wp, m, n, k, splits, ep);                           \
    }
    RG_TILE(222, 2, 2, 2)
    RG_TILE(224, 2, 4, 2)
    RG_TILE(242, 4, 2, 2)
    RG_TILE(244, 4, 4, 2)
    RG_TILE(274, 7, 4, 2)
    RG_TILE(284, 8, 4, 2)
#undef RG_TILE
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}

int rg_gemm_tile_velocity(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    return launch_kg<2, 2, 2, EPI_VELOCITY>(ctx, a, lda, wp, m, n, k, splits, ep);
}
