// The 256-column tiles of the two-group GEMM.
#include "gemm_launch.h"

int rg_gemm_tile_wide(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
#define RG_TILE(CODE, ...)                                                                                                  \
    if (tile == CODE) {                                                                                                     \
        if (ep.kind == EPI_QKV) return launch_pp<__VA_ARGS__, EPI_QKV, false>(ctx, a, lda, wp, m, n, k, splits, ep);     \
        if (ep.kind == EPI_RESID) return launch_pp<__VA_ARGS__, EPI_RESID, false>(ctx, a, lda, wp, m, n, k, splits, ep); \
        return launch_pp<__VA_ARGS__, EPI_PLAIN, false>(ctx, a, lda, wp, m, n, k, splits, ep);                           \
    }
    RG_TILE(44, 4, 4)
    RG_TILE(64, 6, 4)
    RG_TILE(74, 7, 4)
    RG_TILE(84, 8, 4)
#undef RG_TILE
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
