// The E4M3 tiles of the two-group GEMM: shapes whose phase holds a whole K-step, which the 8-bit instruction takes at once.
#include "gemm_launch.h"

int rg_gemm_tile_fp8(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
#define RG_TILE(CODE, ...)                                                                                                  \
    if (tile == CODE) {                                                                                                     \
        if (ep.kind == EPI_QKV) return launch_pp<__VA_ARGS__, EPI_QKV, true>(ctx, a, lda, wp, m, n, k, splits, ep);     \
        if (ep.kind == EPI_RESID) return launch_pp<__VA_ARGS__, EPI_RESID, true>(ctx, a, lda, wp, m, n, k, splits, ep); \
        return launch_pp<__VA_ARGS__, EPI_PLAIN, true>(ctx, a, lda, wp, m, n, k, splits, ep);                           \
    }
    RG_TILE(42, 4, 2)
    RG_TILE(62, 6, 2)
    RG_TILE(82, 8, 2)
    RG_TILE(44, 4, 4)
#undef RG_TILE
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
