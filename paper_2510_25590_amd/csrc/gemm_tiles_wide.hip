// The 256-column tiles of the two-group GEMM.
#include "gemm_launch.h"

int rg_gemm_tile_wide(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE(44, launch_pp, 4, 4)
    RG_TILE(64, launch_pp, 6, 4)
    RG_TILE(74, launch_pp, 7, 4)
    RG_TILE(84, launch_pp, 8, 4)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
