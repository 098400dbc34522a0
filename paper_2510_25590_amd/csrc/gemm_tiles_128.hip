// The 64- and 128-column tiles of the two-group GEMM.
#include "gemm_launch.h"

int rg_gemm_tile_128(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE(222, launch_kg, 2, 2, 2)
    RG_TILE(224, launch_kg, 2, 4, 2)
    RG_TILE(242, launch_kg, 4, 2, 2)
    RG_TILE(244, launch_kg, 4, 4, 2)
    RG_TILE(274, launch_kg, 7, 4, 2)
    RG_TILE(284, launch_kg, 8, 4, 2)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
