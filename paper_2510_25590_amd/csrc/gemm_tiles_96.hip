// The 96-column tiles of the two-group GEMM.
#include "gemm_launch.h"

int rg_gemm_tile_96(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE(426, launch_kg, 2, 6, 4)
    RG_TILE(436, launch_kg, 3, 6, 4)
    RG_TILE(446, launch_kg, 4, 6, 4)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
