// The 192-column tiles of the two-group GEMM whose groups take the two halves of every K-step.
#include "gemm_launch.h"

int rg_gemm_tile_kg(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE(266, launch_kg, 6, 6, 2)
    RG_TILE(276, launch_kg, 7, 6, 2)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
