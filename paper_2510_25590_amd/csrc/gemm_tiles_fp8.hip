// The E4M3 tiles of the two-group GEMM, by kernel (see kTilesFp8 in gemm.hip).
#include "gemm_launch.h"

int rg_gemm_tile_fp8(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE(42, launch_pp_fp8, 4, 2)
    RG_TILE(62, launch_pp_fp8, 6, 2)
    RG_TILE(82, launch_pp_fp8, 8, 2)
    RG_TILE(44, launch_pp_fp8, 4, 4)
    RG_TILE(54, launch_pp8, 5)
    RG_TILE(64, launch_pp8, 6)
    RG_TILE(74, launch_pp8, 7)
    RG_TILE(84, launch_pp8, 8)
    RG_TILE(222, launch_kg8, 2, 2, 2)
    RG_TILE(224, launch_kg8, 2, 4, 2)
    RG_TILE(274, launch_kg8, 7, 4, 2)
    RG_TILE(426, launch_kg8, 2, 6, 4)
    RG_TILE(446, launch_kg8, 4, 6, 4)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
