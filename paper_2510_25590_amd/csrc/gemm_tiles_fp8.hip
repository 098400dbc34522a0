// The E4M3 tiles of the two-group GEMM, by kernel (see kTilesFp8 in gemm.hip).
#include "gemm_launch.h"

int rg_gemm_tile_fp8(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep) {
    RG_TILE_FP8(42, launch_pp_fp8, 4, 2)
    RG_TILE_FP8(62, launch_pp_fp8, 6, 2)
    RG_TILE_FP8(82, launch_pp_fp8, 8, 2)
    RG_TILE_FP8(44, launch_pp_fp8, 4, 4)
    RG_TILE_FP8(54, launch_pp8, 5)
    RG_TILE_FP8(64, launch_pp8, 6)
    RG_TILE_FP8(74, launch_pp8, 7)
    RG_TILE_FP8(84, launch_pp8, 8)
    RG_TILE_FP8(222, launch_kg8, 2, 2, 2)
    RG_TILE_FP8(224, launch_kg8, 2, 4, 2)
    RG_TILE_FP8(274, launch_kg8, 7, 4, 2)
    RG_TILE_FP8(426, launch_kg8, 2, 6, 4)
    RG_TILE_FP8(446, launch_kg8, 4, 6, 4)
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: no tile %d here", tile);
}
