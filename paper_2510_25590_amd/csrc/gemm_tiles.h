// The tile shapes of the two-group GEMM kernels (gemm_pp.h), each set in a translation unit of its own.  A tile's code is
// 10*RF + CF for gemm_pp_kernel and gemm_pp8_kernel and 100*WM + 10*RF + CF for gemm_kg_kernel and gemm_kg8_kernel; ep.kind picks the
// epilogue.
#pragma once
#include "common.h"

int rg_gemm_tile_wide(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep);
int rg_gemm_tile_128(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep);
int rg_gemm_tile_96(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep);
int rg_gemm_tile_kg(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep);
// E4M3 operands; lda and k count pairs of values
int rg_gemm_tile_fp8(regione_ctx* ctx, int tile, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int splits, const GemmEpilogue& ep);
