// Products of few rows, and results of at most 64 columns (the velocity head): launches that are chains of memory latencies rather than arithmetic.
//
// A workgroup owns 16 rows x 32 or 64 columns; its eight waves split K, request all their fragments (activation rows as they lie, the packed
// weights as they lie) before the first MFMA, and meet in LDS, where the sums are formed in wave order.  16x16x32 MFMAs with the weights as the
// first operand, as in the tile kernels, so that a lane holds eight consecutive columns of a row and their epilogue serves here too.
// A product that follows a LayerNorm takes the rows before it: the waves normalise the tile's rows into LDS while the weights are on their way, one
// launch and one trip through memory less.
// Which products come here, and what they took before: small_columns (gemm.hip).  In a block of width 256 and 36 rows the launch of a LayerNorm and that of
// its product took 3.4 + 5.4 us, one launch now 3.7; two such blocks with everything around them 85 -> 62 us.
#pragma once
#include "gemm_epilogue.h"
#include "layernorm_row.h"

namespace {

constexpr int kSmallWaves = 8, kSmallRows = 16;
constexpr int kMergePieces = 4;          // pieces per thread in flight
constexpr int kLnColumns = 1024;         // longest row that is normalised here
enum { LN_NONE = 0, LN_BF16 = 1, LN_F32 = 2 };

template <int CF> struct SmallTile {
    static constexpr int CHUNK = CF == 2 ? 12 : 6;              // K-steps of 32 whose loads are in flight together
    static constexpr unsigned SUM_BYTES = kSmallWaves * CF * 1024u;  // the waves' partial tiles
};
__host__ __device__ constexpr unsigned ln_row_bytes(int k) { return static_cast<unsigned>(k) * 2u + 16u; }   // 16 bytes on: the rows of a fragment start in different banks
// The partial tiles take the place of the normalised rows, which all waves have read by then.
template <int CF> constexpr unsigned small_lds_bytes(bool ln, int k) {
    const unsigned rows = ln ? kSmallRows * ln_row_bytes(k) : 0u;
    return rows > SmallTile<CF>::SUM_BYTES ? rows : SmallTile<CF>::SUM_BYTES;
}
static_assert(small_lds_bytes<4>(true, kLnColumns) <= 65536u, "what a launch may ask for without hipFuncSetAttribute");

template <int CF, int KIND, int LN>
__device__ __forceinline__ void gemm_small_tile(unsigned char* lds, int tile_y, const void* __restrict__ A, int lda, const bf16_t* __restrict__ Wp, int M, int N, int K,
                                                const float* __restrict__ shift, const float* __restrict__ scale, const GemmEpilogue& ep) {
    constexpr int CHUNK = SmallTile<CF>::CHUNK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int n0 = blockIdx.x * (16 * CF), m0 = tile_y * kSmallRows;
    const int steps = K >> 5, per = (steps + kSmallWaves - 1) / kSmallWaves;
    const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;

    // weight fragment 2 b + jl of a lane: column 8*(l16/4) + 4*jl + l16%4 of the tile's block b (see gemm_epilogue16)
    const int n_blocks = (N + 31) >> 5;
    const bf16_t* wp[CF / 2];
#pragma unroll
    for (int b = 0; b < CF / 2; ++b) {
        int nb = (n0 >> 5) + b;
        nb = nb < n_blocks ? nb : n_blocks - 1;                 // blocks past N repeat the last one; their sums are not stored
        wp[b] = Wp + ((static_cast<int64_t>(nb) * (K >> 4) + (quad >> 1)) * 64 + (quad & 1) * 32 + 8 * (l16 >> 2) + (l16 & 3)) * 8;
    }
    int row = m0 + l16;
    row = row < M ? row : M - 1;                                // rows past the end repeat the last one
    const bf16_t* ap = LN == LN_NONE ? static_cast<const bf16_t*>(A) + static_cast<int64_t>(row) * lda + 8 * quad : nullptr;
    const unsigned a_lds = static_cast<unsigned>(l16) * ln_row_bytes(K) + 16u * quad;

    // The launch is a chain of trips to memory: what the epilogue reads is requested first, by the waves that finish the tile (wave b block b of 32 columns)
    const int fin_col = n0 + 32 * wave + 8 * quad;
    const bool finishes = wave < CF / 2, whole = (ep.vec_ok || KIND != EPI_QKV) && fin_col + 8 <= N;
    EpiColumns<KIND, false> fin_cols;
    EpiRow<KIND, false> fin_row;
    Raw8 fin_raw;
    if (finishes && whole) {
        fin_row.load(ep, row);
        fin_cols.load(ep, fin_col);
        if (epi_reads<KIND>()) fin_raw = ep.vec_ok ? epi_load8<KIND, true>(ep, row, fin_col) : epi_load8<KIND, false>(ep, row, fin_col);
    }

    f32x4 acc[CF];
#pragma unroll
    for (int j = 0; j < CF; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[CHUNK], w[CHUNK][CF];
    auto load_w = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CHUNK; ++i)
            if (base + i < s1) {
#pragma unroll
                for (int j = 0; j < CF; ++j) w[i][j] = *reinterpret_cast<const bf16x8*>(wp[j >> 1] + static_cast<int64_t>(base + i) * 1024 + (j & 1) * 32);
            }
    };
    auto load_a = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CHUNK; ++i)
            if (base + i < s1) {
                if (LN == LN_NONE) a[i] = *reinterpret_cast<const bf16x8*>(ap + (base + i) * 32);
                else a[i] = *reinterpret_cast<const bf16x8*>(lds + a_lds + static_cast<unsigned>(base + i) * 64u);
            }
    };
    if (LN != LN_NONE) {
        load_w(s0);
#pragma unroll
        for (int r = 0; r < kSmallRows / kSmallWaves; ++r) {
            const int lr = wave * (kSmallRows / kSmallWaves) + r;
            int hr = m0 + lr;
            hr = hr < M ? hr : M - 1;
            unsigned char* to = lds + static_cast<unsigned>(lr) * ln_row_bytes(K);
            auto put = [&](int g, const float (&o)[8]) { st8<bf16_t>(reinterpret_cast<bf16_t*>(to + g * 16), o); };
            if (LN == LN_BF16) layernorm_row<bf16_t, kLnColumns / 512>(static_cast<const bf16_t*>(A) + static_cast<int64_t>(hr) * lda, K, shift, scale, put);
            else layernorm_row<float, kLnColumns / 512>(static_cast<const float*>(A) + static_cast<int64_t>(hr) * lda, K, shift, scale, put);
        }
        __syncthreads();
    }
    for (int base = s0; base < s1; base += CHUNK) {
        if (LN == LN_NONE || base > s0) load_w(base);
        load_a(base);
#pragma unroll
        for (int i = 0; i < CHUNK; ++i)
            if (base + i < s1) {
#pragma unroll
                for (int j = 0; j < CF; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][j], a[i], acc[j], 0, 0, 0);
            }
    }
    if (LN != LN_NONE) __syncthreads();                         // the rows have been read
    f32x4* sums = reinterpret_cast<f32x4*>(lds) + lane;
#pragma unroll
    for (int j = 0; j < CF; ++j) sums[(wave * CF + j) * 64] = acc[j];
    __syncthreads();
    if (!finishes) return;
    f32x4 sum[2];
#pragma unroll
    for (int jl = 0; jl < 2; ++jl) {
        sum[jl] = sums[(2 * wave + jl) * 64];
#pragma unroll
        for (int v = 1; v < kSmallWaves; ++v) sum[jl] += sums[(v * CF + 2 * wave + jl) * 64];
    }
    if (m0 + l16 >= M || fin_col >= N) return;
    if (!whole) epilogue_ragged<KIND, false>(ep, row, fin_col, N, sum[0], sum[1]);
    else if (ep.vec_ok) epilogue_store8<KIND, false, true>(ep, row, fin_col, sum[0], sum[1], fin_cols, fin_row, fin_raw);
    else epilogue_store8<KIND, false, false>(ep, row, fin_col, sum[0], sum[1], fin_cols, fin_row, fin_raw);
}

template <int CF, int KIND, int LN>
__global__ void __launch_bounds__(kSmallWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
gemm_small_kernel(const void* __restrict__ A, int lda, const bf16_t* __restrict__ Wp, int M, int N, int K,
                  const float* __restrict__ shift, const float* __restrict__ scale, GemmEpilogue ep) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    gemm_small_tile<CF, KIND, LN>(lds, blockIdx.y, A, lda, Wp, M, N, K, shift, scale, ep);
}
// Two products of one shape but for their rows.  Either is a few us of weights' latency that fills part of the chip, behind a gap between two launches that is as long; tiles_p: the
// first product's row tiles.  A block (attention included), us, two launches -> one: hidden 256, 16 + 36 rows 36.8 -> 21.9, 64 + 256 39.3 -> 28.9, 512 + 512 54 -> 47; hidden
// 1024, 16 + 64 rows 59 -> 42; hidden 3072 (the two residual products at most), 16 + 36 rows 153 -> 147.
struct SmallProduct { const void* a; int lda; const bf16_t* w; int m; const float* shift; const float* scale; GemmEpilogue ep; };
template <int CF, int KIND, int LN>
__global__ void __launch_bounds__(kSmallWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
gemm_small_pair_kernel(SmallProduct p, SmallProduct q, int tiles_p, int N, int K) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if (static_cast<int>(blockIdx.y) < tiles_p) gemm_small_tile<CF, KIND, LN>(lds, blockIdx.y, p.a, p.lda, p.w, p.m, N, K, p.shift, p.scale, p.ep);
    else gemm_small_tile<CF, KIND, LN>(lds, blockIdx.y - tiles_p, q.a, q.lda, q.w, q.m, N, K, q.shift, q.scale, q.ep);
}

// The velocity head and, in workgroups of their own behind its tiles, the merge of the hidden rows (dst[index[i]] = src[i] in 16-byte pieces): neither reads what the
// other writes, and both are shorter than what lies between two launches.  820 rows of 3072 values, kernel trace: 8.8 + 5.0 -> 10.5 us.
template <int CF>
__global__ void __launch_bounds__(kSmallWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
gemm_small_merge_kernel(const void* __restrict__ A, int lda, const bf16_t* __restrict__ Wp, int M, int N, int K, GemmEpilogue ep, int head_tiles_y, RowMerge merge) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if (static_cast<int>(blockIdx.y) < head_tiles_y) {
        gemm_small_tile<CF, EPI_VELOCITY, LN_NONE>(lds, blockIdx.y, A, lda, Wp, M, N, K, nullptr, nullptr, ep);
        return;
    }
    const unsigned wg = (blockIdx.y - head_tiles_y) * gridDim.x + blockIdx.x, stride = (gridDim.y - head_tiles_y) * gridDim.x * (kSmallWaves * 64);
    const unsigned total = static_cast<unsigned>(merge.rows) * static_cast<unsigned>(merge.pieces);
    for (unsigned u0 = wg * (kSmallWaves * 64) + threadIdx.x; u0 < total; u0 += kMergePieces * stride) {
        u32x4 v[kMergePieces];
        int64_t to[kMergePieces];
#pragma unroll
        for (int i = 0; i < kMergePieces; ++i) {
            const unsigned u = u0 + i * stride;
            if (u >= total) continue;
            const unsigned row = u / static_cast<unsigned>(merge.pieces);
            to[i] = static_cast<int64_t>(merge.index[row]) * merge.pieces + (u - row * merge.pieces);
            v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(merge.src) + u);
        }
#pragma unroll
        for (int i = 0; i < kMergePieces; ++i)
            if (u0 + i * stride < total) __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4*>(merge.dst) + to[i]);
    }
}

template <int CF>
int launch_small_merge(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, const GemmEpilogue& ep, const RowMerge& merge) {
    const unsigned x = static_cast<unsigned>((n + 16 * CF - 1) / (16 * CF)), y = static_cast<unsigned>((m + kSmallRows - 1) / kSmallRows);
    const unsigned per = kSmallWaves * 64 * kMergePieces;
    unsigned wgs = (static_cast<unsigned>(merge.rows) * static_cast<unsigned>(merge.pieces) + per - 1) / per;
    wgs = wgs < 2048 ? wgs : 2048;
    hipLaunchKernelGGL((gemm_small_merge_kernel<CF>), dim3(x, y + (wgs + x - 1) / x), dim3(kSmallWaves * 64), small_lds_bytes<CF>(false, k), ctx->stream,
                       a, lda, wp, m, n, k, ep, static_cast<int>(y), merge);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

template <int CF, int KIND, int LN>
int launch_small(regione_ctx* ctx, const void* a, int lda, const bf16_t* wp, int m, int n, int k, const float* shift, const float* scale, const GemmEpilogue& ep) {
    hipLaunchKernelGGL((gemm_small_kernel<CF, KIND, LN>), dim3(static_cast<unsigned>((n + 16 * CF - 1) / (16 * CF)), static_cast<unsigned>((m + kSmallRows - 1) / kSmallRows)), dim3(kSmallWaves * 64),
                       small_lds_bytes<CF>(LN != LN_NONE, k), ctx->stream, a, lda, wp, m, n, k, shift, scale, ep);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
template <int CF, int LN>
int launch_small_kind(regione_ctx* ctx, const void* a, int lda, const bf16_t* wp, int m, int n, int k, const float* shift, const float* scale, const GemmEpilogue& ep) {
    if (ep.kind == EPI_QKV) return launch_small<CF, EPI_QKV, LN>(ctx, a, lda, wp, m, n, k, shift, scale, ep);
    if (ep.kind == EPI_PLAIN) return launch_small<CF, EPI_PLAIN, LN>(ctx, a, lda, wp, m, n, k, shift, scale, ep);
    if constexpr (LN == LN_NONE) {
        if (ep.kind == EPI_VELOCITY) return launch_small<CF, EPI_VELOCITY, LN>(ctx, a, lda, wp, m, n, k, shift, scale, ep);
        return launch_small<CF, EPI_RESID, LN>(ctx, a, lda, wp, m, n, k, shift, scale, ep);
    }
    RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_small: epilogue kind %d", ep.kind);
}

inline SmallProduct small_product(const GemmCall& c, const GemmEpilogue& ep) { return {c.a, c.lda, static_cast<const bf16_t*>(c.w), c.m, c.shift, c.scale, ep}; }
template <int CF, int KIND, int LN>
int launch_small_pair(regione_ctx* ctx, const GemmCall& a, const GemmCall& b, const GemmEpilogue& ep_a, const GemmEpilogue& ep_b) {
    const int ya = (a.m + kSmallRows - 1) / kSmallRows, yb = (b.m + kSmallRows - 1) / kSmallRows;
    hipLaunchKernelGGL((gemm_small_pair_kernel<CF, KIND, LN>), dim3(static_cast<unsigned>((a.n + 16 * CF - 1) / (16 * CF)), static_cast<unsigned>(ya + yb)), dim3(kSmallWaves * 64),
                       small_lds_bytes<CF>(LN != LN_NONE, a.k), ctx->stream, small_product(a, ep_a), small_product(b, ep_b), ya, a.n, a.k);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
template <int CF>
int launch_small_pair_kind(regione_ctx* ctx, const GemmCall& a, const GemmCall& b, const GemmEpilogue& ep_a, const GemmEpilogue& ep_b) {
    const int ln = a.norm ? (a.a_f32 ? LN_F32 : LN_BF16) : LN_NONE;
    if (a.ep.kind == EPI_RESID) return launch_small_pair<CF, EPI_RESID, LN_NONE>(ctx, a, b, ep_a, ep_b);
#define RG_PAIR(LN) return a.ep.kind == EPI_QKV ? launch_small_pair<CF, EPI_QKV, LN>(ctx, a, b, ep_a, ep_b) : launch_small_pair<CF, EPI_PLAIN, LN>(ctx, a, b, ep_a, ep_b)
    if (ln == LN_BF16) RG_PAIR(LN_BF16);
    if (ln == LN_F32) RG_PAIR(LN_F32);
    RG_PAIR(LN_NONE);
#undef RG_PAIR
}

// tiles of 16 rows x `columns` (32 or 64); every epilogue kind
int gemm_small(regione_ctx* ctx, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, int columns, const GemmEpilogue& ep) {
    if ((m + kSmallRows - 1) / kSmallRows > 65535) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm_small: %d rows", m);
    return columns == 32 ? launch_small_kind<2, LN_NONE>(ctx, a, lda, wp, m, n, k, nullptr, nullptr, ep) : launch_small_kind<4, LN_NONE>(ctx, a, lda, wp, m, n, k, nullptr, nullptr, ep);
}

// the product of layernorm_mod(h), rows h of k <= 1024 values (bf16 or float32, 16-byte aligned like shift and scale); QKV and plain epilogues
int gemm_small_ln(regione_ctx* ctx, const void* h, int h_f32, const float* shift, const float* scale, const bf16_t* wp, int m, int n, int k, int columns, const GemmEpilogue& ep) {
    if (k > kLnColumns || (m + kSmallRows - 1) / kSmallRows > 65535) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm_small_ln: %d rows of %d", m, k);
    if (h_f32) return columns == 32 ? launch_small_kind<2, LN_F32>(ctx, h, k, wp, m, n, k, shift, scale, ep) : launch_small_kind<4, LN_F32>(ctx, h, k, wp, m, n, k, shift, scale, ep);
    return columns == 32 ? launch_small_kind<2, LN_BF16>(ctx, h, k, wp, m, n, k, shift, scale, ep) : launch_small_kind<4, LN_BF16>(ctx, h, k, wp, m, n, k, shift, scale, ep);
}

}  // namespace
