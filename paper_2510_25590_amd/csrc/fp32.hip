// The float32 context: dense projections on v_mfma_f32_16x16x4_f32 and attention with the Region-Instruction KV
// cache (Eq.6) with float32 operands, float32 sums and a float32 softmax.  This is the arithmetic of the small
// float32 configuration on which the method's path is first checked against the CPU definition at a tight
// tolerance.  Its launches are a few dozen rows wide, so every kernel here is a chain of memory latencies rather than
// arithmetic: the k elements of a product (the keys of an attention) are dealt to the waves of a workgroup, each wave
// reads its operands from global memory straight into fragments, several loads in flight, and the waves' float32
// partial results meet once in LDS, in wave order.
#include <cmath>
#include <type_traits>
#include "common.h"
#include "layernorm_row.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kThreads = 256;
constexpr int FB = 64;   // rows and columns of a tile of the wide form: four waves, one 32 x 32 block each
constexpr int FK = 16;   // k elements per step of the wide form, and per chunk of the other: one 16-byte load per lane and fragment, four MFMAs

__device__ __forceinline__ float gelu_tanh_exact(float x) {
    return 0.5f * x * (1.0f + tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x)));
}

__device__ __forceinline__ void put(void* base, int64_t elem, int as_f32, float v) {
    if (as_f32) static_cast<float*>(base)[elem] = v;
    else static_cast<bf16_t*>(base)[elem] = f32_to_bf16(v);
}

// The epilogue kinds of the bf16 GEMM with float32 activations: q, k, v (and y, resid where flagged) are float arrays.
template <int KIND>
__device__ __forceinline__ void store_f32(const GemmEpilogue& ep, int row, int col, float acc) {
    float val = acc + (ep.bias ? ep.bias[col] : 0.f);
    if (KIND == EPI_PLAIN) {
        if (ep.act == REGIONE_ACT_GELU_TANH && col >= ep.act_from) val = gelu_tanh_exact(val);
        put(ep.y, static_cast<int64_t>(row) * ep.ldy + col, ep.y_f32, val);
    } else if (KIND == EPI_QKV) {
        const int H = ep.hidden;
        if (col < H) {
            reinterpret_cast<float*>(ep.q)[static_cast<int64_t>(row) * ep.ldq + col] = val;
        } else if (col < 3 * H) {
            const int64_t kv_row = epilogue_slot(ep, row);
            if (col < 2 * H) reinterpret_cast<float*>(ep.k)[kv_row * ep.ldkv + (col - H)] = val;
            else reinterpret_cast<float*>(ep.v)[kv_row * ep.ldkv + (col - 2 * H)] = val;
        } else {
            if (ep.act == REGIONE_ACT_GELU_TANH) val = gelu_tanh_exact(val);
            put(ep.y, static_cast<int64_t>(row) * ep.ldy + ep.y_col0 + (col - 3 * H), ep.y_f32, val);
        }
    } else {  // EPI_RESID
        const int64_t ri = static_cast<int64_t>(row) * ep.ldr + col;
        const float res = ep.resid_f32 ? static_cast<const float*>(ep.resid)[ri] : bf16_to_f32(static_cast<const bf16_t*>(ep.resid)[ri]);
        const float gate = ep.gate ? ep.gate[col] : 1.f;
        put(ep.y, static_cast<int64_t>(row) * ep.ldy + col, ep.y_f32, res + gate * val);
    }
}

// C[m, n] = sum_k A[m, k] W[n, k]; A row-major float32 (lda a multiple of 4), W row-major [n, k], K a multiple of 16.
// Rows past M and columns past N are computed on a repeated valid row and never stored.
// A workgroup of NW waves owns a tile of RB*16 x CB*16; the waves split K into NW contiguous ranges of 16-wide chunks.
// Which k of the instruction an element becomes is irrelevant as long as both operands agree: lane l holds row
// (column) l % 16 of the block and, in MFMA e of a chunk, k = 4 * (l / 16) + e, so a chunk of a fragment is one 16-byte
// load per lane, 64 contiguous bytes per row.  PF chunks are requested before the first of them is used.
// 36 rows, float32 (same box, in a loop): 768 columns of K 256 11.1 -> 5.0 us, 256 of K 1024 30.0 -> 5.5, most of it the
// launch; 640 x 256 x 1024 30.6 -> 12.9.
// LDS row stride TN + 4: the four row groups that a store of the accumulator touches fall into different banks.
// LN: A holds the rows before their LayerNorm + modulation (K <= kLnF32Columns, 16-byte aligned like the vectors); the waves normalise the tile's rows into LDS while the weights
// are on their way, which takes the LayerNorm's launch and its trip through memory away: 36 rows of 256,
// kernel trace, 3.3 + 3.9 -> 5.2 us (768 columns), 3.3 + 3.8 -> 4.9 (1024).
constexpr int kLnF32Columns = 512, kLnF32Tiles = 256;
__host__ __device__ constexpr int ln_f32_row(int k) { return k + 4; }     // floats; 16 bytes on: the rows of a fragment start in different banks
template <int KIND, int RB, int CB, int NW, int PF, bool LN>
__device__ __forceinline__ void gemm_f32_tile(float (&part)[NW][RB * 16][CB * 16 + 4], int tile_y, const float* __restrict__ A, int lda, const float* __restrict__ W, int M, int N, int K,
                                              const float* __restrict__ shift, const float* __restrict__ scale, const GemmEpilogue& ep) {
    constexpr int TM = RB * 16, TN = CB * 16;
    const int m0 = tile_y * TM, n0 = blockIdx.x * TN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const float* ap[RB];
    const float* wp[CB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        int r = m0 + 16 * i + l16; r = r < M ? r : M - 1;
        ap[i] = A + static_cast<int64_t>(r) * lda + 4 * lq;
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        int r = n0 + 16 * j + l16; r = r < N ? r : N - 1;
        wp[j] = W + static_cast<int64_t>(r) * K + 4 * lq;
    }
    f32x4 acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto chunks = [&](int c, auto count) __attribute__((always_inline)) {
        constexpr int P = decltype(count)::value;
        f32x4 av[P][RB], wv[P][CB];
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma unroll
            for (int i = 0; i < RB; ++i) av[p][i] = *reinterpret_cast<const f32x4*>(ap[i] + (c + p) * FK);
#pragma unroll
            for (int j = 0; j < CB; ++j) wv[p][j] = *reinterpret_cast<const f32x4*>(wp[j] + (c + p) * FK);
        }
        __builtin_amdgcn_sched_barrier(0);   // every load of the group is on its way before the first product
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < CB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[p][i][e], wv[p][j][e], acc[i][j], 0, 0, 0);
    };
    const int64_t n_chunks = K / FK;
    int c = __builtin_amdgcn_readfirstlane(static_cast<int>(n_chunks * wave / NW));
    const int c_end = __builtin_amdgcn_readfirstlane(static_cast<int>(n_chunks * (wave + 1) / NW));
    if constexpr (LN) {
        constexpr int P = kLnF32Columns / FK / NW;               // a wave's chunks of the longest row
        extern __shared__ __attribute__((aligned(16))) float rows[];
        f32x4 wv[P][CB];
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (c + p < c_end) {
#pragma unroll
                for (int j = 0; j < CB; ++j) wv[p][j] = *reinterpret_cast<const f32x4*>(wp[j] + (c + p) * FK);
            }
#pragma unroll
        for (int r = 0; r < TM / NW; ++r) {
            const int lr = wave * (TM / NW) + r;
            const int hr = m0 + lr < M ? m0 + lr : M - 1;
            layernorm_row<float, kLnF32Columns / 512>(A + static_cast<int64_t>(hr) * lda, K, shift, scale, [&](int g, const float (&o)[8]) { st8<float>(rows + lr * ln_f32_row(K) + g * 8, o); });
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (c + p < c_end) {
                f32x4 av[RB];
#pragma unroll
                for (int i = 0; i < RB; ++i) av[i] = *reinterpret_cast<const f32x4*>(rows + (16 * i + l16) * ln_f32_row(K) + (c + p) * FK + 4 * lq);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < RB; ++i)
#pragma unroll
                        for (int j = 0; j < CB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][e], wv[p][j][e], acc[i][j], 0, 0, 0);
            }
        c = c_end;
    }
    for (; c + PF <= c_end; c += PF) chunks(c, std::integral_constant<int, PF>{});
    for (; c + 2 <= c_end; c += 2) chunks(c, std::integral_constant<int, 2>{});
    if (c < c_end) chunks(c, std::integral_constant<int, 1>{});
    // accumulator r of a lane: row 4*(lane/16) + r, column lane%16 of a 16 x 16 block
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * lq + r][16 * j + l16] = acc[i][j][r];
    __syncthreads();
    for (int e = threadIdx.x; e < TM * TN; e += NW * 64) {
        const int r = e / TN, cc = e % TN;
        if (m0 + r >= M || n0 + cc >= N) continue;
        float sum = part[0][r][cc];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += part[w][r][cc];
        store_f32<KIND>(ep, m0 + r, n0 + cc, sum);
    }
}

template <int KIND, int RB, int CB, int NW, int PF, bool LN>
__global__ void __launch_bounds__(NW * 64)
gemm_f32_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W, int M, int N, int K, const float* __restrict__ shift, const float* __restrict__ scale, GemmEpilogue ep) {
    __shared__ float part[NW][RB * 16][CB * 16 + 4];
    gemm_f32_tile<KIND, RB, CB, NW, PF, LN>(part, blockIdx.y, A, lda, W, M, N, K, shift, scale, ep);
}
// Two products of one shape but for their rows, as in gemm_small_pair_kernel.  A block of hidden 256, 16 + 36 rows: 41.8 -> 24.7 us, 64 + 256 rows: 54.7 -> 45.3.
struct F32Product { const float* a; int lda; const float* w; int m; const float* shift; const float* scale; GemmEpilogue ep; };
template <int KIND, int RB, int CB, int NW, int PF, bool LN>
__global__ void __launch_bounds__(NW * 64)
gemm_f32_pair_kernel(F32Product p, F32Product q, int tiles_p, int N, int K) {
    __shared__ float part[NW][RB * 16][CB * 16 + 4];
    if (static_cast<int>(blockIdx.y) < tiles_p) gemm_f32_tile<KIND, RB, CB, NW, PF, LN>(part, blockIdx.y, p.a, p.lda, p.w, p.m, N, K, p.shift, p.scale, p.ep);
    else gemm_f32_tile<KIND, RB, CB, NW, PF, LN>(part, blockIdx.y - tiles_p, q.a, q.lda, q.w, q.m, N, K, q.shift, q.scale, q.ep);
}

// C[m, n] = sum_k A[m, k] W[n, k]; A row-major float32 (lda a multiple of 4), W row-major [n, k], K a multiple of 16.
// Rows past M and columns past N are computed on a repeated valid row and never stored.
// The form for many tiles: 64 x 64 per workgroup, operands shared through LDS, so that the rows are fetched half as
// often as with 32 x 32 tiles (2000 x 1024 x 256: 16.3 us against 22.2).
template <int KIND>
__global__ void __launch_bounds__(kThreads)
gemm_f32_wide_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W, int M, int N, int K, GemmEpilogue ep) {
    __shared__ float a_lds[FB][FK + 1];   // odd row stride: the 32 rows a fragment read touches fall into 32 banks
    __shared__ float w_lds[FB][FK + 1];
    const int m0 = blockIdx.y * FB, n0 = blockIdx.x * FB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = threadIdx.x >> 2, c4 = (threadIdx.x & 3) * 4;
    int ar = m0 + lrow; ar = ar < M ? ar : M - 1;
    int wr = n0 + lrow; wr = wr < N ? wr : N - 1;
    const float* ap = A + static_cast<int64_t>(ar) * lda + c4;
    const float* wp = W + static_cast<int64_t>(wr) * K + c4;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int k0 = 0; k0 < K; k0 += FK) {
        const f32x4 av = *reinterpret_cast<const f32x4*>(ap + k0);
        const f32x4 wv = *reinterpret_cast<const f32x4*>(wp + k0);
        __syncthreads();   // every wave has finished reading the tiles of the step before
#pragma unroll
        for (int e = 0; e < 4; ++e) { a_lds[lrow][c4 + e] = av[e]; w_lds[lrow][c4 + e] = wv[e]; }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < FK / 2; ++kk) {
            // operand layout of the 32x32x2 instruction: lane l holds row (column) l % 32 at k = l / 32
            const float a = a_lds[wm * 32 + l32][2 * kk + lh];
            const float b = w_lds[wn * 32 + l32][2 * kk + lh];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
        }
    }
    // accumulator r of a lane: row 8*(r/4) + 4*(lane/32) + r%4, column lane%32 of the wave's 32 x 32 block
    const int col = n0 + wn * 32 + l32;
    if (col >= N) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
        if (row < M) store_f32<KIND>(ep, row, col, acc[r]);
    }
}

__global__ void __launch_bounds__(kThreads)
pack_weight_f32_kernel(const float* __restrict__ w, int n, int n_pad, int k, float* __restrict__ wp) {
    const int64_t total = static_cast<int64_t>(n_pad) * k;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < total; i += stride)
        wp[i] = (i / k) < n ? w[i] : 0.f;
}

struct AttnF32Args {
    const float* q; int ldq; int n_q;
    const float* k0; const float* v0; int ldkv0; int n0;
    const float* k1; const float* v1; int ldkv1; int n1; const int32_t* idx1;
    float scale; float* out; int ldo;
    int splits; float* part; int* arrived;      // key ranges of a query tile, each a workgroup; their partial results and the tiles' arrival counters
};

// Eq.6 for 16 query rows of one head per workgroup: the key list is the fresh rows followed by the cache rows in use,
// in groups of 16 that are dealt to the NW waves in contiguous ranges.  A wave forms the transposed scores
// S^T = K Q^T of a group with v_mfma_f32_16x16x4_f32: a lane then holds, for ONE query (l % 16), the scores of keys
// 4 * (l / 16) + r, which is already the "B" operand of O^T = V^T P^T (MFMA r multiplies the keys 4 * (l / 16) + r).
// Row i of V^T block (j, e) is output element d = 64 j + 4 i + e, so a lane reads V in 16-byte pieces, 256 contiguous
// bytes per key, and holds 4 consecutive output elements per accumulator index.  K and V of the next group are
// requested before the present group is used.  The waves' partial results (maximum, sum, O) meet in LDS, in wave order.
// One wave per (query, head) with a serial walk over the values, the form before this one, took 96.5 us for 36 queries
// on 544 keys (4 heads of 64) and 290 for 640 on 1216; now 13.3 and 24.4: the matrix instructions of one CU per 16
// queries and head, and the launch.
// Where the queries and heads leave most of the chip idle, up to kF32Splits workgroups share a query tile's keys; their partial results travel in 16-byte accesses of device
// scope (the sc1 bit of a buffer access), since the workgroups may sit on different XCDs.  36 queries on 544 keys, 4 heads of 64, are twelve workgroups whose matrix
// instructions alone take 4 us: 13.3 -> 8.8 us in five ranges; 100 queries 13.4 -> 9.4, 200 on 800 keys 17.9 -> 14.0, 9 on 544 12.7 -> 8.0.
constexpr int kF32Splits = 8, kF32Workgroups = 128, kF32DeviceScope = 16;
typedef __attribute__((ext_vector_type(4))) unsigned int f32_u32x4;
template <int D, int NW, bool RANGES>
__global__ void __launch_bounds__(NW * 64)
attn_f32_kernel(AttnF32Args a) {
    constexpr int KC = D / 16, VJ = D / 64;
    __shared__ float m_lds[NW][16], l_lds[NW][16];
    __shared__ f32x4 o_lds[NW][16][D / 4 + 1];      // odd row stride in 16-byte pieces
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const int q0 = blockIdx.x * 16, head = blockIdx.y;
    const int n_keys = a.n0 + a.n1;
    const unsigned part_bytes = 16u * (D + 4) * 4u, tile_part = (head * gridDim.x + blockIdx.x) * a.splits * part_bytes;      // the launcher keeps all of them below 2 GiB
    const auto part_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.part, 0, static_cast<int>(gridDim.x * gridDim.y * a.splits * part_bytes), 0x00027000);
    const int64_t all_groups = (static_cast<int64_t>(n_keys) + 15) / 16;
    const int first_group = RANGES ? static_cast<int>(all_groups * blockIdx.z / a.splits) : 0;       // of this workgroup's key range
    const int64_t n_groups = RANGES ? all_groups * (blockIdx.z + 1) / a.splits - first_group : all_groups;
    const int g0 = __builtin_amdgcn_readfirstlane(first_group + static_cast<int>(n_groups * wave / NW));
    const int g1 = __builtin_amdgcn_readfirstlane(first_group + static_cast<int>(n_groups * (wave + 1) / NW));
    f32x4 q[KC];
    {
        int r = q0 + l16; r = r < a.n_q ? r : a.n_q - 1;
        const float* qp = a.q + static_cast<int64_t>(r) * a.ldq + head * D + 4 * lq;
        // rows of q carry no alignment promise beyond their elements'
#pragma unroll
        for (int c = 0; c < KC; ++c) q[c] = f32x4{qp[16 * c], qp[16 * c + 1], qp[16 * c + 2], qp[16 * c + 3]};
    }
    auto row_of = [&](int key, const float* base0, const float* base1) -> const float* {
        key = key < n_keys ? key : n_keys - 1;      // keys past the end repeat a valid one; their weight is zero
        if (key < a.n0) return base0 + static_cast<int64_t>(key) * a.ldkv0 + head * D;
        int64_t r = key - a.n0;
        if (a.idx1) r = a.idx1[r];
        return base1 + r * a.ldkv1 + head * D;
    };
    auto load = [&](int g, f32x4 (&k)[KC], f32x4 (&v)[4][VJ]) __attribute__((always_inline)) {
        const float* kp = row_of(16 * g + l16, a.k0, a.k1) + 4 * lq;
        const float* vp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) vp[r] = row_of(16 * g + 4 * lq + r, a.v0, a.v1) + 4 * l16;
#pragma unroll
        for (int c = 0; c < KC; ++c) k[c] = *reinterpret_cast<const f32x4*>(kp + 16 * c);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < VJ; ++j) v[r][j] = *reinterpret_cast<const f32x4*>(vp[r] + 64 * j);
    };
    f32x4 o[VJ][4];
#pragma unroll
    for (int j = 0; j < VJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;           // l_run: this lane's keys only, until the end
    auto group = [&](int g, const f32x4 (&k)[KC], const f32x4 (&v)[4][VJ]) __attribute__((always_inline)) {
        // two chains of products: even and odd chunks
        f32x4 s = {0.f, 0.f, 0.f, 0.f}, s2 = s;
#pragma unroll
        for (int c = 0; c < KC; c += 2)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c][e], q[c][e], s, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c + 1][e], q[c + 1][e], s2, 0, 0, 0);
            }
        const int live = n_keys - (16 * g + 4 * lq);   // of this lane's four keys, those below `live` exist
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = r < live ? (s[r] + s2[r]) * a.scale : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const float ref = m_new == -INFINITY ? 0.f : m_new;   // only -inf so far: weights 0, not NaN
        const float alpha = expf(m_run - ref);                // 0 for the first group
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int j = 0; j < VJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[j][e] *= alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = r < live ? expf(s[r] - ref) : 0.f;
            l_run += p;
#pragma unroll
            for (int j = 0; j < VJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)   // a repeated row contributes 0 * 0 even where it holds an infinity
                    o[j][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(r < live ? v[r][j][e] : 0.f, p, o[j][e], 0, 0, 0);
        }
    };
    f32x4 ka[KC], va[4][VJ], kb[KC], vb[4][VJ];
    if (g0 < g1) load(g0, ka, va);
    for (int g = g0; g < g1; g += 2) {
        if (g + 1 < g1) load(g + 1, kb, vb);
        __builtin_amdgcn_sched_barrier(0);
        group(g, ka, va);
        if (g + 1 < g1) {
            if (g + 2 < g1) load(g + 2, ka, va);
            __builtin_amdgcn_sched_barrier(0);
            group(g + 1, kb, vb);
        }
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (lq == 0) { m_lds[wave][l16] = m_run; l_lds[wave][l16] = l_run; }
    // accumulator r of block (j, e): query l16, d = 64 j + 4 (4 lq + r) + e
#pragma unroll
    for (int j = 0; j < VJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) o_lds[wave][l16][16 * j + 4 * lq + r] = f32x4{o[j][0][r], o[j][1][r], o[j][2][r], o[j][3][r]};
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * (D / 4); t += NW * 64) {
        const int row = t / (D / 4), piece = t % (D / 4);
        if (q0 + row >= a.n_q) continue;
        float m = m_lds[0][row];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, m_lds[w][row]);
        const float ref = m == -INFINITY ? 0.f : m;
        float l = 0.f;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (n_groups * w / NW == n_groups * (w + 1) / NW) continue;   // a wave without keys
            const float f = expf(m_lds[w][row] - ref);
            l = fmaf(f, l_lds[w][row], l);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = fmaf(f, o_lds[w][row][piece][e], sum[e]);
        }
        if (RANGES) {               // maximum, sum and unnormalised O of the range, past this XCD's own L2
            const unsigned at = tile_part + blockIdx.z * part_bytes + row * (D + 4) * 4u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(f32_u32x4, sum), part_rsrc, at + 16u + 16u * piece, 0, kF32DeviceScope);
            if (piece == 0) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(f32_u32x4, f32x4{m, l, 0.f, 0.f}), part_rsrc, at, 0, kF32DeviceScope);
            continue;
        }
        const float inv = 1.0f / l;
        float* op = a.out + static_cast<int64_t>(q0 + row) * a.ldo + head * D + 4 * piece;
#pragma unroll
        for (int e = 0; e < 4; ++e) op[e] = sum[e] * inv;
    }
    if constexpr (!RANGES) return;
    // The workgroup of the query tile that arrives last joins the ranges, in key order whoever is last.  Nobody waits.
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __syncthreads();
    __shared__ int s_last;
    if (threadIdx.x == 0) {
        int* at = a.arrived + head * gridDim.x + blockIdx.x;
        s_last = __hip_atomic_fetch_add(at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.splits - 1;
        if (s_last) __hip_atomic_store(at, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);     // ready for the next launch
    }
    __syncthreads();
    if (!s_last) return;
    for (int t = threadIdx.x; t < 16 * (D / 4); t += NW * 64) {
        const int row = t / (D / 4), piece = t % (D / 4);
        if (q0 + row >= a.n_q) continue;
        f32x4 ml[kF32Splits], o_part[kF32Splits];
#pragma unroll
        for (int z = 0; z < kF32Splits; ++z)
            if (z < a.splits) {
                const unsigned at = tile_part + z * part_bytes + row * (D + 4) * 4u;
                ml[z] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part_rsrc, at, 0, kF32DeviceScope));
                o_part[z] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part_rsrc, at + 16u + 16u * piece, 0, kF32DeviceScope));
            }
        float m = -INFINITY;
#pragma unroll
        for (int z = 0; z < kF32Splits; ++z) if (z < a.splits) m = fmaxf(m, ml[z][0]);
        const float ref = m == -INFINITY ? 0.f : m;
        float l = 0.f;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int z = 0; z < kF32Splits; ++z)
            if (z < a.splits) {
                const float f = expf(ml[z][0] - ref);
                l = fmaf(f, ml[z][1], l);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = fmaf(f, o_part[z][e], sum[e]);
            }
        const float inv = 1.0f / l;
        float* op = a.out + static_cast<int64_t>(q0 + row) * a.ldo + head * D + 4 * piece;
#pragma unroll
        for (int e = 0; e < 4; ++e) op[e] = sum[e] * inv;
    }
}

void launch_gemm_f32_wide(regione_ctx* ctx, const float* a, int lda, const float* w, int m, int n, int k, const GemmEpilogue& ep) {
    const dim3 grid((n + FB - 1) / FB, (m + FB - 1) / FB);
    switch (ep.kind) {
        case EPI_PLAIN: hipLaunchKernelGGL((gemm_f32_wide_kernel<EPI_PLAIN>), grid, dim3(kThreads), 0, ctx->stream, a, lda, w, m, n, k, ep); break;
        case EPI_QKV: hipLaunchKernelGGL((gemm_f32_wide_kernel<EPI_QKV>), grid, dim3(kThreads), 0, ctx->stream, a, lda, w, m, n, k, ep); break;
        default: hipLaunchKernelGGL((gemm_f32_wide_kernel<EPI_RESID>), grid, dim3(kThreads), 0, ctx->stream, a, lda, w, m, n, k, ep); break;
    }
}

// Rows that are normalised in LDS beside the partial sums: 10 + 33 KiB at most with tiles of 16 x 16, 36 + 65 with 32 x 32.
template <auto KERNEL, int RB, int CB, int NW> int grant_rows(const regione_ctx* ctx) {
    constexpr size_t sums = sizeof(float) * NW * RB * 16 * (CB * 16 + 4), rows = sizeof(float) * RB * 16 * ln_f32_row(kLnF32Columns);
    if constexpr (sums + rows <= 65536) return REGIONE_OK;
    static std::atomic<uint64_t> granted{0};
    return rg_grant_lds(ctx, reinterpret_cast<const void*>(KERNEL), granted, rows);
}
template <int RB, int CB, int NW, int PF, bool LN>
int launch_gemm_f32(regione_ctx* ctx, const float* a, int lda, const float* w, int m, int n, int k, const float* shift, const float* scale, const GemmEpilogue& ep) {
    const dim3 grid((n + CB * 16 - 1) / (CB * 16), (m + RB * 16 - 1) / (RB * 16)), block(NW * 64);
    const size_t lds = LN ? static_cast<size_t>(RB) * 16 * ln_f32_row(k) * sizeof(float) : 0;
#define RG_LAUNCH(KIND) { \
        if constexpr (LN) { if (int rc = grant_rows<&gemm_f32_kernel<KIND, RB, CB, NW, PF, LN>, RB, CB, NW>(ctx)) return rc; } \
        hipLaunchKernelGGL((gemm_f32_kernel<KIND, RB, CB, NW, PF, LN>), grid, block, lds, ctx->stream, a, lda, w, m, n, k, shift, scale, ep); break; }
    switch (ep.kind) {
        case EPI_PLAIN: RG_LAUNCH(EPI_PLAIN)
        case EPI_QKV: RG_LAUNCH(EPI_QKV)
        default: if constexpr (!LN) RG_LAUNCH(EPI_RESID)
    }
#undef RG_LAUNCH
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
int64_t tiles_f32(int m, int n, int64_t b) { return ((m + b - 1) / b) * ((n + b - 1) / b); }

}  // namespace

int rg_pack_weight_f32(regione_ctx* ctx, const float* w, int n, int k, float* w_packed) {
    const int n_pad = (n + 31) / 32 * 32;
    int64_t blocks = (static_cast<int64_t>(n_pad) * k + kThreads - 1) / kThreads;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(pack_weight_f32_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, ctx->stream, w, n, n_pad, k, w_packed);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

int rg_gemm_f32(regione_ctx* ctx, const float* a, int lda, const float* w, int m, int n, int k, const GemmEpilogue& ep) {
    if (m <= 0 || n <= 0) return REGIONE_OK;
    if (k <= 0 || (k % FK) || (lda & 3)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm (float32): k=%d must be a positive multiple of 16 and lda=%d of 4", k, lda);
    if (!rg_aligned16(a) || !rg_aligned16(w)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm (float32): operands must be 16-byte aligned");
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    if ((static_cast<int64_t>(m) + 63) / 64 > 65535) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "gemm (float32): %d rows exceed this simple kernel's grid", m);
    if (ep.kind != EPI_PLAIN && ep.kind != EPI_QKV && ep.kind != EPI_RESID) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm (float32): bad epilogue kind %d", ep.kind);
    // The smaller the tile, the more workgroups share the latency of a short product; the larger, the fewer bytes per
    // product.  Measured (us, tiles of 16 / 32 / 64): 36 x 768 x 256 3.8 / 4.3 / 11, 205 x 256 x 1024 5.6 / 10.3 / 30,
    // 205 x 768 x 256 (624 tiles of 16) 5.0 / 4.5 / 11, 640 x 256 x 1024 (640) 12.6 / 10.4 / 31,
    // 1216 x 768 x 256 (228 tiles of 64) 17 / 11.6 / 11.7, 2000 x 1024 x 256 (512) 34 / 22 / 16.
    if (tiles_f32(m, n, 64) < 256)
        return tiles_f32(m, n, 16) > 512 ? launch_gemm_f32<2, 2, 8, 4, false>(ctx, a, lda, w, m, n, k, nullptr, nullptr, ep)
                                         : launch_gemm_f32<1, 1, 8, 8, false>(ctx, a, lda, w, m, n, k, nullptr, nullptr, ep);
    launch_gemm_f32_wide(ctx, a, lda, w, m, n, k, ep);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

template <int RB, int CB, int NW, int PF>
static int launch_gemm_f32_pair(regione_ctx* ctx, const GemmCall& a, const GemmCall& b) {
    const int ya = (a.m + RB * 16 - 1) / (RB * 16), yb = (b.m + RB * 16 - 1) / (RB * 16);
    const dim3 grid((a.n + CB * 16 - 1) / (CB * 16), ya + yb), block(NW * 64);
    const size_t lds = a.norm ? static_cast<size_t>(RB) * 16 * ln_f32_row(a.k) * sizeof(float) : 0;
    auto product = [](const GemmCall& c) { return F32Product{static_cast<const float*>(c.a), c.lda, static_cast<const float*>(c.w), c.m, c.shift, c.scale, c.ep}; };
#define RG_PAIR(KIND, LN) { \
        if constexpr (LN) { if (int rc = grant_rows<&gemm_f32_pair_kernel<KIND, RB, CB, NW, PF, LN>, RB, CB, NW>(ctx)) return rc; } \
        hipLaunchKernelGGL((gemm_f32_pair_kernel<KIND, RB, CB, NW, PF, LN>), grid, block, lds, ctx->stream, product(a), product(b), ya, a.n, a.k); }
    if (a.ep.kind == EPI_RESID) RG_PAIR(EPI_RESID, false)
    else if (a.ep.kind == EPI_QKV) { if (a.norm) RG_PAIR(EPI_QKV, true) else RG_PAIR(EPI_QKV, false) }
    else { if (a.norm) RG_PAIR(EPI_PLAIN, true) else RG_PAIR(EPI_PLAIN, false) }
#undef RG_PAIR
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
static bool pair_fine(const GemmCall& a, const GemmCall& b) { return tiles_f32(a.m, a.n, 16) + tiles_f32(b.m, b.n, 16) <= 512; }
// The rules of one product for the tiles of both.  Tiles of 32 x 32 only while the pair takes no round of the 256 compute units more than its larger product alone: a product that
// is small alone has tiles of 16 x 16 to fill the chip with.  A block, us, two launches -> one: hidden 512, 128 + 300 rows 105.6 -> 91.7, 64 + 700 169 -> 155; without the rule
// 64 + 500 (288 tiles for 256) 126 -> 136, hidden 1024, 64 + 256 (320 for 256) 187 -> 210.
bool rg_gemm_pairs_f32(const GemmCall& a, const GemmCall& b) {
    if (a.k <= 0 || a.k % FK || (a.norm && (a.k > kLnF32Columns || !a.a_f32))) return false;
    const bool fine = pair_fine(a, b);
    const int64_t ta = tiles_f32(a.m, a.n, fine ? 16 : 32), tb = tiles_f32(b.m, b.n, fine ? 16 : 32);
    if (tiles_f32(a.m, a.n, 64) + tiles_f32(b.m, b.n, 64) >= 256 || (a.norm && ta + tb > kLnF32Tiles)) return false;
    return fine || (ta + tb + 255) / 256 == ((ta > tb ? ta : tb) + 255) / 256;
}
int rg_gemm_pair_f32(regione_ctx* ctx, const GemmCall& a, const GemmCall& b) {
    return pair_fine(a, b) ? launch_gemm_f32_pair<1, 1, 8, 8>(ctx, a, b) : launch_gemm_f32_pair<2, 2, 8, 4>(ctx, a, b);
}

// The product of layernorm_mod(h) in one launch, bit for bit that of the two, where every workgroup of one round of 256 normalises its own rows; *done tells whether it was.
int rg_layernorm_gemm_f32(regione_ctx* ctx, const float* h, const float* shift, const float* scale, const float* w, int m, int n, int k, const GemmEpilogue& ep, bool* done) {
    *done = false;
    if (k <= 0 || k % FK || k > kLnF32Columns || !rg_aligned16(h) || !rg_aligned16(w) || !rg_aligned16(shift) || !rg_aligned16(scale) || (ep.kind != EPI_PLAIN && ep.kind != EPI_QKV)) return REGIONE_OK;
    const bool fine = tiles_f32(m, n, 16) <= 512;
    if (tiles_f32(m, n, fine ? 16 : 32) > kLnF32Tiles || tiles_f32(m, n, 64) >= 256) return REGIONE_OK;
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    *done = true;
    return fine ? launch_gemm_f32<1, 1, 8, 8, true>(ctx, h, k, w, m, n, k, shift, scale, ep) : launch_gemm_f32<2, 2, 8, 4, true>(ctx, h, k, w, m, n, k, shift, scale, ep);
}

int rg_attention_f32(regione_ctx* ctx, const float* q, int ldq, int n_q,
                     const float* k0, const float* v0, int ldkv0, int n0,
                     const float* k1, const float* v1, int ldkv1, int n1, const int32_t* idx1,
                     int heads, int d, float scale, float* out, int ldo) {
    if (n_q <= 0) return REGIONE_OK;
    if (n0 + n1 <= 0) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attention: %d queries but no key", n_q);
    if (d != 64 && d != 128) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention: head dimension %d (64 or 128 supported)", d);
    if ((n0 > 0 && (ldkv0 & 3)) || (n1 > 0 && (ldkv1 & 3))) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attention (float32): row strides must keep 16-byte alignment");
    if (heads > 65535) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention (float32): %d heads", heads);
    ProfScope prof(ctx, REGIONE_PROF_ATTENTION);
    AttnF32Args a = {q, ldq, n_q, k0, v0, ldkv0, n0, k1, v1, ldkv1, n1, idx1, scale > 0.f ? scale : 1.0f / sqrtf(static_cast<float>(d)), out, ldo, 1, ctx->attn_part, ctx->gemm_arrived};
    // key ranges as long as the workgroups stay within half a round of the chip and have six groups of keys each: the meeting costs about as much as that
    const int64_t tiles = static_cast<int64_t>((n_q + 15) / 16) * heads, groups = (static_cast<int64_t>(n0) + n1 + 15) / 16;
    if (tiles <= kMaxSplitTiles && 2 * tiles <= kF32Workgroups) {
        int64_t z = kF32Workgroups / tiles;
        z = z < groups / 6 ? z : groups / 6;
        z = z < kF32Splits ? z : kF32Splits;
        const size_t bytes = static_cast<size_t>(tiles) * (z > 0 ? z : 1) * 16 * (d + 4) * sizeof(float);
        if (z > 1 && bytes <= ctx->attn_part_bytes && bytes < (size_t{1} << 31)) a.splits = static_cast<int>(z);
    }
    const dim3 grid(static_cast<unsigned>((n_q + 15) / 16), static_cast<unsigned>(heads), static_cast<unsigned>(a.splits));
    if (d == 64 && a.splits > 1) hipLaunchKernelGGL((attn_f32_kernel<64, 12, true>), grid, dim3(768), 0, ctx->stream, a);
    else if (d == 64) hipLaunchKernelGGL((attn_f32_kernel<64, 12, false>), grid, dim3(768), 0, ctx->stream, a);
    else if (a.splits > 1) hipLaunchKernelGGL((attn_f32_kernel<128, 4, true>), grid, dim3(256), 0, ctx->stream, a);
    else hipLaunchKernelGGL((attn_f32_kernel<128, 4, false>), grid, dim3(256), 0, ctx->stream, a);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}
