// Memory-bound row kernels: gather / scatter by index list (Algorithm 1, "X[E_index]" and the
// merge line), the adaptive velocity decay cache fused with the Euler update (Eq.9, Eq.4), and
// LayerNorm + modulation of the block.
#include "common.h"
#include "layernorm_row.h"

namespace {

constexpr int kThreads = 256;
typedef unsigned int rows_u32x4 __attribute__((ext_vector_type(4)));

// unit = one 16-byte (or ELEM-byte) piece of one row; GATHER: dst[i] = src[index[i]], else dst[index[i]] = src[i]
template <typename V, bool GATHER>
__global__ void __launch_bounds__(kThreads)
rows_by_index_kernel(const V* __restrict__ src, V* __restrict__ dst, const int32_t* __restrict__ index,
                     const int32_t* __restrict__ n_dev, int64_t n_max, int pieces_per_row) {
    int64_t n = n_max;
    if (n_dev) { const int64_t nd = *n_dev; n = nd < n_max ? (nd < 0 ? 0 : nd) : n_max; }
    const int64_t total = n * pieces_per_row;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t u = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; u < total; u += stride) {
        const int64_t row = u / pieces_per_row;
        const int piece = static_cast<int>(u - row * pieces_per_row);
        const int64_t other = index[row];
        // every row is touched once: non-temporal accesses
        if (GATHER) __builtin_nontemporal_store(__builtin_nontemporal_load(src + other * pieces_per_row + piece), dst + row * pieces_per_row + piece);
        else __builtin_nontemporal_store(__builtin_nontemporal_load(src + row * pieces_per_row + piece), dst + other * pieces_per_row + piece);
    }
}

template <bool GATHER>
int rows_by_index(regione_ctx* ctx, const void* src, void* dst, int32_t row_elems, int32_t dtype,
                  const int32_t* index, const int32_t* n_dev, int64_t n_max, const char* who) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "%s: null context", who);
    if (row_elems <= 0 || n_max < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "%s: row_elems=%d n_max=%lld", who, row_elems, (long long)n_max);
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "%s: bad dtype %d", who, dtype);
    if (n_max == 0) return REGIONE_OK;
    if (!src || !dst || !index) RG_FAIL(REGIONE_ERR_INVALID_ARG, "%s: null tensor", who);
    const int64_t row_bytes = static_cast<int64_t>(row_elems) * (dtype == REGIONE_BF16 ? 2 : 4);
    const bool wide = (row_bytes % 16 == 0) && rg_aligned16(src) && rg_aligned16(dst);
    const int piece_bytes = wide ? 16 : (dtype == REGIONE_BF16 ? 2 : 4);
    const int ppr = static_cast<int>(row_bytes / piece_bytes);
    const int64_t total = n_max * ppr;
    int64_t blocks = (total + kThreads - 1) / kThreads;
    if (blocks > 256 * 64) blocks = 256 * 64;
    dim3 grid(static_cast<unsigned>(blocks));
    ProfScope prof(ctx, REGIONE_PROF_ROWS);
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    if (piece_bytes == 16)
        hipLaunchKernelGGL((rows_by_index_kernel<u32x4, GATHER>), grid, dim3(kThreads), 0, ctx->stream,
                           static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), index, n_dev, n_max, ppr);
    else if (piece_bytes == 4)
        hipLaunchKernelGGL((rows_by_index_kernel<uint32_t, GATHER>), grid, dim3(kThreads), 0, ctx->stream,
                           static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), index, n_dev, n_max, ppr);
    else
        hipLaunchKernelGGL((rows_by_index_kernel<uint16_t, GATHER>), grid, dim3(kThreads), 0, ctx->stream,
                           static_cast<const uint16_t*>(src), static_cast<uint16_t*>(dst), index, n_dev, n_max, ppr);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

// The slot list of a step's fresh rows (regione_fresh_slots) beside the launch that gathers them: the text rows' own by the launch's threads, a gathered row's by whoever moves
// its first piece.
struct FreshSlots { int32_t* slots; int n_txt; };
__device__ __forceinline__ void text_slots(const FreshSlots& f, int64_t thread, int64_t threads) {
    if (f.slots) for (int64_t i = thread; i < f.n_txt; i += threads) f.slots[i] = static_cast<int32_t>(i);
}

// Two tensors by one index list in one launch (the hidden rows and the latent rows of the edited tokens): a row of the
// pair is pa + pb 16-byte pieces, the first pa of tensor A.
template <bool GATHER>
__global__ void __launch_bounds__(kThreads)
rows_pair_by_index_kernel(const rows_u32x4* __restrict__ src_a, rows_u32x4* __restrict__ dst_a, int pa,
                          const rows_u32x4* __restrict__ src_b, rows_u32x4* __restrict__ dst_b, int pb,
                          const int32_t* __restrict__ index, const int32_t* __restrict__ n_dev, int64_t n_max, FreshSlots fresh) {
    int64_t n = n_max;
    if (n_dev) { const int64_t nd = *n_dev; n = nd < n_max ? (nd < 0 ? 0 : nd) : n_max; }
    text_slots(fresh, static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x, static_cast<int64_t>(gridDim.x) * kThreads);
    const int ppr = pa + pb;
    const int64_t total = n * ppr;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t u = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; u < total; u += stride) {
        const int64_t row = u / ppr;
        int piece = static_cast<int>(u - row * ppr);
        const int64_t other = index[row];
        if (fresh.slots && piece == 0) fresh.slots[fresh.n_txt + row] = static_cast<int32_t>(other) + fresh.n_txt;
        const bool first = piece < pa;
        const rows_u32x4* src = first ? src_a : src_b;
        rows_u32x4* dst = first ? dst_a : dst_b;
        const int p = first ? pa : pb;
        piece = first ? piece : piece - pa;
        if (GATHER) __builtin_nontemporal_store(__builtin_nontemporal_load(src + other * p + piece), dst + row * p + piece);
        else __builtin_nontemporal_store(__builtin_nontemporal_load(src + row * p + piece), dst + other * p + piece);
    }
}

template <bool GATHER>
int rows_pair(regione_ctx* ctx, const void* src_a, void* dst_a, int32_t elems_a, int32_t dtype_a, const void* src_b, void* dst_b, int32_t elems_b, int32_t dtype_b,
              const int32_t* index, const int32_t* n_dev, int64_t n_max, const char* who, FreshSlots fresh = {nullptr, 0}) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "%s: null context", who);
    const int64_t bytes_a = static_cast<int64_t>(elems_a) * (dtype_a == REGIONE_BF16 ? 2 : 4), bytes_b = static_cast<int64_t>(elems_b) * (dtype_b == REGIONE_BF16 ? 2 : 4);
    const bool wide = elems_a > 0 && elems_b > 0 && n_max > 0 && src_a && dst_a && src_b && dst_b && index && (bytes_a % 16 == 0) && (bytes_b % 16 == 0) &&
                      rg_aligned16(src_a) && rg_aligned16(dst_a) && rg_aligned16(src_b) && rg_aligned16(dst_b) &&
                      (dtype_a == REGIONE_BF16 || dtype_a == REGIONE_FP32) && (dtype_b == REGIONE_BF16 || dtype_b == REGIONE_FP32);
    if (!wide) {   // anything unusual (odd row widths, empty lists, bad arguments): the single-tensor path, with its checks
        if (int rc = rows_by_index<GATHER>(ctx, src_a, dst_a, elems_a, dtype_a, index, n_dev, n_max, who)) return rc;
        if (fresh.slots)
            if (int rc = regione_fresh_slots(ctx, index, n_dev, n_max, fresh.n_txt, fresh.slots)) return rc;
        return rows_by_index<GATHER>(ctx, src_b, dst_b, elems_b, dtype_b, index, n_dev, n_max, who);
    }
    const int pa = static_cast<int>(bytes_a / 16), pb = static_cast<int>(bytes_b / 16);
    int64_t blocks = (n_max * (pa + pb) + kThreads - 1) / kThreads;
    if (blocks > 256 * 64) blocks = 256 * 64;
    ProfScope prof(ctx, REGIONE_PROF_ROWS);
    hipLaunchKernelGGL((rows_pair_by_index_kernel<GATHER>), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, ctx->stream,
                       static_cast<const rows_u32x4*>(src_a), static_cast<rows_u32x4*>(dst_a), pa, static_cast<const rows_u32x4*>(src_b), static_cast<rows_u32x4*>(dst_b), pb,
                       index, n_dev, n_max, fresh);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

template <typename T> __device__ __forceinline__ float ld(const T* p);
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }
template <> __device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <typename T> __device__ __forceinline__ void st(T* p, float v);
template <> __device__ __forceinline__ void st<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }
template <> __device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }

template <typename T>
__global__ void __launch_bounds__(kThreads)
velocity_cache_kernel(int reuse, float factor, float dt, const T* __restrict__ v_fresh, T* __restrict__ c_a,
                      T* __restrict__ v_out, T* __restrict__ x_e, const int32_t* __restrict__ n_dev, int64_t n_max, int c) {
    int64_t n = n_max;
    if (n_dev) { const int64_t nd = *n_dev; n = nd < n_max ? (nd < 0 ? 0 : nd) : n_max; }
    const int64_t total = n * c;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < total; i += stride) {
        float vu;
        if (reuse) {
            vu = __fmul_rn(factor, ld<T>(c_a + i));
        } else {
            vu = ld<T>(v_fresh + i);
            st<T>(c_a + i, vu);
        }
        if (v_out) st<T>(v_out + i, vu);
        st<T>(x_e + i, __fsub_rn(ld<T>(x_e + i), __fmul_rn(dt, vu)));
    }
}

// LayerNorm over H with modulation, one wave per row (see layernorm_row): rows of at most 1024 values, and longer ones whose sums are kept.  Bound by the latency of its loads: 36 float32 rows of 256 values take
// 5.2 us in the kernel of scalar loads below, 3.2 here, with registers and code for as many rounds of 512 values as the row has (in a kernel trace).  8704 rows: of 256 values
// 4.8 us (bf16), 5.5 (float32); of 1024 7.8, 14.6.  U: the output's storage type (bf16, or float32 in a float32 context).
template <typename T, typename U, int MAXV>
__global__ void __launch_bounds__(kThreads)
layernorm_mod_vec_kernel(const T* __restrict__ h, int n, int hidden, const float* __restrict__ shift,
                         const float* __restrict__ scale, U* __restrict__ u) {
    const int row = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= n) return;
    U* ur = u + static_cast<int64_t>(row) * hidden;
    layernorm_row<T, MAXV>(h + static_cast<int64_t>(row) * hidden, hidden, shift, scale, [&](int g, const float (&o)[8]) { st8<U>(ur + g * 8, o); });
}

// Rows of more than 1024 values: a workgroup per row (layernorm_rows_wide).
template <typename T, typename U, int W>
__global__ void __launch_bounds__(64 * W)
layernorm_mod_wide_kernel(const T* __restrict__ h, int n, int hidden, const float* __restrict__ shift,
                          const float* __restrict__ scale, U* __restrict__ u) {
    __shared__ float2 part[2][W];
    layernorm_rows_wide<T, W>(h, n, hidden, shift, scale, part, [](int row) -> int64_t { return row; },
                              [&](int row, int g, bool live, const LnRaw<T>&, const float (&o)[8]) { if (live) st8<U>(u + static_cast<int64_t>(row) * hidden + g * 8, o); });
}

// The same on rows picked by an index list, which go to h_rows on the way, and the latent rows of the same tokens beside them.
template <typename T, typename U, int W>
__global__ void __launch_bounds__(64 * W)
gather_layernorm_kernel(const T* __restrict__ h_full, const int32_t* __restrict__ index, int n, int hidden, const float* __restrict__ shift, const float* __restrict__ scale,
                        T* __restrict__ h_rows, U* __restrict__ u, const rows_u32x4* __restrict__ x_t, rows_u32x4* __restrict__ x_e, int x_pieces, FreshSlots fresh) {
    __shared__ float2 part[2][W];
    text_slots(fresh, static_cast<int64_t>(blockIdx.x) * (64 * W) + threadIdx.x, static_cast<int64_t>(gridDim.x) * (64 * W));
    if (fresh.slots && threadIdx.x == 0)
        for (int row = blockIdx.x; row < n; row += gridDim.x) fresh.slots[fresh.n_txt + row] = index[row] + fresh.n_txt;
    for (int row = blockIdx.x; row < n; row += gridDim.x)
        for (int p = threadIdx.x; p < x_pieces; p += 64 * W) x_e[static_cast<int64_t>(row) * x_pieces + p] = x_t[static_cast<int64_t>(index[row]) * x_pieces + p];
    layernorm_rows_wide<T, W>(h_full, n, hidden, shift, scale, part, [&](int row) -> int64_t { return index[row]; },
                              [&](int row, int g, bool live, const LnRaw<T>& raw, const float (&o)[8]) {
        if (!live) return;
        const int64_t at = static_cast<int64_t>(row) * hidden + g * 8;
        raw.store(h_rows + at);
        st8<U>(u + at, o);
    });
}

// Any H: scalar loads, three passes over the row.
template <typename T, typename U>
__global__ void __launch_bounds__(kThreads)
layernorm_mod_kernel(const T* __restrict__ h, int n, int hidden, const float* __restrict__ shift,
                     const float* __restrict__ scale, U* __restrict__ u) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= n) return;
    const T* hr = h + static_cast<int64_t>(row) * hidden;
    float sum = 0.f;
    for (int c = lane; c < hidden; c += 64) sum += ld<T>(hr + c);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
    const float mean = sum / hidden;
    float sq = 0.f;
    for (int c = lane; c < hidden; c += 64) { const float d = ld<T>(hr + c) - mean; sq += d * d; }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sq += __shfl_xor(sq, m, 64);
    const float rstd = rsqrtf(sq / hidden + 1e-6f);
    U* ur = u + static_cast<int64_t>(row) * hidden;
    for (int c = lane; c < hidden; c += 64) {
        float y = (ld<T>(hr + c) - mean) * rstd;
        const float sc = scale ? scale[c] : 0.f, sh = shift ? shift[c] : 0.f;
        y = y * (1.f + sc) + sh;
        st<U>(ur + c, y);
    }
}

// element-wise conversion between the two storage types (round to nearest even towards bf16)
template <typename S, typename D>
__global__ void __launch_bounds__(kThreads) cast_kernel(const S* __restrict__ src, D* __restrict__ dst, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride) st<D>(dst + i, ld<S>(src + i));
}

// Eq.9 / Eq.4 for 16-byte aligned tensors whose element count is a multiple of eight: eight elements per thread and
// step, the same per-element arithmetic as velocity_cache_kernel (separately rounded product and difference).
// streamed once: non-temporal on both sides
template <typename T> __device__ __forceinline__ void ld8_nt(const T* p, float (&v)[8]);
template <> __device__ __forceinline__ void ld8_nt<bf16_t>(const bf16_t* p, float (&v)[8]) {
    const ln_bf16x8 x = __builtin_nontemporal_load(reinterpret_cast<const ln_bf16x8*>(p));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<float>(x[e]);
}
template <> __device__ __forceinline__ void ld8_nt<float>(const float* p, float (&v)[8]) {
    const ln_f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const ln_f32x4*>(p)), b = __builtin_nontemporal_load(reinterpret_cast<const ln_f32x4*>(p + 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}
template <typename T> __device__ __forceinline__ void st8_nt(T* p, const float (&v)[8]);
template <> __device__ __forceinline__ void st8_nt<bf16_t>(bf16_t* p, const float (&v)[8]) {
    ln_bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(v[e]);
    __builtin_nontemporal_store(o, reinterpret_cast<ln_bf16x8*>(p));
}
template <> __device__ __forceinline__ void st8_nt<float>(float* p, const float (&v)[8]) {
    __builtin_nontemporal_store(ln_f32x4{v[0], v[1], v[2], v[3]}, reinterpret_cast<ln_f32x4*>(p));
    __builtin_nontemporal_store(ln_f32x4{v[4], v[5], v[6], v[7]}, reinterpret_cast<ln_f32x4*>(p + 4));
}
template <typename T>
__global__ void __launch_bounds__(kThreads)
velocity_cache_vec_kernel(int reuse, float factor, float dt, const T* __restrict__ v_fresh, T* __restrict__ c_a,
                          T* __restrict__ v_out, T* __restrict__ x_e, const int32_t* __restrict__ n_dev, int64_t n_max, int c) {
    int64_t n = n_max;
    if (n_dev) { const int64_t nd = *n_dev; n = nd < n_max ? (nd < 0 ? 0 : nd) : n_max; }
    const int64_t groups = n * c / 8;          // c is a multiple of 8 on this path
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    const T* vsrc = reuse ? c_a : v_fresh;
    constexpr int U = 2;                       // groups per thread in flight (four measured the same): all loads of a round before its first store
    for (int64_t g0 = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; g0 < groups; g0 += U * stride) {
        float vu[U][8], x[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t g = g0 + u * stride;
            if (g < groups) { ld8_nt<T>(x_e + g * 8, x[u]); ld8_nt<T>(vsrc + g * 8, vu[u]); }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t g = g0 + u * stride;
            if (g >= groups) continue;
            const int64_t i = g * 8;
            if (reuse) {
#pragma unroll
                for (int e = 0; e < 8; ++e) vu[u][e] = __fmul_rn(factor, vu[u][e]);
            } else {
                st8_nt<T>(c_a + i, vu[u]);
            }
            if (v_out) st8_nt<T>(v_out + i, vu[u]);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[u][e] = __fsub_rn(x[u][e], __fmul_rn(dt, vu[u][e]));
            st8_nt<T>(x_e + i, x[u]);
        }
    }
}

// same storage type on both sides: a plain copy in 16-byte pieces; every workgroup owns one contiguous range and every
// thread requests U pieces before it stores the first (non-temporal on both sides: the data is streamed once)
typedef unsigned int copy_u32x4 __attribute__((ext_vector_type(4)));
template <int U, int THREADS>
__global__ void __launch_bounds__(THREADS) copy16_chunk_kernel(const copy_u32x4* __restrict__ src, copy_u32x4* __restrict__ dst, int64_t n16) {
    const int64_t per = (n16 + gridDim.x - 1) / gridDim.x;
    const int64_t begin = blockIdx.x * per;
    int64_t end = begin + per; end = end < n16 ? end : n16;
    int64_t i = begin + threadIdx.x;
    for (; i + (U - 1) * THREADS < end; i += U * THREADS) {
        copy_u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + i + u * THREADS);
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_nontemporal_store(v[u], dst + i + u * THREADS);
    }
    for (; i < end; i += THREADS) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// the same for 16-byte aligned tensors, eight elements per thread and step (n8 groups of eight)
template <typename S, typename D>
__global__ void __launch_bounds__(kThreads) cast8_kernel(const S* __restrict__ src, D* __restrict__ dst, int64_t n8) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; g < n8; g += stride) {
        float v[8];
        ld8<S>(src + g * 8, v);
        if constexpr (sizeof(D) == 2) {
            ln_bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(v[e]);
            *reinterpret_cast<ln_bf16x8*>(dst + g * 8) = o;
        } else {
            *reinterpret_cast<ln_f32x4*>(dst + g * 8) = ln_f32x4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<ln_f32x4*>(dst + g * 8 + 4) = ln_f32x4{v[4], v[5], v[6], v[7]};
        }
    }
}

}  // namespace

extern "C" int regione_gather(regione_ctx* ctx, const void* src, int32_t row_elems, int32_t dtype,
                              const int32_t* index, const int32_t* n_dev, int64_t n_max, void* dst) {
    return rows_by_index<true>(ctx, src, dst, row_elems, dtype, index, n_dev, n_max, "gather");
}

extern "C" int regione_scatter(regione_ctx* ctx, void* dst_full, int32_t row_elems, int32_t dtype,
                               const int32_t* index, const int32_t* n_dev, int64_t n_max, const void* src) {
    return rows_by_index<false>(ctx, src, dst_full, row_elems, dtype, index, n_dev, n_max, "scatter");
}

int rg_gather_pair_slots(regione_ctx* ctx, const void* src_a, int32_t row_elems_a, int32_t dtype_a, void* dst_a, const void* src_b, int32_t row_elems_b, int32_t dtype_b, void* dst_b,
                         const int32_t* index, const int32_t* n_dev, int64_t n_max, int32_t* slots, int n_txt) {
    return rows_pair<true>(ctx, src_a, dst_a, row_elems_a, dtype_a, src_b, dst_b, row_elems_b, dtype_b, index, n_dev, n_max, "gather_pair", FreshSlots{slots, n_txt});
}

extern "C" int regione_gather_pair(regione_ctx* ctx, const void* src_a, int32_t row_elems_a, int32_t dtype_a, void* dst_a,
                                   const void* src_b, int32_t row_elems_b, int32_t dtype_b, void* dst_b,
                                   const int32_t* index, const int32_t* n_dev, int64_t n_max) {
    return rows_pair<true>(ctx, src_a, dst_a, row_elems_a, dtype_a, src_b, dst_b, row_elems_b, dtype_b, index, n_dev, n_max, "gather_pair");
}

extern "C" int regione_scatter_pair(regione_ctx* ctx, void* dst_full_a, int32_t row_elems_a, int32_t dtype_a, const void* src_a,
                                    void* dst_full_b, int32_t row_elems_b, int32_t dtype_b, const void* src_b,
                                    const int32_t* index, const int32_t* n_dev, int64_t n_max) {
    return rows_pair<false>(ctx, src_a, dst_full_a, row_elems_a, dtype_a, src_b, dst_full_b, row_elems_b, dtype_b, index, n_dev, n_max, "scatter_pair");
}

extern "C" int regione_velocity_cache(regione_ctx* ctx, int32_t reuse, float factor, float dt,
                                      const void* v_fresh_opt, void* c_a, void* v_out_opt, void* x_e,
                                      const int32_t* n_dev, int64_t n_max, int32_t c, int32_t dtype) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "velocity_cache: null context");
    if (c <= 0 || n_max < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "velocity_cache: c=%d n_max=%lld", c, (long long)n_max);
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "velocity_cache: bad dtype %d", dtype);
    if (n_max == 0) return REGIONE_OK;
    if (!c_a || !x_e) RG_FAIL(REGIONE_ERR_INVALID_ARG, "velocity_cache: null c_a or x_e");
    if (!reuse && !v_fresh_opt) RG_FAIL(REGIONE_ERR_INVALID_ARG, "velocity_cache: a fresh step needs v_fresh");
    const int64_t total = n_max * c;
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    const bool wide = (c % 8 == 0) && rg_aligned16(c_a) && rg_aligned16(x_e) && (!v_fresh_opt || rg_aligned16(v_fresh_opt)) &&
                      (!v_out_opt || rg_aligned16(v_out_opt));
    if (wide) {
        int64_t vb = (total / 8 + kThreads - 1) / kThreads;
        if (vb > 256 * 32) vb = 256 * 32;
        const dim3 vgrid(static_cast<unsigned>(vb));
        if (dtype == REGIONE_BF16)
            hipLaunchKernelGGL(velocity_cache_vec_kernel<bf16_t>, vgrid, dim3(kThreads), 0, ctx->stream, reuse, factor, dt,
                               static_cast<const bf16_t*>(v_fresh_opt), static_cast<bf16_t*>(c_a), static_cast<bf16_t*>(v_out_opt),
                               static_cast<bf16_t*>(x_e), n_dev, n_max, c);
        else
            hipLaunchKernelGGL(velocity_cache_vec_kernel<float>, vgrid, dim3(kThreads), 0, ctx->stream, reuse, factor, dt,
                               static_cast<const float*>(v_fresh_opt), static_cast<float*>(c_a), static_cast<float*>(v_out_opt),
                               static_cast<float*>(x_e), n_dev, n_max, c);
        RG_LAUNCH_CHECK();
        return REGIONE_OK;
    }
    int64_t blocks = (total + kThreads - 1) / kThreads;
    if (blocks > 256 * 32) blocks = 256 * 32;
    dim3 grid(static_cast<unsigned>(blocks));
    if (dtype == REGIONE_BF16)
        hipLaunchKernelGGL(velocity_cache_kernel<bf16_t>, grid, dim3(kThreads), 0, ctx->stream, reuse, factor, dt,
                           static_cast<const bf16_t*>(v_fresh_opt), static_cast<bf16_t*>(c_a), static_cast<bf16_t*>(v_out_opt),
                           static_cast<bf16_t*>(x_e), n_dev, n_max, c);
    else
        hipLaunchKernelGGL(velocity_cache_kernel<float>, grid, dim3(kThreads), 0, ctx->stream, reuse, factor, dt,
                           static_cast<const float*>(v_fresh_opt), static_cast<float*>(c_a), static_cast<float*>(v_out_opt),
                           static_cast<float*>(x_e), n_dev, n_max, c);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

// ---- one-step estimate of listed rows in place (Eq.5): the unedited rows' jump to the end of a segment, written where the
// merge would put it, so that neither a gather before it nor a scatter after it is needed
namespace {
template <typename T, int VEC>
__global__ void __launch_bounds__(kThreads)
euler_rows_kernel(T* __restrict__ x_full, const T* __restrict__ v_full, const int32_t* __restrict__ index,
                  const int32_t* __restrict__ n_dev, int64_t n_max, int c, float dt) {
    int64_t n = n_max;
    if (n_dev) { const int64_t nd = *n_dev; n = nd < n_max ? (nd < 0 ? 0 : nd) : n_max; }
    const int groups = c / VEC;                 // pieces of VEC elements per row
    const int64_t total = n * groups;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t u = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; u < total; u += stride) {
        const int64_t row = u / groups;
        const int g = static_cast<int>(u - row * groups);
        const int64_t at = static_cast<int64_t>(index[row]) * c + g * VEC;
        if constexpr (VEC == 8) {
            float x[8], v[8];
            ld8<T>(x_full + at, x); ld8<T>(v_full + at, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = __fsub_rn(x[e], __fmul_rn(dt, v[e]));   // product and difference rounded separately, as in Eq.4's kernel
            st8<T>(x_full + at, x);
        } else {
            st<T>(x_full + at, __fsub_rn(ld<T>(x_full + at), __fmul_rn(dt, ld<T>(v_full + at))));
        }
    }
}
}  // namespace

extern "C" int regione_euler_rows(regione_ctx* ctx, void* x_full, const void* v_full, const int32_t* index, const int32_t* n_dev,
                                  int64_t n_max, int32_t c, int32_t dtype, float dt) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "euler_rows: null context");
    if (c <= 0 || n_max < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "euler_rows: c=%d n_max=%lld", c, (long long)n_max);
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "euler_rows: bad dtype %d", dtype);
    if (n_max == 0) return REGIONE_OK;
    if (!x_full || !v_full || !index) RG_FAIL(REGIONE_ERR_INVALID_ARG, "euler_rows: null tensor");
    if (x_full == v_full) RG_FAIL(REGIONE_ERR_INVALID_ARG, "euler_rows: x and v are the same tensor");
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    const bool wide = (c % 8 == 0) && rg_aligned16(x_full) && rg_aligned16(v_full);
    const int64_t total = n_max * (wide ? c / 8 : c);
    int64_t blocks = (total + kThreads - 1) / kThreads;
    if (blocks > 256 * 32) blocks = 256 * 32;
    const dim3 grid(static_cast<unsigned>(blocks));
#define RG_EULER(T, V) hipLaunchKernelGGL((euler_rows_kernel<T, V>), grid, dim3(kThreads), 0, ctx->stream, static_cast<T*>(x_full), static_cast<const T*>(v_full), index, n_dev, n_max, c, dt)
    if (dtype == REGIONE_BF16) { if (wide) RG_EULER(bf16_t, 8); else RG_EULER(bf16_t, 1); }
    else { if (wide) RG_EULER(float, 8); else RG_EULER(float, 1); }
#undef RG_EULER
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

extern "C" int regione_cast(regione_ctx* ctx, const void* src, int32_t src_dtype, void* dst, int32_t dst_dtype, int64_t n_elems) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "cast: null context");
    if ((src_dtype != REGIONE_BF16 && src_dtype != REGIONE_FP32) || (dst_dtype != REGIONE_BF16 && dst_dtype != REGIONE_FP32))
        RG_FAIL(REGIONE_ERR_INVALID_ARG, "cast: bad dtype %d -> %d", src_dtype, dst_dtype);
    if (n_elems < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "cast: n_elems=%lld", (long long)n_elems);
    if (n_elems == 0) return REGIONE_OK;
    if (!src || !dst) RG_FAIL(REGIONE_ERR_INVALID_ARG, "cast: null tensor");
    ProfScope prof(ctx, REGIONE_PROF_ROWS);
    const size_t src_elem = src_dtype == REGIONE_FP32 ? 4 : 2, dst_elem = dst_dtype == REGIONE_FP32 ? 4 : 2;
    auto grid_for = [](int64_t items) { int64_t b = (items + kThreads - 1) / kThreads; return dim3(static_cast<unsigned>(b > 256 * 32 ? 256 * 32 : b)); };
    // aligned tensors: everything but a tail of fewer than eight elements goes through the wide kernels
    int64_t done = 0;
    if (rg_aligned16(src) && rg_aligned16(dst) && n_elems >= 8) {
        const int64_t n8 = n_elems / 8;
        if (src_dtype == dst_dtype) {
            const int64_t n16 = n8 * 8 * static_cast<int64_t>(src_elem) / 16;
            // few, long-running workgroups (eight per CU): each thread keeps four 16-byte requests in flight
            // one long-running workgroup of 1024 threads per CU, each on a contiguous range, eight requests in flight per
            // thread: 5.9 TB/s on a 1 GiB copy; the same with the ranges interleaved (grid stride) 5.4-5.6, 2048 workgroups
            // of four requests per thread 4.4, one request per thread 5.0-5.2 - all measured in one process (the HIP
            // runtime's copy kernel: 6.1 TB/s in a kernel trace)
            constexpr int U = 8, THREADS = 1024;
            int64_t b = (n16 + U * THREADS - 1) / (U * THREADS);
            if (b > 256) b = 256;
            hipLaunchKernelGGL((copy16_chunk_kernel<U, THREADS>), dim3(static_cast<unsigned>(b)), dim3(THREADS), 0, ctx->stream,
                               static_cast<const copy_u32x4*>(src), static_cast<copy_u32x4*>(dst), n16);
        } else if (src_dtype == REGIONE_FP32) {
            hipLaunchKernelGGL((cast8_kernel<float, bf16_t>), grid_for(n8), dim3(kThreads), 0, ctx->stream, static_cast<const float*>(src), static_cast<bf16_t*>(dst), n8);
        } else {
            hipLaunchKernelGGL((cast8_kernel<bf16_t, float>), grid_for(n8), dim3(kThreads), 0, ctx->stream, static_cast<const bf16_t*>(src), static_cast<float*>(dst), n8);
        }
        RG_LAUNCH_CHECK();
        done = n8 * 8;
        if (done == n_elems) return REGIONE_OK;
    }
    const int64_t rest = n_elems - done;
    const void* s2 = static_cast<const char*>(src) + done * src_elem;
    void* d2 = static_cast<char*>(dst) + done * dst_elem;
    const dim3 grid = grid_for(rest);
    if (src_dtype == REGIONE_FP32 && dst_dtype == REGIONE_BF16)
        hipLaunchKernelGGL((cast_kernel<float, bf16_t>), grid, dim3(kThreads), 0, ctx->stream, static_cast<const float*>(s2), static_cast<bf16_t*>(d2), rest);
    else if (src_dtype == REGIONE_BF16 && dst_dtype == REGIONE_FP32)
        hipLaunchKernelGGL((cast_kernel<bf16_t, float>), grid, dim3(kThreads), 0, ctx->stream, static_cast<const bf16_t*>(s2), static_cast<float*>(d2), rest);
    else if (src_dtype == REGIONE_FP32)
        hipLaunchKernelGGL((cast_kernel<float, float>), grid, dim3(kThreads), 0, ctx->stream, static_cast<const float*>(s2), static_cast<float*>(d2), rest);
    else
        hipLaunchKernelGGL((cast_kernel<bf16_t, bf16_t>), grid, dim3(kThreads), 0, ctx->stream, static_cast<const bf16_t*>(s2), static_cast<bf16_t*>(d2), rest);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

template <typename T, typename U>
static void launch_layernorm(regione_ctx* ctx, const T* h, int n, int hidden, const float* shift, const float* scale, U* u, bool keep_sums) {
    const dim3 grid((n + kThreads / 64 - 1) / (kThreads / 64));
    const bool vec = (hidden % 8 == 0) && hidden <= 64 * 8 * 8 && rg_aligned16(h) && rg_aligned16(u) &&
                     (!shift || rg_aligned16(shift)) && (!scale || rg_aligned16(scale));
    // as many registers and as much code as the row has rounds of 512 elements
    if (vec && hidden <= 512) hipLaunchKernelGGL((layernorm_mod_vec_kernel<T, U, 1>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
    else if (vec && hidden <= 1024) hipLaunchKernelGGL((layernorm_mod_vec_kernel<T, U, 2>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
    else if (vec && keep_sums) {
        if (hidden <= 2048) hipLaunchKernelGGL((layernorm_mod_vec_kernel<T, U, 4>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
        else if (hidden <= 3072) hipLaunchKernelGGL((layernorm_mod_vec_kernel<T, U, 6>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
        else hipLaunchKernelGGL((layernorm_mod_vec_kernel<T, U, 8>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
    } else if (vec) {
#define RG_LN_WIDE(W) case W: hipLaunchKernelGGL((layernorm_mod_wide_kernel<T, U, W>), dim3(n < ln_wide_grid(W) ? n : ln_wide_grid(W)), dim3(64 * W), 0, ctx->stream, h, n, hidden, shift, scale, u); break;
        switch ((hidden / 8 + 63) / 64) { RG_LN_WIDE(3) RG_LN_WIDE(4) RG_LN_WIDE(5) RG_LN_WIDE(6) RG_LN_WIDE(7) RG_LN_WIDE(8) }
#undef RG_LN_WIDE
    }
    else hipLaunchKernelGGL((layernorm_mod_kernel<T, U>), grid, dim3(kThreads), 0, ctx->stream, h, n, hidden, shift, scale, u);
}

int rg_layernorm_mod(regione_ctx* ctx, const void* h, int h_f32, int n, int hidden, const float* shift, const float* scale, void* u, bool keep_sums) {
    if (n <= 0) return REGIONE_OK;
    ProfScope prof(ctx, REGIONE_PROF_LAYERNORM);
    if (ctx->f32 && h_f32) launch_layernorm(ctx, static_cast<const float*>(h), n, hidden, shift, scale, static_cast<float*>(u), keep_sums);
    else if (ctx->f32) launch_layernorm(ctx, static_cast<const bf16_t*>(h), n, hidden, shift, scale, static_cast<float*>(u), keep_sums);
    else if (h_f32) launch_layernorm(ctx, static_cast<const float*>(h), n, hidden, shift, scale, static_cast<bf16_t*>(u), keep_sums);
    else launch_layernorm(ctx, static_cast<const bf16_t*>(h), n, hidden, shift, scale, static_cast<bf16_t*>(u), keep_sums);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

bool rg_gather_layernorm_ok(const void* h_full, const void* h_rows, const void* u, const float* shift, const float* scale, const void* x_t, const void* x_e, int hidden, int64_t x_row_bytes) {
    return hidden > 1024 && hidden <= 4096 && hidden % 8 == 0 && x_row_bytes > 0 && x_row_bytes % 16 == 0 && rg_aligned16(h_full) && rg_aligned16(h_rows) && rg_aligned16(u) &&
           rg_aligned16(shift) && rg_aligned16(scale) && rg_aligned16(x_t) && rg_aligned16(x_e);
}
template <typename T, typename U>
static void launch_gather_layernorm(regione_ctx* ctx, const void* h_full, const int32_t* index, int n, int hidden, const float* shift, const float* scale, void* h_rows, void* u,
                                    const void* x_t, void* x_e, int x_pieces, FreshSlots fresh) {
#define RG_LN_WIDE(W) case W: hipLaunchKernelGGL((gather_layernorm_kernel<T, U, W>), dim3(n < ln_wide_grid(W) ? n : ln_wide_grid(W)), dim3(64 * W), 0, ctx->stream, \
        static_cast<const T*>(h_full), index, n, hidden, shift, scale, static_cast<T*>(h_rows), static_cast<U*>(u), static_cast<const rows_u32x4*>(x_t), static_cast<rows_u32x4*>(x_e), x_pieces, fresh); break;
    switch ((hidden / 8 + 63) / 64) { RG_LN_WIDE(3) RG_LN_WIDE(4) RG_LN_WIDE(5) RG_LN_WIDE(6) RG_LN_WIDE(7) RG_LN_WIDE(8) }
#undef RG_LN_WIDE
}
int rg_gather_layernorm(regione_ctx* ctx, const void* h_full, int h_f32, const int32_t* index, int n, int hidden, const float* shift, const float* scale, void* h_rows, void* u,
                        const void* x_t, void* x_e, int x_pieces, int32_t* slots, int n_txt) {
    if (n <= 0) return REGIONE_OK;
    const FreshSlots fresh = {slots, n_txt};
    ProfScope prof(ctx, REGIONE_PROF_LAYERNORM);
    if (ctx->f32) launch_gather_layernorm<float, float>(ctx, h_full, index, n, hidden, shift, scale, h_rows, u, x_t, x_e, x_pieces, fresh);
    else if (h_f32) launch_gather_layernorm<float, bf16_t>(ctx, h_full, index, n, hidden, shift, scale, h_rows, u, x_t, x_e, x_pieces, fresh);
    else launch_gather_layernorm<bf16_t, bf16_t>(ctx, h_full, index, n, hidden, shift, scale, h_rows, u, x_t, x_e, x_pieces, fresh);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

namespace {
// The velocity step of a fresh head (Eq.9, Eq.4: the arithmetic of velocity_cache_vec_kernel) with the merge of the updated latent rows, and in workgroups of their own
// the merge of the hidden rows: three launches of a few microseconds in one.
template <typename T>
__global__ void __launch_bounds__(kThreads)
velocity_merge_kernel(const T* v, T* c_a, T* __restrict__ x_e, T* __restrict__ x_full, const int32_t* __restrict__ index, float dt, int groups, int c, int step_wgs, RowMerge merge) {
    if (static_cast<int>(blockIdx.x) < step_wgs) {
        const int g = blockIdx.x * kThreads + threadIdx.x;
        if (g >= groups) return;
        const int per_row = c / 8, row = g / per_row;
        const int64_t i = static_cast<int64_t>(g) * 8;
        const int64_t to = static_cast<int64_t>(index[row]) * c + (g - row * per_row) * 8;
        float vu[8], x[8];
        ld8<T>(v + i, vu);
        ld8<T>(x_e + i, x);
        if (c_a != v) st8<T>(c_a + i, vu);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = __fsub_rn(x[e], __fmul_rn(dt, vu[e]));
        st8<T>(x_e + i, x);
        st8<T>(x_full + to, x);
        return;
    }
    const unsigned total = static_cast<unsigned>(merge.rows) * static_cast<unsigned>(merge.pieces), stride = (gridDim.x - step_wgs) * kThreads;
    for (unsigned u = (blockIdx.x - step_wgs) * kThreads + threadIdx.x; u < total; u += stride) {
        const unsigned row = u / static_cast<unsigned>(merge.pieces);
        static_cast<rows_u32x4*>(merge.dst)[static_cast<int64_t>(merge.index[row]) * merge.pieces + (u - row * merge.pieces)] = static_cast<const rows_u32x4*>(merge.src)[u];
    }
}
}  // namespace

int rg_velocity_merge(regione_ctx* ctx, const void* v, void* c_a, void* x_e, void* x_full, const int32_t* index, float dt, int n, int c, int dtype, const RowMerge& merge) {
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    const int groups = n * c / 8, step_wgs = (groups + kThreads - 1) / kThreads;
    int64_t wgs = (static_cast<int64_t>(merge.rows) * merge.pieces + kThreads - 1) / kThreads;
    if (wgs > 256 * 32) wgs = 256 * 32;
    const dim3 grid(static_cast<unsigned>(step_wgs + wgs));
    if (dtype == REGIONE_BF16)
        hipLaunchKernelGGL(velocity_merge_kernel<bf16_t>, grid, dim3(kThreads), 0, ctx->stream, static_cast<const bf16_t*>(v), static_cast<bf16_t*>(c_a), static_cast<bf16_t*>(x_e),
                           static_cast<bf16_t*>(x_full), index, dt, groups, c, step_wgs, merge);
    else
        hipLaunchKernelGGL(velocity_merge_kernel<float>, grid, dim3(kThreads), 0, ctx->stream, static_cast<const float*>(v), static_cast<float*>(c_a), static_cast<float*>(x_e),
                           static_cast<float*>(x_full), index, dt, groups, c, step_wgs, merge);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

// ---- squared norms of velocity vectors: the data the timestep-aware factor of Eq.7 is fitted on
namespace {

// One workgroup per vector.  Squares and sums in float64; the order of the sums is fixed by the launch shape, so
// the result is reproducible.
template <typename T>
__global__ void __launch_bounds__(kThreads)
sq_norms_kernel(const T* __restrict__ x, int64_t vec_elems, double* __restrict__ out) {
    const T* v = x + static_cast<int64_t>(blockIdx.x) * vec_elems;
    double acc = 0.0;
    const int64_t groups = vec_elems >> 3;
    for (int64_t g = threadIdx.x; g < groups; g += kThreads) {
        float e[8];
        ld8<T>(v + g * 8, e);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fma(static_cast<double>(e[i]), static_cast<double>(e[i]), acc);
    }
    for (int64_t i = (groups << 3) + threadIdx.x; i < vec_elems; i += kThreads) {
        float f;
        if constexpr (sizeof(T) == 2) f = bf16_to_f32(v[i]); else f = v[i];
        acc = fma(static_cast<double>(f), static_cast<double>(f), acc);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    __shared__ double part[kThreads / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) s += part[w];
        out[blockIdx.x] = s;
    }
}

}  // namespace

extern "C" int regione_sq_norms(regione_ctx* ctx, const void* x, int32_t dtype, int64_t n_vectors, int64_t vec_elems, double* out) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "sq_norms: null context");
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "sq_norms: bad dtype %d", dtype);
    if (n_vectors < 0 || vec_elems < 0 || n_vectors > INT32_MAX) RG_FAIL(REGIONE_ERR_INVALID_ARG, "sq_norms: n_vectors=%lld vec_elems=%lld", static_cast<long long>(n_vectors), static_cast<long long>(vec_elems));
    if (n_vectors == 0) return REGIONE_OK;
    if (!out || (!x && vec_elems > 0)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "sq_norms: null operand");
    const size_t elem = dtype == REGIONE_BF16 ? 2 : 4;
    if (!rg_aligned16(x) || (vec_elems * elem) % 16) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "sq_norms: vectors must start 16-byte aligned");
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    if (dtype == REGIONE_BF16) hipLaunchKernelGGL(sq_norms_kernel<bf16_t>, dim3(static_cast<unsigned>(n_vectors)), dim3(kThreads), 0, ctx->stream, static_cast<const bf16_t*>(x), vec_elems, out);
    else hipLaunchKernelGGL(sq_norms_kernel<float>, dim3(static_cast<unsigned>(n_vectors)), dim3(kThreads), 0, ctx->stream, static_cast<const float*>(x), vec_elems, out);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

// ---- classifier-free guidance: the velocity the sampler uses is v_uncond + scale * (v_cond - v_uncond)
namespace {
template <typename T>
__global__ void __launch_bounds__(kThreads)
guidance_combine_kernel(const T* __restrict__ vc, const T* __restrict__ vu, float scale, T* __restrict__ out, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride) {
        float c, u;
        if constexpr (sizeof(T) == 2) { c = bf16_to_f32(vc[i]); u = bf16_to_f32(vu[i]); } else { c = vc[i]; u = vu[i]; }
        const float r = u + scale * (c - u);
        if constexpr (sizeof(T) == 2) out[i] = f32_to_bf16(r); else out[i] = r;
    }
}
}  // namespace

extern "C" int regione_guidance_combine(regione_ctx* ctx, const void* v_cond, const void* v_uncond, float scale, void* out,
                                        int64_t n_elems, int32_t dtype) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "guidance_combine: null context");
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "guidance_combine: bad dtype %d", dtype);
    if (n_elems < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "guidance_combine: n_elems=%lld", static_cast<long long>(n_elems));
    if (n_elems == 0) return REGIONE_OK;
    if (!v_cond || !v_uncond || !out) RG_FAIL(REGIONE_ERR_INVALID_ARG, "guidance_combine: null operand");
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    int64_t blocks = (n_elems + kThreads - 1) / kThreads;
    if (blocks > 256 * 16) blocks = 256 * 16;
    if (dtype == REGIONE_BF16)
        hipLaunchKernelGGL(guidance_combine_kernel<bf16_t>, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, ctx->stream,
                           static_cast<const bf16_t*>(v_cond), static_cast<const bf16_t*>(v_uncond), scale, static_cast<bf16_t*>(out), n_elems);
    else
        hipLaunchKernelGGL(guidance_combine_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, ctx->stream,
                           static_cast<const float*>(v_cond), static_cast<const float*>(v_uncond), scale, static_cast<float*>(out), n_elems);
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

// ---- relative change of two velocities: the sums behind |a - b|_2 / |b|_2 (a data-dependent reuse trigger that a
// benchmark description asks for beside the paper's schedule-only criterion of Eq.8)
namespace {
template <typename T>
__global__ void __launch_bounds__(1024)
rel_change_kernel(const T* __restrict__ a, const T* __restrict__ b, int64_t n, double* __restrict__ out) {
    double sd = 0.0, sb = 0.0;                       // one workgroup: the order of the sums is fixed
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
        float x, y;
        if constexpr (sizeof(T) == 2) { x = bf16_to_f32(a[i]); y = bf16_to_f32(b[i]); } else { x = a[i]; y = b[i]; }
        const double d = static_cast<double>(x) - static_cast<double>(y);
        sd = fma(d, d, sd);
        sb = fma(static_cast<double>(y), static_cast<double>(y), sb);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) { sd += __shfl_xor(sd, m, 64); sb += __shfl_xor(sb, m, 64); }
    __shared__ double part[2][16];
    if ((threadIdx.x & 63) == 0) { part[0][threadIdx.x >> 6] = sd; part[1][threadIdx.x >> 6] = sb; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) { s0 += part[0][w]; s1 += part[1][w]; }
        out[0] = s0;
        out[1] = s1;
    }
}
}  // namespace

extern "C" int regione_rel_change(regione_ctx* ctx, const void* v_new, const void* v_old, int64_t n_elems, int32_t dtype, double* out,
                                  double* out_host_opt) {
    if (!ctx || !out) RG_FAIL(REGIONE_ERR_INVALID_ARG, "rel_change: null context or output");
    if (dtype != REGIONE_BF16 && dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "rel_change: bad dtype %d", dtype);
    if (n_elems < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "rel_change: n_elems=%lld", static_cast<long long>(n_elems));
    if (n_elems > 0 && (!v_new || !v_old)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "rel_change: null operand");
    ProfScope prof(ctx, REGIONE_PROF_VELOCITY);
    if (dtype == REGIONE_BF16)
        hipLaunchKernelGGL(rel_change_kernel<bf16_t>, dim3(1), dim3(1024), 0, ctx->stream, static_cast<const bf16_t*>(v_new), static_cast<const bf16_t*>(v_old), n_elems, out);
    else
        hipLaunchKernelGGL(rel_change_kernel<float>, dim3(1), dim3(1024), 0, ctx->stream, static_cast<const float*>(v_new), static_cast<const float*>(v_old), n_elems, out);
    RG_LAUNCH_CHECK();
    if (out_host_opt) {   // the decision is taken on the host: 16 bytes back, after the stream has caught up
        RG_HIP(hipMemcpyAsync(out_host_opt, out, 2 * sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
        RG_HIP(hipStreamSynchronize(ctx->stream));
    }
    return REGIONE_OK;
}
