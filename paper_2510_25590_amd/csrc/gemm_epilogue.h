// Epilogues of the matrix-core GEMM kernels: what happens to a wave's accumulators once the sum over K is complete, and
// the order in which a launch's workgroups visit the tiles of the result.
#pragma once
#include "common.h"
#include <math.h>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // a native 16-byte vector: copies are single loads/stores
typedef __attribute__((ext_vector_type(8))) int i32x8;            // operand of the 8-bit MFMA: 32 E4M3 values per lane

// 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3).  Both sides of the quotient are divided by four, so that the divisor, in [1/4, inf], has a normal
// reciprocal up to where the exponential overflows; then the reciprocal, one correction of the quotient and the fix-up of the special values give what the general division gives (but for
// the last bit of |x| < 2^-124), without its scaling and with fewer instructions: the epilogue of 820 x 12288 results is bound by them (one tile per CU, 96 values per thread); the whole
// product, K 3072, 68.0 -> 65.5 us in a kernel trace.  Without the factor, which costs a call 0.1 to 0.6 % (20 % edited 342.1 -> 343.0 us), results between 4e-38 and
// 1.6e-37 (x = -13) came out as zero.
__device__ __forceinline__ float gelu_tanh_f32(float x) {
    constexpr float kLin = -2.0f * 0.7978845608028654f * 1.4426950408889634f, kCub = kLin * 0.044715f;   // -2u log2(e) = x (kLin + kCub x^2)
    const float e = __builtin_amdgcn_exp2f(x * __builtin_fmaf(x * x, kCub, kLin));
    const float n = 0.25f * x, d = __builtin_fmaf(0.25f, e, 0.25f);
    const float r = __builtin_amdgcn_rcpf(d);
    float q = n * r;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, n), r, q);
    return __builtin_amdgcn_div_fixupf(q, d, n);
}

// Row of the key/value destination for output row `row` (its cache slot when a slot list is given).
template <int KIND>
__device__ __forceinline__ int64_t epilogue_kv_row(const GemmEpilogue& ep, int row) {
    return KIND == EPI_QKV ? epilogue_slot(ep, row) : row;
}

template <int KIND>
__device__ __forceinline__ void epilogue_store(const GemmEpilogue& ep, int row, int64_t kv_row, int col, float acc, float bias, float gate) {
    float val = acc + bias;
    if (KIND == EPI_PLAIN) {
        if (ep.act == REGIONE_ACT_GELU_TANH && col >= ep.act_from) val = gelu_tanh_f32(val);
        const int64_t o = static_cast<int64_t>(row) * ep.ldy + col;
        if (ep.y_f32) static_cast<float*>(ep.y)[o] = val;
        else static_cast<bf16_t*>(ep.y)[o] = f32_to_bf16(val);
    } else if (KIND == EPI_QKV) {
        const int H = ep.hidden;
        if (col < H) {
            ep.q[static_cast<int64_t>(row) * ep.ldq + col] = f32_to_bf16(val);
        } else if (col < 3 * H) {
            if (col < 2 * H) ep.k[kv_row * ep.ldkv + (col - H)] = f32_to_bf16(val);
            else ep.v[kv_row * ep.ldkv + (col - 2 * H)] = f32_to_bf16(val);
        } else {
            if (ep.act == REGIONE_ACT_GELU_TANH) val = gelu_tanh_f32(val);
            static_cast<bf16_t*>(ep.y)[static_cast<int64_t>(row) * ep.ldy + ep.y_col0 + (col - 3 * H)] = f32_to_bf16(val);
        }
    } else if (KIND == EPI_VELOCITY) {
        // the velocity in its storage type, the cache takes it (Eq.9, fresh branch), the Euler update (Eq.4) with the
        // product and the difference rounded separately, and the row written where the merge by position puts it
        const int64_t o = static_cast<int64_t>(row) * ep.ldy + col;
        const int64_t full = ep.vel_index ? static_cast<int64_t>(ep.vel_index[row]) * ep.ldy + col : o;
        if (ep.y_f32) {
            if (ep.y) static_cast<float*>(ep.y)[o] = val;
            static_cast<float*>(ep.vel_ca)[o] = val;
            const float x = __fsub_rn(static_cast<float*>(ep.vel_xe)[o], __fmul_rn(ep.vel_dt, val));
            static_cast<float*>(ep.vel_xe)[o] = x;
            if (ep.vel_xfull) static_cast<float*>(ep.vel_xfull)[full] = x;
        } else {
            const bf16_t vb = f32_to_bf16(val);
            const float v = bf16_to_f32(vb);
            if (ep.y) static_cast<bf16_t*>(ep.y)[o] = vb;
            static_cast<bf16_t*>(ep.vel_ca)[o] = vb;
            const bf16_t xb = f32_to_bf16(__fsub_rn(bf16_to_f32(static_cast<bf16_t*>(ep.vel_xe)[o]), __fmul_rn(ep.vel_dt, v)));
            static_cast<bf16_t*>(ep.vel_xe)[o] = xb;
            if (ep.vel_xfull) static_cast<bf16_t*>(ep.vel_xfull)[full] = xb;
        }
    } else {  // EPI_RESID
        const int64_t ri = static_cast<int64_t>(row) * ep.ldr + col;
        const float res = ep.resid_f32 ? static_cast<const float*>(ep.resid)[ri] : bf16_to_f32(static_cast<const bf16_t*>(ep.resid)[ri]);
        val = res + gate * val;
        const int64_t o = static_cast<int64_t>(row) * ep.ldy + col;
        if (ep.y_f32) static_cast<float*>(ep.y)[o] = val;
        else static_cast<bf16_t*>(ep.y)[o] = f32_to_bf16(val);
    }
}

// eight consecutive elements: 32 bytes (float32) or 16 (bf16), of which only an element's own alignment is promised unless ALIGNED
template <bool ALIGNED> struct Pieces { typedef f32x4 f32; typedef bf16x8 b16; };
template <> struct Pieces<false> {
    typedef f32x4 __attribute__((aligned(4))) f32;
    typedef bf16x8 __attribute__((aligned(2))) b16;
};
template <bool ALIGNED>
__device__ __forceinline__ void store8(void* base, int64_t elem, int as_f32, const float (&v)[8]) {
    if (as_f32) {
        typedef typename Pieces<ALIGNED>::f32 piece;
        float* p = static_cast<float*>(base) + elem;
        *reinterpret_cast<piece*>(p) = f32x4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<piece*>(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
    } else {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(v[e]);
        *reinterpret_cast<typename Pieces<ALIGNED>::b16*>(static_cast<bf16_t*>(base) + elem) = o;
    }
}

// Eight elements of a row as they lie in memory: float32 fills both halves, bf16 the first.  Kept raw between the load and the use, so that a conversion
// does not wait for the load.
struct Raw8 { u32x4 a, b; };
template <bool ALIGNED>
__device__ __forceinline__ Raw8 load_raw8(const void* base, int64_t elem, int as_f32) {
    Raw8 r;
    if (as_f32) {
        typedef typename Pieces<ALIGNED>::f32 piece;
        const float* p = static_cast<const float*>(base) + elem;
        r.a = __builtin_bit_cast(u32x4, static_cast<f32x4>(*reinterpret_cast<const piece*>(p)));
        r.b = __builtin_bit_cast(u32x4, static_cast<f32x4>(*reinterpret_cast<const piece*>(p + 4)));
    } else {
        r.a = __builtin_bit_cast(u32x4, static_cast<bf16x8>(*reinterpret_cast<const typename Pieces<ALIGNED>::b16*>(static_cast<const bf16_t*>(base) + elem)));
        r.b = u32x4{0u, 0u, 0u, 0u};
    }
    return r;
}
__device__ __forceinline__ void raw_values(const Raw8& r, int as_f32, float (&v)[8]) {
    if (as_f32) {
        const f32x4 a = __builtin_bit_cast(f32x4, r.a), b = __builtin_bit_cast(f32x4, r.b);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
    } else {
        const bf16x8 a = __builtin_bit_cast(bf16x8, r.a);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = static_cast<float>(a[e]);
    }
}

// What an epilogue reads besides the sums, in three parts that can be requested ahead of their use: of eight columns, of a row, and of eight elements.
template <int KIND, bool SCALED> struct EpiColumns {
    float bias[8], gate[KIND == EPI_RESID ? 8 : 1], scale[SCALED ? 8 : 1];
    __device__ __forceinline__ void load(const GemmEpilogue& ep, int col0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bias[e] = ep.bias ? ep.bias[col0 + e] : 0.f;
            if (KIND == EPI_RESID) gate[e] = ep.gate ? ep.gate[col0 + e] : 1.f;
            if (SCALED) scale[e] = ep.col_scale[col0 + e];
        }
    }
};
template <int KIND, bool SCALED> struct EpiRow {
    int32_t place;      // cache slot (QKV) or row of the full latent (velocity step)
    float scale;
    __device__ __forceinline__ void load(const GemmEpilogue& ep, int row) {
        place = row;
        if (KIND == EPI_QKV) place = epilogue_slot(ep, row);
        if (KIND == EPI_VELOCITY && ep.vel_index) place = ep.vel_index[row];
        scale = SCALED ? ep.row_scale[row] : 1.f;
    }
};
template <int KIND> constexpr bool epi_reads() { return KIND == EPI_RESID || KIND == EPI_VELOCITY; }
template <int KIND, bool ALIGNED>
__device__ __forceinline__ Raw8 epi_load8(const GemmEpilogue& ep, int row, int col0) {
    if (KIND == EPI_RESID) return load_raw8<ALIGNED>(ep.resid, static_cast<int64_t>(row) * ep.ldr + col0, ep.resid_f32);
    return load_raw8<ALIGNED>(ep.vel_xe, static_cast<int64_t>(row) * ep.ldy + col0, ep.y_f32);
}

// Eight consecutive columns col0..col0+7 of one row (all inside N, col0 a multiple of 8; a group never straddles two destinations): wide
// stores only, of whole 16-byte pieces if ALIGNED.  SCALED (the 8-bit GEMM): the sums are first multiplied by their row's and column's scale.
template <int KIND, bool SCALED, bool ALIGNED>
__device__ __forceinline__ void epilogue_store8(const GemmEpilogue& ep, int row, int col0, const f32x4& acc0, const f32x4& acc1, const EpiColumns<KIND, SCALED>& c, const EpiRow<KIND, SCALED>& r,
                                                const Raw8& raw) {
    float val[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float a = e < 4 ? acc0[e & 3] : acc1[e & 3];
        val[e] = (SCALED ? a * (r.scale * c.scale[SCALED ? e : 0]) : a) + c.bias[e];
    }
    if (KIND == EPI_VELOCITY) {
        // the velocity step, as in epilogue_store
        const int64_t o = static_cast<int64_t>(row) * ep.ldy + col0;
        float x[8];
        raw_values(raw, ep.y_f32, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (!ep.y_f32) val[e] = static_cast<float>(static_cast<__bf16>(val[e]));
            x[e] = __fsub_rn(x[e], __fmul_rn(ep.vel_dt, val[e]));
        }
        if (ep.y) store8<ALIGNED>(ep.y, o, ep.y_f32, val);
        store8<ALIGNED>(ep.vel_ca, o, ep.y_f32, val);
        store8<ALIGNED>(ep.vel_xe, o, ep.y_f32, x);
        if (ep.vel_xfull) store8<ALIGNED>(ep.vel_xfull, static_cast<int64_t>(r.place) * ep.ldy + col0, ep.y_f32, x);
    } else if (KIND == EPI_PLAIN) {
        if (ep.act == REGIONE_ACT_GELU_TANH) {
#pragma unroll
            for (int e = 0; e < 8; ++e) if (col0 + e >= ep.act_from) val[e] = gelu_tanh_f32(val[e]);
        }
        store8<ALIGNED>(ep.y, static_cast<int64_t>(row) * ep.ldy + col0, ep.y_f32, val);
    } else if (KIND == EPI_QKV) {
        const int H = ep.hidden;   // a multiple of 8
        if (col0 < H) {
            store8<ALIGNED>(ep.q, static_cast<int64_t>(row) * ep.ldq + col0, 0, val);
        } else if (col0 < 3 * H) {
            const int64_t kv_row = r.place;
            if (col0 < 2 * H) store8<ALIGNED>(ep.k, kv_row * ep.ldkv + (col0 - H), 0, val);
            else store8<ALIGNED>(ep.v, kv_row * ep.ldkv + (col0 - 2 * H), 0, val);
        } else {
            if (ep.act == REGIONE_ACT_GELU_TANH) {
#pragma unroll
                for (int e = 0; e < 8; ++e) val[e] = gelu_tanh_f32(val[e]);
            }
            store8<ALIGNED>(ep.y, static_cast<int64_t>(row) * ep.ldy + ep.y_col0 + (col0 - 3 * H), 0, val);
        }
    } else {  // EPI_RESID
        float res[8];
        raw_values(raw, ep.resid_f32, res);
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = res[e] + c.gate[KIND == EPI_RESID ? e : 0] * val[e];
        store8<ALIGNED>(ep.y, static_cast<int64_t>(row) * ep.ldy + col0, ep.y_f32, val);
    }
}

// One element at a time, for column groups that run past N and for Q, K, V rows out of alignment.  The velocity step looks the row's place up once and
// requests every element of x_e before its first store.
template <int KIND, bool SCALED>
__device__ __forceinline__ void epilogue_ragged(const GemmEpilogue& ep, int row, int col0, int N, const f32x4& acc0, const f32x4& acc1) {
    if (KIND == EPI_VELOCITY) {
        const int64_t o = static_cast<int64_t>(row) * ep.ldy + col0;
        const int64_t full = ep.vel_index ? static_cast<int64_t>(ep.vel_index[row]) * ep.ldy + col0 : o;
        const int n = N - col0;
        float v[8], x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < n) x[e] = ep.y_f32 ? static_cast<const float*>(ep.vel_xe)[o + e] : bf16_to_f32(static_cast<const bf16_t*>(ep.vel_xe)[o + e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = (e < 4 ? acc0[e & 3] : acc1[e & 3]) + (ep.bias && e < n ? ep.bias[col0 + e] : 0.f);
            if (!ep.y_f32) v[e] = static_cast<float>(static_cast<__bf16>(v[e]));
            x[e] = __fsub_rn(x[e], __fmul_rn(ep.vel_dt, v[e]));
        }
        auto put = [&](void* base, int64_t at, const float (&w)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < n) {
                    if (ep.y_f32) static_cast<float*>(base)[at + e] = w[e];
                    else static_cast<bf16_t*>(base)[at + e] = f32_to_bf16(w[e]);
                }
        };
        if (ep.y) put(ep.y, o, v);
        put(ep.vel_ca, o, v);
        put(ep.vel_xe, o, x);
        if (ep.vel_xfull) put(ep.vel_xfull, full, x);
        return;
    }
    const float rs = SCALED ? ep.row_scale[row] : 1.f;
    const int64_t kv_row = epilogue_kv_row<KIND>(ep, row);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int col = col0 + e;
        if (col < N) {
            const float a = (e < 4 ? acc0[e & 3] : acc1[e & 3]) * (SCALED ? rs * ep.col_scale[col] : 1.f);
            epilogue_store<KIND>(ep, row, kv_row, col, a, ep.bias ? ep.bias[col] : 0.f, (KIND == EPI_RESID && ep.gate) ? ep.gate[col] : 1.f);
        }
    }
}

// Writes rows [I0, I1) of a wave's accumulators, those of 16x16 matrix instructions whose FIRST operand were the weights: acc[i][j] of a lane
// holds row 16*i + lane%16 of the wave tile and the four columns 32*(j/2) + 8*(lane/16) + 4*(j%2) + 0..3 (the order in which
// the caller presents the weight columns), i.e. eight consecutive columns per pair j = 2b, 2b+1.  A lane writes 16 bytes
// (bf16) of its row per pair, the four lanes of a row 64 contiguous bytes: no transposition, no LDS, no barrier.
// The matrix cores are done by now and only two waves share a SIMD, so that every trip to memory that a store waits for is idle time: the slots and scales of all rows are
// requested before the first store, the vectors of a pair of columns one pair and residual rows one chunk ahead of their use.  With the slot of each row looked up before its store the
// QKV projection of 820 rows (K 3072) took 48.7 us, now 47.3 in a kernel trace; whole calls 1.3 % less (20 % edited 351 -> 346 us, E4M3 block 269 -> 263).
template <int KIND, bool SCALED, int I0, int I1, int RF, int CF, bool ALIGNED>
__device__ __forceinline__ void gemm_epilogue16_wide(const f32x4 (&acc)[RF][CF], int M, int N, int m0, int n0w, const GemmEpilogue& ep) {
    constexpr int R = I1 - I0, P = CF / 2, Q = R * P, MOST = KIND == EPI_VELOCITY || (CF >= 6 && R >= 3) ? 1 : Q >= 12 ? 2 : 4, CH = Q < MOST ? Q : MOST, CHUNKS = (Q + CH - 1) / CH;
    const int l16 = threadIdx.x & 15, c0 = n0w + 8 * ((threadIdx.x & 63) >> 4);
    EpiColumns<KIND, SCALED> cols[2];
    EpiRow<KIND, SCALED> rows[R];
    Raw8 raw[2][CH];
    auto fetch = [&](int c) __attribute__((always_inline)) {
        if (!epi_reads<KIND>()) return;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int q = c * CH + k, row = m0 + 16 * (I0 + q % R) + l16, col = c0 + 32 * (q / R);
            if (q < Q && col + 8 <= N) raw[c & 1][k] = epi_load8<KIND, ALIGNED>(ep, row < M ? row : M - 1, col);
        }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = m0 + 16 * (I0 + r) + l16;
        rows[r].load(ep, row < M ? row : M - 1);
    }
    if (c0 + 8 <= N) cols[0].load(ep, c0);
    fetch(0);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        if (c + 1 < CHUNKS) fetch(c + 1);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int q = c * CH + k, r = q % R, p = q / R;
            const int row = m0 + 16 * (I0 + r) + l16, col = c0 + 32 * p;
            if (r == 0 && p + 1 < P && col + 40 <= N) cols[(p + 1) & 1].load(ep, col + 32);
            if (q < Q && row < M && col + 8 <= N)
                epilogue_store8<KIND, SCALED, ALIGNED>(ep, row, col, acc[I0 + r][q < Q ? 2 * p : 0], acc[I0 + r][q < Q ? 2 * p + 1 : 0], cols[p & 1], rows[r], raw[c & 1][k]);
        }
    }
}
template <int KIND, bool SCALED, int I0, int I1, int RF, int CF>
__device__ __forceinline__ void gemm_epilogue16(const f32x4 (&acc)[RF][CF], int M, int N, int m0, int n0w, const GemmEpilogue& ep) {
    if (ep.vec_ok) {                    // N is a multiple of 8
        gemm_epilogue16_wide<KIND, SCALED, I0, I1, RF, CF, true>(acc, M, N, m0, n0w, ep);
        return;
    }
    // odd widths or unaligned tensors: the same pieces without their alignment, which the memory path takes as it is.  One element at
    // a time cost as much as the product (us): 11844 x 9156 x 832 358 -> 171, 543 x 9522 x 384 24 -> 13, 10605 x 201 x 5568 55 -> 45;
    // velocity heads on 8704 rows of 65 channels 37 -> 27, of 100 45 -> 27
    if (KIND != EPI_QKV) gemm_epilogue16_wide<KIND, SCALED, I0, I1, RF, CF, false>(acc, M, N, m0, n0w, ep);
    const int l16 = threadIdx.x & 15, c0 = n0w + 8 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int p = 0; p < CF / 2; ++p)
        if (c0 + 32 * p < N && (KIND == EPI_QKV || c0 + 32 * p + 8 > N)) {
#pragma unroll
            for (int i = I0; i < I1; ++i) {
                const int row = m0 + 16 * i + l16;
                if (row < M) epilogue_ragged<KIND, SCALED>(ep, row, c0 + 32 * p, N, acc[i][2 * p], acc[i][2 * p + 1]);
            }
        }
}
// one operand of the 8-bit instruction out of the two 16-byte pieces that the 16-bit form feeds to two instructions
__device__ __forceinline__ i32x8 pp_pair(const bf16x8& lo, const bf16x8& hi) {
    const u32x4 a = __builtin_bit_cast(u32x4, lo), b = __builtin_bit_cast(u32x4, hi);
    return i32x8{(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)b[0], (int)b[1], (int)b[2], (int)b[3]};
}

// Tile order inside the launch: groups of `gh` row tiles; inside a group all column tiles, and for each column tile
// the group's row tiles consecutively.  The workgroups that run at the same time on an XCD then share a weight line
// among gh CUs and an activation line among the rest, instead of all of them hammering the same weight lines.
__device__ __forceinline__ void tile_coords(int tile, int m_tiles, int n_tiles, int gh, int& m_tile, int& n_tile) {
    const int per_group = gh * n_tiles;
    const int group = tile / per_group, rem = tile - group * per_group;
    int rows = m_tiles - group * gh;
    rows = rows < gh ? rows : gh;
    n_tile = rem / rows;
    m_tile = group * gh + (rem - n_tile * rows);
}

}  // namespace
