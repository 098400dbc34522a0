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

__device__ __forceinline__ float gelu_tanh_f32(float x) {
    // 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3)
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    return x / (1.0f + __expf(-2.0f * u));
}

// Row of the key/value destination for output row `row` (its cache slot when a slot list is given).
template <int KIND>
__device__ __forceinline__ int64_t epilogue_kv_row(const GemmEpilogue& ep, int row) {
    if (KIND != EPI_QKV) return row;
    return ep.slot ? static_cast<int64_t>(ep.slot[row]) + ep.slot_offset : row;
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

template <bool ALIGNED>
__device__ __forceinline__ void load8(const void* base, int64_t elem, int as_f32, float (&v)[8]) {
    if (as_f32) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 a = *reinterpret_cast<const typename Pieces<ALIGNED>::f32*>(static_cast<const float*>(base) + elem + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = a[e];
        }
    } else {
        const bf16x8 a = *reinterpret_cast<const typename Pieces<ALIGNED>::b16*>(static_cast<const bf16_t*>(base) + elem);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = static_cast<float>(a[e]);
    }
}

// The velocity step (see epilogue_store) on columns col0..col0+n-1 of a row, n <= 8.  WIDE: all eight, in whole pieces.  Otherwise one
// at a time, but the row's place is looked up once and every element of x_e requested before the first store.
template <bool WIDE, bool ALIGNED>
__device__ __forceinline__ void epilogue_velocity(const GemmEpilogue& ep, int row, int col0, int n, float (&val)[8]) {
    const int64_t o = static_cast<int64_t>(row) * ep.ldy + col0;
    const int64_t full = ep.vel_index ? static_cast<int64_t>(ep.vel_index[row]) * ep.ldy + col0 : o;
    float x[8];
    if (WIDE) {
        load8<ALIGNED>(ep.vel_xe, o, ep.y_f32, x);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < n) x[e] = ep.y_f32 ? static_cast<const float*>(ep.vel_xe)[o + e] : bf16_to_f32(static_cast<const bf16_t*>(ep.vel_xe)[o + e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (!ep.y_f32) val[e] = static_cast<float>(static_cast<__bf16>(val[e]));
        x[e] = __fsub_rn(x[e], __fmul_rn(ep.vel_dt, val[e]));
    }
    auto put = [&](void* base, int64_t at, const float (&v)[8]) __attribute__((always_inline)) {
        if (WIDE) { store8<ALIGNED>(base, at, ep.y_f32, v); return; }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < n) {
                if (ep.y_f32) static_cast<float*>(base)[at + e] = v[e];
                else static_cast<bf16_t*>(base)[at + e] = f32_to_bf16(v[e]);
            }
    };
    if (ep.y) put(ep.y, o, val);
    put(ep.vel_ca, o, val);
    put(ep.vel_xe, o, x);
    if (ep.vel_xfull) put(ep.vel_xfull, full, x);
}

// Epilogue for the eight consecutive columns col0..col0+7 of one row (all inside N, col0 a multiple of 8; a group never
// straddles two destinations): wide loads and stores only, of whole 16-byte pieces if ALIGNED.
template <int KIND, bool ALIGNED>
__device__ __forceinline__ void epilogue_store8(const GemmEpilogue& ep, int row, int col0, const float (&acc)[8],
                                                const float (&bias)[8], const float (&gate)[8]) {
    float val[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) val[e] = acc[e] + bias[e];
    if (KIND == EPI_VELOCITY) {
        epilogue_velocity<true, ALIGNED>(ep, row, col0, 8, val);
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
            const int64_t kv_row = epilogue_kv_row<KIND>(ep, row);
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
        load8<ALIGNED>(ep.resid, static_cast<int64_t>(row) * ep.ldr + col0, ep.resid_f32, res);
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = res[e] + gate[e] * val[e];
        store8<ALIGNED>(ep.y, static_cast<int64_t>(row) * ep.ldy + col0, ep.y_f32, val);
    }
}
// Writes a wave's accumulators, those of 16x16 matrix instructions whose FIRST operand were the weights: acc[i][j] of a lane
// holds row 16*i + lane%16 of the wave tile and the four columns 32*(j/2) + 8*(lane/16) + 4*(j%2) + 0..3 (the order in which
// the caller presents the weight columns), i.e. eight consecutive columns per pair j = 2b, 2b+1.  A lane writes 16 bytes
// (bf16) of its row per pair, the four lanes of a row 64 contiguous bytes: no transposition, no LDS, no barrier.
// SCALED (the 8-bit GEMM): every sum is first multiplied by ep.row_scale[row] * ep.col_scale[column].
template <int KIND, bool SCALED, int I0, int I1, int RF, int CF, int B, bool ALIGNED>
__device__ __forceinline__ void gemm_epilogue16_wide(f32x4 (&acc)[RF][CF], int M, int m0, int col0, const GemmEpilogue& ep) {
    const int l16 = threadIdx.x & 15;
    float bias[8], gate[8], cscale[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bias[e] = ep.bias ? ep.bias[col0 + e] : 0.f;
        gate[e] = (KIND == EPI_RESID && ep.gate) ? ep.gate[col0 + e] : 1.f;
        cscale[e] = SCALED ? ep.col_scale[col0 + e] : 1.f;
    }
#pragma unroll
    for (int i = I0; i < I1; ++i) {
        const int row = m0 + 16 * i + l16;
        if (row < M) {
            const float rs = SCALED ? ep.row_scale[row] : 1.f;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = SCALED ? acc[i][2 * B + (e >> 2)][e & 3] * (rs * cscale[e]) : acc[i][2 * B + (e >> 2)][e & 3];
            epilogue_store8<KIND, ALIGNED>(ep, row, col0, v, bias, gate);
        }
    }
}
template <int KIND, bool SCALED, int I0, int I1, int RF, int CF, int B>
__device__ __forceinline__ void gemm_epilogue16_pair(f32x4 (&acc)[RF][CF], int M, int N, int m0, int n0w, const GemmEpilogue& ep) {
    const int lane = threadIdx.x & 63, l16 = lane & 15;
    const int col0 = n0w + 32 * B + 8 * (lane >> 4);
    if (ep.vec_ok) {
        if (col0 < N) gemm_epilogue16_wide<KIND, SCALED, I0, I1, RF, CF, B, true>(acc, M, m0, col0, ep);    // N is a multiple of 8 on this path
    } else if (KIND != EPI_QKV && col0 + 8 <= N) {
        // odd widths or unaligned tensors: the same pieces without their alignment, which the memory path takes as it is.  One element at
        // a time cost as much as the product (us): 11844 x 9156 x 832 358 -> 171, 543 x 9522 x 384 24 -> 13, 10605 x 201 x 5568 55 -> 45;
        // velocity heads on 8704 rows of 65 channels 37 -> 27, of 100 45 -> 27
        gemm_epilogue16_wide<KIND, SCALED, I0, I1, RF, CF, B, false>(acc, M, m0, col0, ep);
    } else {
#pragma unroll
        for (int i = I0; i < I1; ++i) {
            const int row = m0 + 16 * i + l16;
            if (row < M) {
                if (KIND == EPI_VELOCITY) {
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = acc[i][2 * B + (e >> 2)][e & 3] + (ep.bias && col0 + e < N ? ep.bias[col0 + e] : 0.f);
                    epilogue_velocity<false, false>(ep, row, col0, N - col0, v);
                    continue;
                }
                const float rs = SCALED ? ep.row_scale[row] : 1.f;
                const int64_t kv_row = epilogue_kv_row<KIND>(ep, row);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int col = col0 + e;
                    if (col < N) {
                        const float a = acc[i][2 * B + (e >> 2)][e & 3] * (SCALED ? rs * ep.col_scale[col] : 1.f);
                        epilogue_store<KIND>(ep, row, kv_row, col, a, ep.bias ? ep.bias[col] : 0.f, (KIND == EPI_RESID && ep.gate) ? ep.gate[col] : 1.f);
                    }
                }
            }
        }
    }
}
// rows of fragments [I0, I1)
template <int KIND, bool SCALED, int I0, int I1, int RF, int CF>
__device__ __forceinline__ void gemm_epilogue16(f32x4 (&acc)[RF][CF], int M, int N, int m0, int n0w, const GemmEpilogue& ep) {
    gemm_epilogue16_pair<KIND, SCALED, I0, I1, RF, CF, 0>(acc, M, N, m0, n0w, ep);
    if constexpr (CF >= 4) gemm_epilogue16_pair<KIND, SCALED, I0, I1, RF, CF, 1>(acc, M, N, m0, n0w, ep);
    if constexpr (CF >= 6) gemm_epilogue16_pair<KIND, SCALED, I0, I1, RF, CF, 2>(acc, M, N, m0, n0w, ep);
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
