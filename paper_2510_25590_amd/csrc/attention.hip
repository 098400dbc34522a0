// Attention with the Region-Instruction KV cache, Eq.6:
//   O = softmax(Q [K_fresh; K_cache]^T * scale) [V_fresh; V_cache]        (per head)
// Queries are the fresh (edited / text) rows only; the key list is the fresh rows followed by the
// cache rows in use, addressed as one virtual list so that a tile may straddle the two.
//
// Flash-style streaming with an online softmax.  A wave owns 32 queries of one head, whose Q fragments stay in registers; keys and
// values come into LDS by asynchronous global->LDS copies, 64 rows at a time (32 in the DEALT form).  Four forms of workgroup share this tile
// work in different ways (see the forms and the choice between them, plan_attention, below).  The scores are computed
// TRANSPOSED, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: a lane then holds, for ONE query
// (column lane%32), 16 of every 32 keys, so the running maximum and the rescaling factor are
// per-lane scalars, and the exponentiated scores are already in the register layout of the "B"
// operand of the second product O^T = V^T P^T.  The V^T "A" operand (8 consecutive keys per lane
// for one d) is read from the row-major V tile with ds_read_b64_tr_b16, the transposing LDS read
// of gfx950.  The k-slot of the second product pairs lane-half h, slot s of both operands, so the
// only requirement is that both sides enumerate keys identically: slot s of half h of MFMA (kb,j)
// is key kb*32 + 16*j + 8*(s/4) + 4*h + s%4, which is exactly the row order of the S^T accumulator.
#include <cfloat>
#include <cmath>
#include "common.h"
#include "e4m3.h"
#include "layernorm_row.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kThreads = 256;
constexpr int KT = 64;  // keys per tile
constexpr int kMaxSplits = 32;   // key ranges of a query tile

struct AttnArgs {
    const bf16_t* q; int ldq; int n_q;
    const bf16_t* k0; const bf16_t* v0; int ldkv0; int n0;       // fresh rows
    const bf16_t* k1; const bf16_t* v1; int ldkv1; int n1;       // cache rows
    int ld, fast;                                               // fast: one row stride for both arrays, and byte offsets of rows fit 32 bits
    const int32_t* idx1; int rows1;                             // optional row list into the cache, rows of the cache
    int heads; float scale_log2e;
    bf16_t* out; int ldo;
    // split-KV
    int splits; int tiles_per_split; float* part;  // [splits][heads][n_q_pad][D + 4] when splits > 1: O, maximum, sum, two unused (rows stay 16-byte aligned)
    int n_q_pad;
    int q_tiles;
    // Even ranges (see plan_ranges): after `full_blocks` workgroups, each with one key range of one of the first
    // q_full query tiles of a head, range_wgs workgroups take `range` consecutive key tiles each of the list (head, query tile >= q_full,
    // key tile).  A range that covers a query tile's keys only in part leaves its partial result in slot 2 w (the range's
    // first query tile) or 2 w + 1 (its last), rows of the query tile, D + 4 floats each as above.
    int full_blocks, q_full, range, range_wgs;
    int halves;   // SPLIT workgroups: the two wave groups take a key range each (tiles_per_split tiles), else the tiles of one range in turns
};

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;   // native 16-byte vector (plain loads/stores, no memcpy)

// LDS swizzles (16-byte chunk index -> physical chunk).  K tile: the 16 rows read together with one logical chunk
// must cover all 64 banks once; rows are 256 bytes (D = 128) or 128 bytes (D = 64).  V tile: a transposing read
// touches, per lane half, 4 consecutive keys x 4 consecutive chunks.
template <int D> __device__ __forceinline__ int k_swz(int row, int chunk) {
    return D == 128 ? (chunk ^ (row & 15)) : (chunk ^ ((row >> 1) & 7));
}
template <int D> __device__ __forceinline__ int v_swz(int row, int chunk) {
    return D == 128 ? (chunk ^ ((row & 3) << 2)) : (chunk ^ (((row >> 1) & 1) << 2));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr float kRescaleSlack = 8.0f;      // log2 of the largest probability weight kept without moving the reference
constexpr float kRescaleLimit = 256.0f;    // 2^kRescaleSlack: a lane's sum of a tile's weights up to it holds no weight above it
// The value of lane l and of lane l ^ 32, in both lanes: gfx950's v_permlane32_swap exchanges the upper half of its
// first operand with the lower half of its second, so two copies of x become (x of the lower lane, x of the upper
// lane) everywhere.  A vector ALU instruction: no trip through the LDS as with a bpermute.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const unsigned a = r[0], b = r[1];   // elements copied out before the casts: a bit cast applied to r[1] directly reads r[0]
    lo = __uint_as_float(a);
    hi = __uint_as_float(b);
}
__device__ __forceinline__ float max_across_halves(float x) { float lo, hi; both_halves(x, lo, hi); return fmaxf(lo, hi); }
__device__ __forceinline__ float sum_across_halves(float x) { float lo, hi; both_halves(x, lo, hi); return lo + hi; }

// Asynchronous global -> LDS copy of one 16-byte chunk per lane (gfx950 global_load_lds_dwordx4): lane l of the wave
// writes LDS[lds_base + 16*l].  The copy bypasses the VGPRs and is counted in vmcnt; it is written in assembly so
// that the compiler's wait-count pass does not see it (it would wait for it before every later LDS read); the kernel
// waits by hand before the barrier that publishes a stage.
__device__ __forceinline__ void async_copy16(const bf16_t* src, unsigned lds_base_bytes) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "s"(lds_base_bytes) : "memory", "m0");
}

// Same copy with the address split into a wave-uniform 64-bit base (scalar registers) and a 32-bit byte offset per
// lane: the base moves from tile to tile with scalar arithmetic and the lanes' offsets never change.
__device__ __forceinline__ void async_copy16_sbase(unsigned lane_off_bytes, const bf16_t* base, unsigned lds_base_bytes) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(lane_off_bytes), "s"(base), "s"(lds_base_bytes) : "memory", "m0");
}

// The N copies of a wave that belong together (1 KiB each, one after the other in LDS), their addresses split into a wave-uniform 64-bit base
// (scalar registers) and a 32-bit byte offset per lane.  The instruction's offset counts on both sides, so one write of m0 serves them all; on
// the global side it is taken back by `copy_bias`, which keeps every lane's offset positive.  A scalar instruction costs its wave as much
// time as a vector one: with m0 and a masked exec written for each copy the vector phase took 300 cycles longer.
constexpr unsigned copy_bias(int n, int i) { return static_cast<unsigned>(n - 1 - i) * 1024u; }
template <int N, int I> __device__ __forceinline__ void async_copy_of(const unsigned (&off)[N], const char* base, unsigned lds_base_bytes) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
                 :: "v"(off[I]), "s"(base - copy_bias(N, 0)), "s"(lds_base_bytes), "n"(I * 1024) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void async_copy_of(int i, const unsigned (&off)[N], const char* base, unsigned lds_base_bytes) {   // i: known after unrolling
    if (i == 0) async_copy_of<N, 0>(off, base, lds_base_bytes);
    else if (i == 1) async_copy_of<N, 1>(off, base, lds_base_bytes);
    else if (N > 2 && i == 2) async_copy_of<N, (N > 2 ? 2 : 0)>(off, base, lds_base_bytes);
    else if (N > 2 && i == 3) async_copy_of<N, (N > 2 ? 3 : 0)>(off, base, lds_base_bytes);
}
// All N if wanted > 0: copies that are not wanted keep their place in the wave's count but move nothing.
template <int N> __device__ __forceinline__ void async_copies_if(int wanted, const unsigned (&off)[N], const char* base, unsigned lds_base_bytes) {
    base -= copy_bias(N, 0);
    if constexpr (N == 2)
        asm volatile("s_cmp_gt_i32 %4, 0\n\ts_cselect_b64 exec, -1, 0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:1024\n\ts_mov_b64 exec, -1"
                     :: "v"(off[0]), "v"(off[1]), "s"(base), "s"(lds_base_bytes), "s"(wanted) : "memory", "m0", "scc");
    else
        asm volatile("s_cmp_gt_i32 %6, 0\n\ts_cselect_b64 exec, -1, 0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %4\n\t"
                     "global_load_lds_dwordx4 %1, %4 offset:1024\n\tglobal_load_lds_dwordx4 %2, %4 offset:2048\n\tglobal_load_lds_dwordx4 %3, %4 offset:3072\n\ts_mov_b64 exec, -1"
                     :: "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "s"(lds_base_bytes), "s"(wanted) : "memory", "m0", "scc");
}

// At most N of this wave's copies still in flight.  The wait is the compiler's own builtin, not assembly: its
// wait-count pass then knows that its own earlier loads (query fragments, index entries) have landed too and does
// not put waits of its own for them into the tile loop, where they would also wait for the copies just issued.
template <int N> __device__ __forceinline__ void wait_async_copies() {
    static_assert(N >= 0 && N < 64, "vmcnt is a six-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));   // vmcnt(N), other counters untouched
    asm volatile("" ::: "memory");
}
// At most N of this wave's LDS reads still on their way (they arrive in order).
template <int N> __device__ __forceinline__ void wait_lds_reads() { __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (N << 8) | (3 << 14)); }
__device__ __forceinline__ void phase_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Which rows a call reads: one contiguous array (fresh rows only, or the whole cache), fresh rows followed by cache
// rows, or cache rows picked by an index list.
enum { SRC_CONTIG = 0, SRC_TWO = 1, SRC_INDEXED = 2 };

// Three-input maximum in assembly (plain fmaxf costs an extra canonicalising instruction per MFMA result).  The
// compiler does not check what an assembly statement reads against the MFMAs still in flight, so the FIRST read of an
// accumulator after its last MFMA must be an ordinary expression (first_max below), which gets the required wait
// states; everything chained behind it is late enough.
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float first_max(float a, float b) { return __builtin_fmaxf(a, b); }
// Issues the copies of one 64-key tile into an LDS stage.  The tile is 64 * CPR chunks; wave w issues blocks
// b = w*LD_N + i of 64 consecutive chunk positions, position P = row*CPR + physical chunk.  Since the LDS side is
// linear in the lane, the swizzle is applied on the global side: the lane that owns physical chunk p of a row loads
// the logical chunk p ^ f(row) (both swizzles are XORs, hence their own inverses).
template <int D, int NW, int MODE>
__device__ __forceinline__ void kv_tile_issue(const AttnArgs& a, int head, int key0, int n_keys, unsigned stage_base_bytes) {
    constexpr int CPR = D / 8, LD_N = KT * CPR / (NW * 64), TILE = KT * D;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // All addresses first, the copies afterwards: an index entry is an ordinary load, and a wait for it placed between
    // two copies would wait for the earlier copy as well.
    const bf16_t* ksrc[LD_N];
    const bf16_t* vsrc[LD_N];
#pragma unroll
    for (int i = 0; i < LD_N; ++i) {
        const int pos = (wave * LD_N + i) * 64 + lane;
        const int row = pos / CPR, phys = pos % CPR;
        int key = key0 + row;
        key = key < n_keys ? key : n_keys - 1;   // tail rows repeat a valid row; their scores are masked
        const bool fresh = key < a.n0;
        int64_t grow = fresh ? key : key - a.n0;
        if (MODE == SRC_INDEXED) { if (!fresh) grow = a.idx1[grow]; }
        const int64_t base = grow * (fresh ? a.ldkv0 : a.ldkv1) + head * D;
        ksrc[i] = (fresh ? a.k0 : a.k1) + base + (k_swz<D>(row, phys) << 3);
        vsrc[i] = (fresh ? a.v0 : a.v1) + base + (v_swz<D>(row, phys) << 3);
    }
#pragma unroll
    for (int i = 0; i < LD_N; ++i) asm volatile("" : "+v"(ksrc[i]), "+v"(vsrc[i]));   // pins the order: addresses, then copies
#pragma unroll
    for (int i = 0; i < LD_N; ++i) {
        const unsigned lds_blk = __builtin_amdgcn_readfirstlane(stage_base_bytes + static_cast<unsigned>(wave * LD_N + i) * 1024u);
        async_copy16(ksrc[i], lds_blk);
        async_copy16(vsrc[i], lds_blk + TILE * 2u);
    }
}
// One 64-key tile for the QB*32 queries of a wave.  STAGE selects the LDS buffer (compile time, so that every LDS
// address is a per-lane constant plus an immediate).  K and V fragments are read once and used for all QB query blocks.
template <int D, int STAGE, int QB, bool MASK>
__device__ __forceinline__ void attn_tile(const bf16_t* smem, int t, int n_keys, float c, int lh,
                                          const int (&koff)[D / 16], const int (&voff)[D / 32], const bf16x8 (&qf)[QB][D / 16],
                                          f32x16 (&o)[QB][D / 32], float (&m_run)[QB], float (&l_run)[QB]) {
    constexpr int DB = D / 32, KK = D / 16, TILE = KT * D;
    const bf16_t* kt = smem + STAGE * 2 * TILE;
    const bf16_t* vt = kt + TILE;

    // ---- S^T = K Q^T for the two 32-key blocks
    f32x16 s[QB][2];
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;   // becomes the inline constant 0 of the first MFMA's accumulator operand
    // K fragments are fetched two k-steps (four reads) ahead of their MFMAs
    constexpr int PF = 2;
    bf16x8 kf[KK][2];
#pragma unroll
    for (int kk = 0; kk < PF; ++kk)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) kf[kk][kb] = *reinterpret_cast<const bf16x8*>(kt + koff[kk] + kb * 32 * D);
    s16x4 vlo[DB], vhi[DB];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        if (kk + PF < KK) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) kf[kk + PF][kb] = *reinterpret_cast<const bf16x8*>(kt + koff[kk + PF] + kb * 32 * D);
        } else if (kk + PF == KK) {
            // first group of V^T fragments: in flight during the last MFMAs of S and the softmax
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                vlo[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + voff[db]));
                vhi[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + voff[db] + 8 * D));
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                s[qb][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk][kb], qf[qb][kk], kk == 0 ? zero : s[qb][kb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- online softmax on raw scores; accumulator r of block kb is key t*64 + kb*32 + 8*(r/4) + 4*lh + r%4
    if (MASK) {   // only the last tile of the key list can run past it: the kernel peels that tile off its main loop
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (t * KT + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= n_keys) s[qb][kb][r] = -INFINITY;
    }
    bf16x8 pf[QB][2][2];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        // maximum of the lane's 32 scores with three-input maxima (plain fmaxf costs an extra canonicalising
        // instruction per MFMA result); -inf entries of a masked tail are ordinary operands
        float mx = first_max(s[qb][0][0], s[qb][0][1]);   // waits for the last MFMA of block 0
#pragma unroll
        for (int r = 2; r < 16; r += 2) mx = max3(mx, s[qb][0][r], s[qb][0][r + 1]);
        mx = first_max(mx, s[qb][1][0]);                  // and of block 1, issued later
        mx = max3(mx, s[qb][1][1], s[qb][1][15]);
#pragma unroll
        for (int r = 2; r < 14; r += 2) mx = max3(mx, s[qb][1][r], s[qb][1][r + 1]);
        mx = max3(mx, s[qb][1][14], s[qb][1][14]);
        mx = max_across_halves(mx);
        // m_run is the REFERENCE of the exponentials, not the exact running maximum: it only moves when the tile's
        // maximum exceeds it by more than kRescaleSlack (in the log2 domain), so exp2((s - m_run) c) <= 2^kRescaleSlack
        // and the 64-multiplication rescale of the accumulators becomes rare.  Any reference gives the same quotient
        // O / l; the probabilities keep their relative precision in bf16 whatever their scale.
        const bool move = (mx - m_run[qb]) * c > kRescaleSlack;     // the first tile: m_run is the most negative reference
        float m_new = m_run[qb];
        if (__builtin_amdgcn_ballot_w64(move) != 0) {               // wave-uniform branch
            m_new = move ? mx : m_run[qb];
            const float alpha = move ? fast_exp2((m_run[qb] - m_new) * c) : 1.0f;
            l_run[qb] *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[qb][db][r] *= alpha;
            m_run[qb] = m_new;
        }
        const float neg_mc = -m_new * c;
        float psum = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float p = fast_exp2(__builtin_fmaf(s[qb][kb][8 * j + e], c, neg_mc));
                    psum += p;
                    pf[qb][kb][j][e] = static_cast<__bf16>(p);
                }
        l_run[qb] += psum;
    }

    // ---- O^T += V^T P^T, one (kb, j) group of DB*QB MFMAs at a time, the next group's fragments in flight
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int kb = g >> 1, j = g & 1;
        bf16x8 vf[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const s16x8 both = {vlo[db][0], vlo[db][1], vlo[db][2], vlo[db][3], vhi[db][0], vhi[db][1], vhi[db][2], vhi[db][3]};
            vf[db] = __builtin_bit_cast(bf16x8, both);
        }
        if (g < 3) {
            const int row_off = (((g + 1) >> 1) * 32 + 16 * ((g + 1) & 1)) * D;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                vlo[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + voff[db] + row_off));
                vhi[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + voff[db] + row_off + 8 * D));
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int db = 0; db < DB; ++db) o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db], pf[qb][kb][j], o[qb][db], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Four waves of 32 queries, copies one tile ahead in two LDS stages.
// RANGED: the grid holds even ranges (AttnArgs); a form of its own because the loop over query tiles costs registers.
template <int D, int MODE, bool RANGED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_narrow_kernel(AttnArgs a) {
    constexpr int NW = 4, QB = 1;
    constexpr int DB = D / 32;   // 32-wide d blocks of the output
    constexpr int KK = D / 16;   // k-steps of the first product
    constexpr int CPR = D / 8, LD_N = KT * CPR / (NW * 64), TILE = KT * D;
    constexpr int QW = NW * QB * 32;                    // queries per workgroup
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];   // two stages of (K tile, V tile)
    bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);
    const unsigned smem_bytes0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(smem_raw)));   // LDS byte address

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    // XCD-aware numbering (workgroup i runs on XCD i % 8): all query tiles of one (head, key split) get consecutive
    // slots on ONE XCD, so that the K/V range they share is filled into a single L2 once instead of once per query tile;
    // for the same reason an XCD's even ranges are consecutive ones.
    const int xcd = blockIdx.x & 7;
    const int n_keys = a.n0 + a.n1;
    const int n_tiles = (n_keys + KT - 1) / KT;
    const bool ranged = RANGED && static_cast<int>(blockIdx.x) >= a.full_blocks;
    int head, q_tile, tile_begin, tile_end, left = 0, slot = 0;
    if (!ranged) {
        const int local = blockIdx.x >> 3;
        const int group = (local / a.q_full) * 8 + xcd;            // (head, split) pair
        if (group >= a.heads * a.splits) return;
        q_tile = local % a.q_full;
        head = group % a.heads;
        slot = group / a.heads;
        tile_begin = slot * a.tiles_per_split;
        tile_end = tile_begin + a.tiles_per_split;
        tile_end = tile_end < n_tiles ? tile_end : n_tiles;
    } else {
        const int per_xcd = (a.range_wgs + 7) / 8;
        const int w = xcd * per_xcd + ((static_cast<int>(blockIdx.x) - a.full_blocks) >> 3);
        const int q_rest = a.q_tiles - a.q_full;
        const int first = w * a.range;
        const int total = a.heads * q_rest * n_tiles;              // the launcher keeps it below 2^30
        if (w >= a.range_wgs || first >= total) return;
        left = total - first < a.range ? total - first : a.range;
        const int seg = first / n_tiles;
        head = seg / q_rest;
        q_tile = a.q_full + seg % q_rest;
        tile_begin = first - seg * n_tiles;
        tile_end = tile_begin + left < n_tiles ? tile_begin + left : n_tiles;
        slot = 2 * w;
    }
    head = __builtin_amdgcn_readfirstlane(head); q_tile = __builtin_amdgcn_readfirstlane(q_tile); slot = __builtin_amdgcn_readfirstlane(slot);
    tile_begin = __builtin_amdgcn_readfirstlane(tile_begin); tile_end = __builtin_amdgcn_readfirstlane(tile_end); left = __builtin_amdgcn_readfirstlane(left);

    // per-lane LDS offsets (elements) of the fragment reads
    int koff[KK], voff[DB];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) koff[kk] = l32 * D + (k_swz<D>(l32, kk * 2 + lh) << 3);
    {
        const int src_key = 4 * lh + ((lane & 15) >> 2);      // row this lane addresses in a transposing read (plus a multiple of 8)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int d_src = db * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);   // 4 consecutive d = 8 bytes
            voff[db] = src_key * D + (v_swz<D>(src_key, d_src >> 3) << 3) + (d_src & 7);
        }
    }

    const float c = a.scale_log2e;
    // the reference of a row that has met no score above -inf: finite and finite times c, so that such keys weigh exp2(-inf) = 0
    // (with a reference of -inf they would weigh exp2(-inf + inf) = NaN), and no larger than any finite score worth keeping
    const float m_floor = c <= 1.0f ? -FLT_MAX : -FLT_MAX * 0.999999f / c;

    // Two LDS stages, copies one tile ahead.  Per tile: wait until this tile's copies have landed, barrier (publishes
    // them and retires the stage read one tile ago), issue the copies of the next tile into that retired stage, compute.
    // Tiles past the end re-copy the last tile so that the copy count per tile is constant.
    constexpr unsigned STAGE_BYTES = 2u * TILE * 2u;
    // contiguous source: per-lane byte offsets of this thread's chunk positions inside a tile, for K and for V
    const bf16_t* const src_k = a.n0 > 0 ? a.k0 : a.k1;
    const bf16_t* const src_v = a.n0 > 0 ? a.v0 : a.v1;
    const int src_ld = a.n0 > 0 ? a.ldkv0 : a.ldkv1;
    unsigned off_k[LD_N], off_v[LD_N];
    if (MODE == SRC_CONTIG) {
#pragma unroll
        for (int i = 0; i < LD_N; ++i) {
            const int pos = (wave * LD_N + i) * 64 + lane;
            const int row = pos / CPR, phys = pos % CPR;
            const unsigned row_off = static_cast<unsigned>(row) * static_cast<unsigned>(src_ld);
            off_k[i] = (row_off + static_cast<unsigned>(k_swz<D>(row, phys) << 3)) * 2u;
            off_v[i] = (row_off + static_cast<unsigned>(v_swz<D>(row, phys) << 3)) * 2u;
        }
    }
    const unsigned wave_lds = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(wave * LD_N) * 1024u);
    auto issue_tile = [&](int t, unsigned stage_bytes) __attribute__((always_inline)) {
        const int tc = t < tile_end ? t : tile_end - 1;
        if (MODE == SRC_CONTIG && (tc + 1) * KT <= n_keys) {     // a full tile of one array: scalar base + fixed lane offsets
            const bf16_t* kb = src_k + static_cast<int64_t>(tc) * KT * src_ld + head * D;
            const bf16_t* vb = src_v + static_cast<int64_t>(tc) * KT * src_ld + head * D;
#pragma unroll
            for (int i = 0; i < LD_N; ++i) {
                const unsigned lds_blk = stage_bytes + wave_lds + static_cast<unsigned>(i) * 1024u;
                async_copy16_sbase(off_k[i], kb, lds_blk);
                async_copy16_sbase(off_v[i], vb, lds_blk + TILE * 2u);
            }
        } else {
            kv_tile_issue<D, NW, MODE == SRC_CONTIG ? SRC_TWO : MODE>(a, head, tc * KT, n_keys, stage_bytes);
        }
    };
    for (;;) {   // one query tile and key range; an even range may run on into further query tiles
        if (tile_begin < tile_end) issue_tile(tile_begin, smem_bytes0);
        const int q_base = q_tile * QW + wave * (QB * 32);
        // Q fragments ("B" operand): lane holds query l32 of the block, d = kk*16 + 8*lh + 0..7
        bf16x8 qf[QB][KK];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            int qrow = q_base + qb * 32 + l32;
            qrow = qrow < a.n_q ? qrow : a.n_q - 1;
            const bf16_t* qp = a.q + static_cast<int64_t>(qrow) * a.ldq + head * D + 8 * lh;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) qf[qb][kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
        }
        f32x16 o[QB][DB];
        float m_run[QB], l_run[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            m_run[qb] = m_floor;
            l_run[qb] = 0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[qb][db][r] = 0.f;
        }
#define RG_ATTN_TILE(T, STAGE, MASK)                                                                      \
        {                                                                                                     \
            const int t_ = (T);                                                                               \
            wait_async_copies<0>();                                                                           \
            __syncthreads();                                                                                  \
            issue_tile(t_ + 1, smem_bytes0 + ((STAGE) ^ 1) * STAGE_BYTES);                                    \
            attn_tile<D, STAGE, QB, MASK>(smem, t_, n_keys, c, lh, koff, voff, qf, o, m_run, l_run);          \
        }
        // only the very last tile of the key list can be partial; it runs outside the main loop with the masking code
        const bool last_partial = tile_end * KT > n_keys;
        const int full_end = last_partial ? tile_end - 1 : tile_end;
        for (int t = tile_begin; t < full_end; t += 2) {
            RG_ATTN_TILE(t, 0, false)
            if (t + 1 < full_end) RG_ATTN_TILE(t + 1, 1, false)
        }
        if (full_end < tile_end && tile_begin < tile_end) {   // its stage follows from the number of full tiles before it
            if (((full_end - tile_begin) & 1) == 0) RG_ATTN_TILE(full_end, 0, true) else RG_ATTN_TILE(full_end, 1, true)
        }
#undef RG_ATTN_TILE
        wait_async_copies<0>();   // nothing may still be writing LDS when the workgroup ends

        const bool whole = ranged ? tile_begin == 0 && tile_end == n_tiles : a.splits == 1;
        // ---- finish: O^T accumulator r of d-block db: d = db*32 + 8*(r/4) + 4*lh + r%4, query = l32
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int qrow = q_base + qb * 32 + l32;
            const float l_tot = sum_across_halves(l_run[qb]);
            if (qrow >= a.n_q) continue;
            if (whole) {
                const float inv = 1.0f / l_tot;
                bf16_t* op = a.out + static_cast<int64_t>(qrow) * a.ldo + head * D;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int d = db * 32 + 8 * g + 4 * lh;
                        bf16x4 pk;
#pragma unroll
                        for (int e = 0; e < 4; ++e) pk[e] = static_cast<__bf16>(o[qb][db][4 * g + e] * inv);
                        *reinterpret_cast<bf16x4*>(op + d) = pk;
                    }
            } else {
                // partial result: unnormalised O, running max (log2 domain) and sum
                const int64_t prow = ranged ? static_cast<int64_t>(slot) * QW + (qrow - q_tile * QW) : (static_cast<int64_t>(slot) * a.heads + head) * a.n_q_pad + qrow;
                float* pp = a.part + prow * (D + 4);
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int d = db * 32 + 8 * g + 4 * lh;
                        *reinterpret_cast<f32x4*>(pp + d) = f32x4{o[qb][db][4 * g], o[qb][db][4 * g + 1], o[qb][db][4 * g + 2], o[qb][db][4 * g + 3]};
                    }
                if (lh == 0) { pp[D] = m_run[qb] * c; pp[D + 1] = l_tot; }   // maximum in the log2 domain, as the merge kernel expects
            }
        }
        left -= tile_end - tile_begin;
        if (!ranged || left <= 0) break;
        __syncthreads();   // every wave has read its last tile before the next query tile's first copies
        slot |= 1;         // only the last query tile of a range can be partial from here on
        tile_begin = 0;
        tile_end = left < n_tiles ? left : n_tiles;
        if (++q_tile == a.q_tiles) { q_tile = a.q_full; ++head; }
    }
}

// DEALT: few queries on not too many keys.  A workgroup takes 32 queries of one head and deals the key range, in blocks of 32 keys, to its eight waves.
// Bound by latency: the kernel below spends 8 us outside its tile loop (groups that wait for each other, partial results of 128 queries through memory and
// a second launch to join them).  Here every wave works on its own, without a barrier in its loop: its K and V blocks come into LDS of its own,
// leave it for registers as fragments at once, and the next block is copied meanwhile; partial results meet in LDS.  us, key ranges and their merge
// launch before -> now: 36 queries x 544 keys, 4 heads of 64, 8.5 -> 5.8; 544 x 544 9.4 -> 5.9; 1022 x 1022, 8 heads of 128, 23.1 -> 11.6; 95 x 759, 24
// heads, 13.6 -> 9.8.
template <int D> struct DealtTile {
    static constexpr int DB = D / 32, KK = D / 16, CPR = D / 8;
    static constexpr int COPIES = 32 * CPR / 64;            // copies per lane for the K (or V) rows of a block
    static constexpr int COPY_ROWS = 64 / CPR;              // rows per copy
    static constexpr unsigned BLOCK = 32u * D * 2u;         // K (or V) rows of a block
    static constexpr unsigned WAVE = 2u * BLOCK;            // a wave's LDS: K block, V block; its accumulators at the end
    static constexpr unsigned ML_BASE = 8u * WAVE;          // reference and sum of every wave and query
    static constexpr unsigned LIST_BASE = ML_BASE + 8u * 32u * 8u;
    static_assert(WAVE == DB * 4096u, "a wave's accumulators fit where its blocks were");
};
constexpr int kDealtKeys = 4096;                            // the longest list of rows kept in LDS

template <int D, bool INDEXED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_dealt_kernel(AttnArgs a) {
    using T = DealtTile<D>;
    constexpr int DB = T::DB, KK = T::KK, CPR = T::CPR, COPIES = T::COPIES;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds)));   // LDS byte address
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    // XCD-aware numbering, as below
    const int local = blockIdx.x >> 3;
    const int group = (local / a.q_tiles) * 8 + (blockIdx.x & 7);   // (head, key split) pair
    if (group >= a.heads * a.splits) return;
    const int q_tile = local % a.q_tiles, head = group % a.heads, slot = group / a.heads;
    const int n_keys = a.n0 + a.n1;
    const int key_begin = slot * a.tiles_per_split * KT;
    int key_end = key_begin + a.tiles_per_split * KT;
    key_end = key_end < n_keys ? key_end : n_keys;
    const int blocks = key_end > key_begin ? (key_end - key_begin + 31) / 32 : 0;
    const int mine = blocks > wave ? (blocks - wave + 7) / 8 : 0;   // blocks wave, wave + 8, ... of the range
    const float c = a.scale_log2e;
    const float m_floor = c <= 1.0f ? -FLT_MAX : -FLT_MAX * 0.999999f / c;   // see the kernel below

    int32_t* list = reinterpret_cast<int32_t*>(lds + T::LIST_BASE);  // INDEXED: the range's cache rows (complete at the barrier after the first scores)
    const int list0 = key_begin > a.n0 ? key_begin : a.n0;           // the key of its first entry

    const int copy_row = lane / CPR;
    const unsigned ld_bytes = static_cast<unsigned>(a.ld) * 2u;
    const unsigned wave_lds = lds0 + static_cast<unsigned>(wave) * T::WAVE;
    // The rows of a wave's first two blocks come straight from the index list (entry l32 in lane l32), those of later ones from its copy in LDS.
    int first_rows[2];
    if (INDEXED) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            int e = key_begin + (wave + 8 * x) * 32 + l32;
            e = (e < key_end ? e : key_end - 1) - a.n0;
            first_rows[x] = a.idx1[e > 0 ? e : 0];
        }
    }
    auto listed_row = [&](int nth, int row, int key) __attribute__((always_inline)) {   // nth: block of the wave, 2 for all later ones
        return nth < 2 ? __builtin_amdgcn_ds_bpermute(row * 4, first_rows[nth & 1]) : list[key - list0];
    };
    // copies the K (V) rows of the block that begins at key `key0`; past the end of the range it repeats the last row
    auto issue = [&](const bf16_t* s0, const bf16_t* s1, bool is_v, int key0, unsigned dst, int nth) __attribute__((always_inline)) {
        const bool in0 = key0 + 32 <= a.n0, in1 = key0 >= a.n0 && key0 + 32 <= key_end;
        if (a.fast && (in0 || in1)) {
            const bf16_t* base = (in0 ? s0 + static_cast<int64_t>(key0) * a.ld : s1 + (INDEXED ? int64_t{0} : static_cast<int64_t>(key0 - a.n0) * a.ld)) + head * D;
#pragma unroll
            for (int i = 0; i < COPIES; ++i) {
                const int row = copy_row + i * T::COPY_ROWS;
                unsigned off = static_cast<unsigned>(row);
                if (INDEXED && !in0) off = static_cast<unsigned>(listed_row(nth, row, key0 + row));
                const int swz = is_v ? v_swz<D>(row, lane % CPR) : k_swz<D>(row, lane % CPR);
                async_copy16_sbase(off * ld_bytes + static_cast<unsigned>(swz << 4), base, dst + i * 1024u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) {
                const int row = copy_row + i * T::COPY_ROWS;
                int key = key0 + row;
                key = key < key_end ? key : key_end - 1;
                const bool fresh = key < a.n0;
                int64_t r = fresh ? key : key - a.n0;
                if (INDEXED) { const int in_list = listed_row(nth, row, fresh ? list0 : key); if (!fresh) r = in_list; }
                const int swz = is_v ? v_swz<D>(row, lane % CPR) : k_swz<D>(row, lane % CPR);
                async_copy16((fresh ? s0 : s1) + r * (fresh ? a.ldkv0 : a.ldkv1) + head * D + (swz << 3), dst + i * 1024u);
            }
        }
    };
    // Q fragments ("B" operand): lane holds query l32 of the tile, d = kk*16 + 8*lh + 0..7
    const int q_row = q_tile * 32 + l32;
    bf16x8 qf[KK];
    {
        const bf16_t* qp = a.q + static_cast<int64_t>(q_row < a.n_q ? q_row : a.n_q - 1) * a.ldq + head * D + 8 * lh;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
    }
    const int key_first = key_begin + wave * 32;
    if (mine > 0) {
        issue(a.k0, a.k1, false, key_first, wave_lds, 0);
        issue(a.v0, a.v1, true, key_first, wave_lds + T::BLOCK, 0);
    }
    if (INDEXED) {
        const int first = key_begin > a.n0 ? key_begin - a.n0 : 0, last = key_end - a.n0;
        for (int e = first + static_cast<int>(threadIdx.x); e < last; e += 512) list[e - first] = a.idx1[e];
    }
    unsigned koff[KK], voff[DB];                                     // per-lane LDS byte offsets of the fragment reads
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) koff[kk] = wave * T::WAVE + static_cast<unsigned>(l32 * D * 2) + static_cast<unsigned>(k_swz<D>(l32, kk * 2 + lh) << 4);
    const int src_key = 4 * lh + ((lane & 15) >> 2);                 // row this lane addresses in a transposing read (plus a multiple of 8)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        const int d_src = db * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        voff[db] = wave * T::WAVE + T::BLOCK + static_cast<unsigned>(src_key * D * 2) + static_cast<unsigned>(v_swz<D>(src_key, d_src >> 3) << 4) + static_cast<unsigned>((d_src & 7) * 2);
    }
    f32x16 o[DB], s, zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = zero;
    float m_run = m_floor, l_run = 0.f;

    // S^T = K Q^T of block i, whose K rows leave LDS for registers first, so that the next block's can follow
#define RG_DEALT_SCORES(I, AHEAD, NTH)                                                                                  \
    {                                                                                                       \
        bf16x8 kf[KK];                                                                                      \
        _Pragma("unroll") for (int kk = 0; kk < KK; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(lds + koff[kk]); \
        wait_lds_reads<0>();                                                                                \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        if (AHEAD) issue(a.k0, a.k1, false, key_first + ((I) + 1) * 256, wave_lds, NTH);                    \
        _Pragma("unroll") for (int kk = 0; kk < KK; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], kk == 0 ? zero : s, 0, 0, 0); \
        const int key0_ = key_first + (I) * 256;                                                            \
        if (key0_ + 32 > key_end) {                                                                         \
            _Pragma("unroll") for (int r = 0; r < 16; ++r)                                                  \
                if (key0_ + 8 * (r >> 2) + 4 * lh + (r & 3) >= key_end) s[r] = -INFINITY;                   \
        }                                                                                                   \
    }
#define RG_DEALT_MAX(MX)                                                                                    \
    float MX = fmaxf(s[0], s[1]);                                                                           \
    _Pragma("unroll") for (int r = 2; r < 16; ++r) MX = fmaxf(MX, s[r]);                                    \
    MX = max_across_halves(MX);
#define RG_DEALT_WEIGH()                                                                                    \
    {                                                                                                       \
        const float neg_mc_ = -m_run * c;                                                                   \
        float sum_[2] = {0.f, 0.f};                                                                         \
        _Pragma("unroll") for (int r = 0; r < 16; ++r) {                                                    \
            const float p_ = fast_exp2(__builtin_fmaf(s[r], c, neg_mc_));                                   \
            sum_[r & 1] += p_;                                                                              \
            pf[r >> 3][r & 7] = static_cast<__bf16>(p_);                                                    \
        }                                                                                                   \
        psum = sum_[0] + sum_[1];                                                                           \
    }
    // A wave's reference is the maximum of its own first block; see the kernel below for what a reference is and when it moves.  The weight of a reference's
    // key is exactly one, so eight references of 32 keys each round fewer of the large weights than one of 64 keys for all waves did, and no wave waits for another
    // one's scores.  Error against 64 bits (2-norm; scores of spread 2), shared reference -> own ones: 95 queries on 759 keys by index list, 24 heads of 128,
    // 2.31e-3 -> 2.11e-3 (key ranges of four waves 2.03e-3), 100 x 3000, 8 heads of 128, 2.21e-3 -> 1.89e-3, 36 x 544, 4 heads of 64, 2.24e-3 -> 2.05e-3 (2.09e-3).
    // us: 64 x 513, 24 heads, 9.85 -> 8.45; 100 x 3000 14.5 -> 13.75; 36 x 544 6.4 -> 6.0.
    if (mine > 0) {
        wait_async_copies<0>();
        RG_DEALT_SCORES(0, mine > 1, 1)
        RG_DEALT_MAX(mx)
        m_run = fmaxf(m_floor, mx);
    }
    if (INDEXED) __syncthreads();                                    // the list is complete
    for (int i = 0; i < mine; ++i) {
        bf16x8 pf[2];
        float psum;
        RG_DEALT_WEIGH()
        if (__builtin_amdgcn_ballot_w64(!(psum <= kRescaleLimit)) != 0) {
            RG_DEALT_MAX(mx)
            const float m_new = fmaxf(m_run, mx);
            const float alpha = m_new > m_run ? fast_exp2((m_run - m_new) * c) : 1.0f;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
            m_run = m_new;
            RG_DEALT_WEIGH()
        }
        l_run += psum;
        // V of this block; the K copies of the next one, if any, are younger
        if (i + 1 < mine) wait_async_copies<COPIES>(); else wait_async_copies<0>();
        s16x4 vlo[2][DB], vhi[2][DB];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const unsigned char* p = lds + (voff[db] + g * 16 * D * 2);
                vlo[g][db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
                vhi[g][db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 8 * D * 2));
            }
        wait_lds_reads<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < mine) issue(a.v0, a.v1, true, key_first + (i + 1) * 256, wave_lds + T::BLOCK, 2);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const s16x8 both = {vlo[g][db][0], vlo[g][db][1], vlo[g][db][2], vlo[g][db][3], vhi[g][db][0], vhi[g][db][1], vhi[g][db][2], vhi[g][db][3]};
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[g], o[db], 0, 0, 0);
            }
        if (i + 1 < mine) {
            wait_async_copies<COPIES>();                             // K of the next block; its V copies are younger
            RG_DEALT_SCORES(i + 1, i + 2 < mine, 2)
        }
    }
#undef RG_DEALT_WEIGH
#undef RG_DEALT_MAX
#undef RG_DEALT_SCORES

    // ---- the waves' results meet in LDS: every wave sums its share of the accumulators over all waves
    l_run = sum_across_halves(l_run);
    float2* ml = reinterpret_cast<float2*>(lds + T::ML_BASE);
    if (lh == 0) ml[wave * 32 + l32] = float2{m_run, l_run};
    f32x4* mine4 = reinterpret_cast<f32x4*>(lds + wave * T::WAVE) + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) mine4[(db * 4 + g) * 64] = f32x4{o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]};
    __syncthreads();
    float m = m_floor, l_tot = 0.f, weight[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) { const float2 x = ml[w * 32 + l32]; weight[w] = x.x; m = fmaxf(m, x.x); }
#pragma unroll
    for (int w = 0; w < 8; ++w) { weight[w] = fast_exp2((weight[w] - m) * c); l_tot += weight[w] * ml[w * 32 + l32].y; }
    if (q_row < a.n_q) {
        const float inv = 1.0f / l_tot;
        const int64_t prow = (static_cast<int64_t>(slot) * a.heads + head) * a.n_q_pad + q_row;
#pragma unroll
        for (int j = 0; j < DB / 2; ++j) {
            const int f = wave * (DB / 2) + j;                       // accumulators 4 (f % 4) .. of d block f / 4
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 8; ++w) x += weight[w] * (reinterpret_cast<const f32x4*>(lds + w * T::WAVE) + lane)[f * 64];
            const int d = (f >> 2) * 32 + 8 * (f & 3) + 4 * lh;
            if (a.splits == 1) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk[e] = static_cast<__bf16>(x[e] * inv);
                *reinterpret_cast<bf16x4*>(a.out + static_cast<int64_t>(q_row) * a.ldo + head * D + d) = pk;
            } else {
                *reinterpret_cast<f32x4*>(a.part + prow * (D + 4) + d) = x;
            }
        }
        if (a.splits > 1 && wave == 0 && lh == 0) { a.part[prow * (D + 4) + D] = m * c; a.part[prow * (D + 4) + D + 1] = l_tot; }
    }
}

// Head dimension 128: eight waves, two per SIMD, in two groups that take turns.  While one group is at the matrix cores (scores of its next tile,
// then the second product of this one: 32 MFMAs) the other forms its softmax and starts the copies of later tiles; a barrier ends each phase.  On this
// chip a wave's vector instructions pass beside another wave's MFMAs at full rate on both sides (probe: 32.0 cycles per MFMA beside 7 FMAs of another
// wave), but two waves of a SIMD that run freely meet in the same phase half of the time.  Per tile and wave: 1024 cycles of MFMAs, and some 110 vector
// instructions (32 of them exponentials at 8 cycles).  The chip is then bound by its power: the clock falls to 1.64 GHz with
// the matrix cores busy in 79 % of the SIMD-cycles (counters, 19456 x 19456; 72 % at 8704 x 8704), and any work left out (copies, LDS
// reads, vector instructions) gives time in proportion to its energy, so tiles are shared by as many queries as the shape allows.
//
// How the groups share a workgroup's work.  SPLIT: 128 queries; the groups take the key tiles of one range in turns, or a range each, and their results
// are joined at the end.  SHARE: 256 queries; both groups take every key tile, so that a tile is copied into LDS once for twice as many
// queries (a tenth of the time went into copies).  24 heads, us, workgroups of four free waves before -> now: 8704 queries x 8704 keys 832 -> 766,
// 2560 x 8704 259 -> 225, 1382 x 19456 374 -> 319, 1332 x 8704 by index list 220 -> 167 (SHARE); 820 x 8704 105 -> 96, 205 x 8704
// 41 -> 35 (SPLIT).  16x16x32 MFMAs (less power, but twice the issue slots and eight more registers) were 3 % faster in unsplit calls and slower in all others.
template <int D, bool SHARE> struct AttnTile {
    static constexpr int DB = D / 32;                       // 32-wide d blocks of the output
    static constexpr int KK = D / 16;                       // k-steps of the first product
    static constexpr int CPR = D / 8;                       // 16-byte chunks per row
    static constexpr int QW = SHARE ? 256 : 128;            // queries per workgroup
    static constexpr int LD_N = KT * CPR / (SHARE ? 512 : 256);   // copies per thread for the K (or V) rows of a tile
    static constexpr unsigned BYTES = KT * D * 2u;          // K (or V) rows of a tile
    static constexpr int SLOTS = SHARE ? 4 : 2;             // tiles whose K rows (and V rows) are in LDS, per group or for both
    static constexpr int K_AHEAD = SLOTS - SHARE;           // a round copies K of the tile so many further on, V of the one before that
    static constexpr unsigned V_BASE = SLOTS * BYTES;       // K rows, then V rows
    static constexpr unsigned GROUP_BYTES = SHARE ? 0u : 4u * BYTES;
    static constexpr unsigned REF_BASE = 8u * BYTES;        // SPLIT: references of the first tile, one per query
    static constexpr unsigned LDS_BYTES = REF_BASE + (SHARE ? 0u : 128u * 4u);
    static constexpr unsigned EX_WAVE = DB * 4096u;         // SPLIT, the join of the groups: accumulators on their way, per pair of waves
    static_assert(4u * EX_WAVE + 8u * 512u <= REF_BASE, "the join fits where the tiles were");
};

// INDEXED: cache rows are named by an index list.  RANGED: the grid holds even ranges (AttnArgs); a form of its own because
// the loop over query tiles costs registers.
template <int D, bool SHARE, bool INDEXED, bool RANGED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_kvcache_kernel(AttnArgs a) {
    using T = AttnTile<D, SHARE>;
    constexpr int DB = T::DB, KK = T::KK, CPR = T::CPR, LD_N = T::LD_N, QW = T::QW, SLOTS = T::SLOTS, AHEAD = T::K_AHEAD;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds)));   // LDS byte address

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2, w4 = wave & 3;
    const int copy_wave = SHARE ? wave : w4;
    const int l32 = lane & 31, lh = lane >> 5;
    // XCD-aware numbering (workgroup i runs on XCD i % 8): all query tiles of one (head, key split) get consecutive
    // slots on ONE XCD, so that the K/V range they share is filled into a single L2 once instead of once per query tile;
    // for the same reason an XCD's even ranges are consecutive ones.
    const int xcd = blockIdx.x & 7;
    const int n_keys = a.n0 + a.n1;
    const int n_tiles = (n_keys + KT - 1) / KT;
    const bool ranged = RANGED && static_cast<int>(blockIdx.x) >= a.full_blocks;
    const bool halves = !SHARE && !RANGED && a.halves;
    const int stride = SHARE || halves ? 1 : 2;                // from one tile of a group to its next
    int head, q_tile, tile_begin, tile_end, left = 0, slot = 0;
    if (!ranged) {
        const int local = blockIdx.x >> 3;
        const int group = (local / a.q_full) * 8 + xcd;            // (head, split) pair
        if (group >= a.heads * a.splits) return;
        q_tile = local % a.q_full;
        head = group % a.heads;
        slot = group / a.heads;
        tile_begin = (halves ? 2 * slot + grp : slot) * a.tiles_per_split;
        tile_end = tile_begin + a.tiles_per_split;
        tile_end = tile_end < n_tiles ? tile_end : n_tiles;
    } else {
        const int per_xcd = (a.range_wgs + 7) / 8;
        const int w = xcd * per_xcd + ((static_cast<int>(blockIdx.x) - a.full_blocks) >> 3);
        const int q_rest = a.q_tiles - a.q_full;
        const int first = w * a.range;
        const int total = a.heads * q_rest * n_tiles;              // the launcher keeps it below 2^30
        if (w >= a.range_wgs || first >= total) return;
        left = total - first < a.range ? total - first : a.range;
        const int seg = first / n_tiles;
        head = seg / q_rest;
        q_tile = a.q_full + seg % q_rest;
        tile_begin = first - seg * n_tiles;
        tile_end = tile_begin + left < n_tiles ? tile_begin + left : n_tiles;
        slot = 2 * w;
    }
    head = __builtin_amdgcn_readfirstlane(head); q_tile = __builtin_amdgcn_readfirstlane(q_tile); slot = __builtin_amdgcn_readfirstlane(slot);
    tile_begin = __builtin_amdgcn_readfirstlane(tile_begin); tile_end = __builtin_amdgcn_readfirstlane(tile_end); left = __builtin_amdgcn_readfirstlane(left);

    // per-lane LDS byte offsets of the fragment reads, the group's place included
    unsigned koff[KK], voff[DB];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) koff[kk] = grp * T::GROUP_BYTES + static_cast<unsigned>(l32 * D * 2) + static_cast<unsigned>(k_swz<D>(l32, kk * 2 + lh) << 4);
    {
        const int src_key = 4 * lh + ((lane & 15) >> 2);         // row this lane addresses in a transposing read (plus a multiple of 8)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int d_src = db * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);   // 4 consecutive d = 8 bytes
            voff[db] = grp * T::GROUP_BYTES + T::V_BASE + static_cast<unsigned>(src_key * D * 2) + static_cast<unsigned>(v_swz<D>(src_key, d_src >> 3) << 4) + static_cast<unsigned>((d_src & 7) * 2);
        }
    }

    const float c = a.scale_log2e;
    // the reference of a row that has met no score above -inf: finite and finite times c, so that such keys weigh exp2(-inf) = 0
    // (with a reference of -inf they would weigh exp2(-inf + inf) = NaN), and no larger than any finite score worth keeping
    const float m_floor = c <= 1.0f ? -FLT_MAX : -FLT_MAX * 0.999999f / c;

    // Copies: the tile's rows are cut into 16-byte chunks, position P = row*CPR + physical chunk; the waves that
    // use the tile copy 64*LD_N positions each.  The LDS side is linear in the lane, so the swizzle is applied on the global side: the lane that
    // owns physical chunk p of a row loads the logical chunk p ^ f(row) (both swizzles are XORs, hence their own inverses).
    const unsigned copy_dst = lds0 + grp * T::GROUP_BYTES + static_cast<unsigned>(copy_wave * LD_N) * 1024u;
    const int copy_row = (copy_wave * LD_N * 64 + lane) / CPR;          // of the lane's first position; the next ones are 64 / CPR rows apart
    constexpr int COPY_ROWS = 64 / CPR;
    unsigned k_chunk[LD_N], v_chunk[LD_N];                       // byte offset of a lane's chunk inside its row, and the copy's bias
#pragma unroll
    for (int i = 0; i < LD_N; ++i) {
        const int row = copy_row + i * COPY_ROWS, phys = lane % CPR;
        k_chunk[i] = static_cast<unsigned>(k_swz<D>(row, phys) << 4) + copy_bias(LD_N, i);
        v_chunk[i] = static_cast<unsigned>(v_swz<D>(row, phys) << 4) + copy_bias(LD_N, i);
    }
    const unsigned ld_bytes = static_cast<unsigned>(a.ld) * 2u;
    unsigned row_off[LD_N], row_prev[LD_N];                      // indexed rows: byte offsets of this lane's rows of the tile whose K comes next, and of the one before
    int idx_next[LD_N];                                          // index entries of the tile after it
    auto load_index = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LD_N; ++i) {
            int e = t * KT + copy_row + i * COPY_ROWS - a.n0;
            e = e < a.n1 ? e : a.n1 - 1;
            idx_next[i] = a.idx1[e > 0 ? e : 0];
        }
    };
    // Where the rows of full tile t of one array begin, and the lanes' offsets from there.
    auto tile_base = [&](const bf16_t* s0, const bf16_t* s1, int t) __attribute__((always_inline)) {
        const int key0 = t * KT;
        return reinterpret_cast<const char*>((key0 < a.n0 ? s0 + static_cast<int64_t>(key0) * a.ld : s1 + (INDEXED ? int64_t{0} : static_cast<int64_t>(key0 - a.n0) * a.ld)) + head * D);
    };
    auto lane_offsets = [&](unsigned (&off)[LD_N], const unsigned (&chunk)[LD_N], const unsigned (&listed)[LD_N], bool fresh) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LD_N; ++i) {
            off[i] = static_cast<unsigned>(copy_row + i * COPY_ROWS) * ld_bytes;
            if (INDEXED) off[i] = fresh ? off[i] : listed[i];
            off[i] += chunk[i];
        }
    };
    // any other tile (and any tile of arrays that 32-bit offsets do not reach)
    auto issue_any = [&](const bf16_t* s0, const bf16_t* s1, const unsigned (&chunk)[LD_N], int t, unsigned dst) __attribute__((always_inline)) {
        // All addresses first, the copies afterwards: an index entry is an ordinary load, and a wait for it placed between
        // two copies would wait for the earlier copy as well.
        const bf16_t* src[LD_N];
#pragma unroll
        for (int i = 0; i < LD_N; ++i) {
            int key = t * KT + copy_row + i * COPY_ROWS;
            key = key < n_keys ? key : n_keys - 1;               // tail rows repeat a valid row; their scores are masked
            const bool fresh = key < a.n0;
            int64_t row = fresh ? key : key - a.n0;
            if (INDEXED) { if (!fresh) row = a.idx1[row]; }
            src[i] = (fresh ? s0 : s1) + row * (fresh ? a.ldkv0 : a.ldkv1) + head * D + ((chunk[i] - copy_bias(LD_N, i)) >> 1);
        }
#pragma unroll
        for (int i = 0; i < LD_N; ++i) asm volatile("" : "+v"(src[i]));   // pins the order: addresses, then copies
#pragma unroll
        for (int i = 0; i < LD_N; ++i) async_copy16(src[i], __builtin_amdgcn_readfirstlane(dst + i * 1024u));
    };
    // Tiles before `first1` lie in the fresh rows, from `begin1` on in the cache rows; one between them has rows of both.
    const int first1 = a.n0 / KT, begin1 = first1 + (a.n0 % KT != 0);
    const int full_tiles = n_keys / KT;
    // copies the K (V) rows of tile t, or nothing if wanted <= 0 (past the end of the wave's range)
    auto issue = [&](const bf16_t* s0, const bf16_t* s1, const unsigned (&chunk)[LD_N], const unsigned (&listed)[LD_N], int t, int wanted, unsigned dst) __attribute__((always_inline)) {
        const int tc = t < tile_end ? t : tile_end - 1;
        if (a.fast && tc < full_tiles && (tc < first1 || tc >= begin1)) {
            unsigned off[LD_N];
            lane_offsets(off, chunk, listed, tc < first1);
            async_copies_if<LD_N>(wanted, off, tile_base(s0, s1, tc), dst);
        } else {
            issue_any(s0, s1, chunk, tc, dst);
        }
    };
    // the rows of tile t come next: their offsets from the entries loaded before, and the entries of the tile two further on
    auto next_rows = [&](int t_after) __attribute__((always_inline)) {
        if (!INDEXED) return;
#pragma unroll
        for (int i = 0; i < LD_N; ++i) { row_prev[i] = row_off[i]; row_off[i] = static_cast<unsigned>(idx_next[i]) * ld_bytes; }
        load_index(t_after < tile_end ? t_after : tile_end - 1);
    };
    if (INDEXED) {
#pragma unroll
        for (int i = 0; i < LD_N; ++i) { row_off[i] = 0; row_prev[i] = 0; idx_next[i] = 0; }
    }

    for (;;) {   // one query tile and key range; an even range may run on into further query tiles
        const int n = tile_end - tile_begin;
        const int mine = SHARE || halves ? n : (n + 1 - grp) >> 1;   // tiles of this wave's group, not positive if there are none
        int rounds = SHARE ? n : (n + 1) >> 1;                   // the first group has no fewer
        if (halves) rounds = grp == 0 ? n : n_tiles - 2 * slot * a.tiles_per_split < a.tiles_per_split ? n_tiles - 2 * slot * a.tiles_per_split : a.tiles_per_split;
        const int t0 = SHARE || halves ? tile_begin : tile_begin + grp;
        const int q_base = q_tile * QW + (SHARE ? wave : w4) * 32;
        const bool alive = q_base < a.n_q;                       // a wave past the last query only copies
        const int q_row = q_base + l32;
        f32x16 o[DB];
        float m_run = m_floor, l_run = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] = 0.f;

        if (rounds > 0) {
            f32x16 s[2], zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;          // becomes the inline constant 0 of an accumulator operand
            bf16x8 pf[2][2];
            bf16x8 kf[3][4];                                     // K fragments of the steps in flight
            s16x4 vlo[3][4], vhi[3][4];                          // V fragments of the steps in flight
            // The queries come through LDS too, so that they are counted with the copies and the first products start while the second tile and
            // the first values are still on their way.  Their place is that of tiles copied after the barrier (SPLIT: the second values of either
            // group, 16 rows by the wave of each group; SHARE: 32 rows by every wave for itself).
            unsigned q_lds;
            {
                constexpr int ROWS = SHARE ? 32 : 16;
                const unsigned half = T::V_BASE + T::BYTES + static_cast<unsigned>(w4) * (16u * D * 2u);                       // SPLIT: in either group
                q_lds = SHARE ? (grp == 0 ? 2u * T::BYTES : T::V_BASE + T::BYTES) + static_cast<unsigned>(w4) * (32u * D * 2u) : half;
                const unsigned dst = lds0 + q_lds + (SHARE ? 0u : grp * T::GROUP_BYTES);
#pragma unroll
                for (int i = 0; i < ROWS * CPR / 64; ++i) {
                    const int row = (SHARE ? 0 : grp * 16) + i * COPY_ROWS + lane / CPR;
                    const int qr = q_base + row < a.n_q ? q_base + row : a.n_q - 1;
                    async_copy16(a.q + static_cast<int64_t>(qr) * a.ldq + head * D + (k_swz<D>(row, lane % CPR) << 3), dst + i * 1024u);
                }
            }
            if (INDEXED) {
                load_index(t0 < tile_end ? t0 : tile_end - 1);
                next_rows(t0 + stride);
#pragma unroll
                for (int i = 0; i < LD_N; ++i) asm volatile("" : "+v"(idx_next[i]));   // waited for here, not behind the first copies
            }
            issue(a.k0, a.k1, k_chunk, row_off, t0, mine, copy_dst);
            next_rows(t0 + 2 * stride);
            issue(a.k0, a.k1, k_chunk, row_off, t0 + stride, mine - 1, copy_dst + T::BYTES);
            issue(a.v0, a.v1, v_chunk, row_prev, t0, mine, copy_dst + T::V_BASE);
            wait_async_copies<2 * LD_N>();                       // the queries and K of the first tile
            if (!SHARE) phase_barrier();
            // Q fragments ("B" operand): lane holds query l32 of the wave, d = kk*16 + 8*lh + 0..7
            bf16x8 qf[KK];
            {
                const unsigned char* qp = lds + q_lds + (SHARE ? static_cast<unsigned>(l32) * (D * 2u) : (l32 >> 4) * T::GROUP_BYTES + static_cast<unsigned>(l32 & 15) * (D * 2u));
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + (k_swz<D>(l32, kk * 2 + lh) << 4));
            }
            wait_lds_reads<0>();
            if (SHARE) {
                phase_barrier();
                next_rows(t0 + 3 * stride);
                issue(a.k0, a.k1, k_chunk, row_off, t0 + 2 * stride, mine - 2, copy_dst + 2u * T::BYTES);
                issue(a.v0, a.v1, v_chunk, row_prev, t0 + stride, mine - 1, copy_dst + T::V_BASE + T::BYTES);
            }
            if (grp == 1) {                                      // the second group runs one phase behind the first
                wait_async_copies<SHARE ? 2 * LD_N : LD_N>();    // its part of K of the second tile has landed where the first group looks for it (SHARE)
                phase_barrier();
            }
            // Matrix work goes in steps of four MFMAs, whose four fragments were requested two steps before.
#define RG_K_READ1(STEP, F, SLOT) kf[(STEP) % 3][F] = *reinterpret_cast<const bf16x8*>(lds + (koff[2 * (STEP) + ((F) >> 1)] + ((SLOT) * T::BYTES + ((F) & 1) * 32 * D * 2)));
#define RG_K_READ(STEP, SLOT)   /* two k-steps of both 32-key blocks */                                     \
            _Pragma("unroll") for (int f = 0; f < 4; ++f) { RG_K_READ1(STEP, f, SLOT) }
            // of the 4 * DB products of 16 keys with a d block
            constexpr int PV = DB, SS = KK / 2;                  // steps of the second and of the first product
#define RG_V_READ(STEP, SLOT)                                                                               \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                 \
                const unsigned char* p_ = lds + (voff[(4 * (STEP) + j) % DB] + ((SLOT) * T::BYTES + ((4 * (STEP) + j) / DB) * 16 * D * 2)); \
                vlo[(STEP) % 3][j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p_));             \
                vhi[(STEP) % 3][j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p_ + 8 * D * 2)); \
            }
            // A step's own requests are spread between its MFMAs.
#define RG_SPREAD(READS)                                                                                    \
            _Pragma("unroll") for (int x_ = 0; x_ < 4; ++x_) {                                              \
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                                            \
                if ((READS) >= 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                        \
                if ((READS) >= 8) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                        \
            }                                                                                               \
            __builtin_amdgcn_sched_barrier(0);
            // S^T = K Q^T; the fragments of the first two steps have arrived before
#define RG_S_STEPS(SLOT, VSLOT, WITH_V)                                                                     \
            _Pragma("unroll") for (int st = 0; st < SS; ++st) {                                             \
                if (st >= 2) { if (st + 1 < SS) wait_lds_reads<4>(); else wait_lds_reads<(WITH_V) ? 8 : 0>(); } \
                __builtin_amdgcn_sched_barrier(0);                                                          \
                if (st + 2 < SS) { RG_K_READ(st + 2, SLOT) }                                                \
                else if (WITH_V) { RG_V_READ(st + 2 - SS, VSLOT) }                                          \
                _Pragma("unroll") for (int f = 0; f < 4; ++f)                                               \
                    s[f & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st % 3][f], qf[2 * st + (f >> 1)], st == 0 && f < 2 ? zero : s[f & 1], 0, 0, 0); \
                RG_SPREAD(st + 2 < SS ? 4 : (WITH_V) ? 8 : 0)                                               \
            }
            // O^T += V^T P^T; the fragments of the first two steps have been requested before
#define RG_PV_STEPS(VSLOT)                                                                                  \
            _Pragma("unroll") for (int st = 0; st < PV; ++st) {                                             \
                if (st + 1 < PV) { wait_lds_reads<8>(); } else { wait_lds_reads<0>(); }                     \
                __builtin_amdgcn_sched_barrier(0);                                                          \
                if (st + 2 < PV) { RG_V_READ(st + 2, VSLOT) }                                               \
                _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                             \
                    const s16x4 lo_ = vlo[st % 3][j], hi_ = vhi[st % 3][j];                                 \
                    const s16x8 both_ = {lo_[0], lo_[1], lo_[2], lo_[3], hi_[0], hi_[1], hi_[2], hi_[3]};   \
                    const int g_ = (4 * st + j) / DB, db_ = (4 * st + j) % DB;                              \
                    o[db_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both_), pf[g_ >> 1][g_ & 1], o[db_], 0, 0, 0); \
                }                                                                                           \
                RG_SPREAD(st + 2 < PV ? 8 : 0)                                                              \
            }
            if (mine > 0 && alive) {
                RG_K_READ(0, 0)
                RG_K_READ(1, 0)
                wait_lds_reads<0>();
                RG_S_STEPS(0, 0, false)
            }
            wait_async_copies<SHARE ? 2 * LD_N : LD_N>();        // K of the second tile
            phase_barrier();
            // Weights of the scores in chunks of four accumulators, a chunk summed and rounded while the next one is formed; AFTER(chunk) stands
            // for what else is to be started there.  Accumulator r of block kb is key kb*32 + 8*(r/4) + 4*lh + r%4 of the tile.
#define RG_WEIGH(AFTER)                                                                                     \
            {                                                                                               \
                const float neg_mc_ = -m_run * c;                                                           \
                float p_[2][4], sum_[2] = {0.f, 0.f};                                                       \
                _Pragma("unroll") for (int ch = 0; ch <= 8; ++ch) {                                         \
                    if (ch < 8)                                                                             \
                        _Pragma("unroll") for (int r = 0; r < 4; ++r)                                       \
                            p_[ch & 1][r] = fast_exp2(__builtin_fmaf(s[ch >> 2][(ch & 3) * 4 + r], c, neg_mc_)); \
                    if (ch > 0)                                                                             \
                        _Pragma("unroll") for (int r = 0; r < 4; ++r) {                                     \
                            sum_[r & 1] += p_[(ch - 1) & 1][r];                                             \
                            pf[(ch - 1) >> 2][((ch - 1) >> 1) & 1][((ch - 1) & 1) * 4 + r] = static_cast<__bf16>(p_[(ch - 1) & 1][r]); \
                        }                                                                                   \
                    if (ch < 8) { AFTER(ch) }                                                               \
                }                                                                                           \
                psum = sum_[0] + sum_[1];                                                                   \
            }
#define RG_NOTHING(CH)
            // The vector phase's copies, and the first K fragments of the next matrix phase, spread over the chunks: the copies of the waves
            // pass the address unit at 16 cycles each, and a wave that issues several in a row waits there.
#define RG_COPY(CH)                                                                                         \
                if ((CH) < LD_N) async_copy_of<LD_N>((CH), off_k, k_src, k_dst);                            \
                else if ((CH) < 2 * LD_N) async_copy_of<LD_N>((CH) - LD_N, off_v, v_src, v_dst);
#define RG_MEMORY(CH)                                                                                       \
            {                                                                                               \
                RG_K_READ1((CH) / 4, (CH) % 4, slot_n)                                                      \
                RG_COPY(CH)                                                                                 \
                __builtin_amdgcn_sched_barrier(0);                                                          \
            }
            // The scores' weights, and their reference: m_run is not the exact running maximum.  It only moves when a lane's sum of a tile's weights
            // exceeds kRescaleLimit (or is NaN), so that no weight does and the rescale of the accumulators becomes rare; no maximum is formed for that.
            // Any reference gives the same quotient O / l; the probabilities keep their relative precision in bf16 whatever their scale.
            // Where the limit is met the reference becomes the maximum so far, whatever it exceeds the old one by: a lane's sum of a tile like this one is then
            // at most 32.  (Moving only for a weight above the limit left it where weights of 8 to 256 add up to more than the limit, and every later tile
            // formed its weights twice: keys that score 3 to 5 above the first tile's, 24 heads, 2560 x 8704 312 us for 228, 1332 x 8704 by index list 222 for 171.)
#define RG_MAX(MX)                                                                                          \
            float MX = fmaxf(s[0][0], s[1][0]);                                                             \
            _Pragma("unroll") for (int r = 1; r < 16; ++r) MX = fmaxf(MX, fmaxf(s[0][r], s[1][r]));         \
            MX = max_across_halves(MX);
#define RG_SOFTMAX(AFTER)                                                                                   \
            {                                                                                               \
                float psum;                                                                                 \
                RG_WEIGH(AFTER)                                                                             \
                if (__builtin_amdgcn_ballot_w64(!(psum <= kRescaleLimit)) != 0) {                           \
                    RG_MAX(mx)                                                                              \
                    const float m_new = fmaxf(m_run, mx);                                                   \
                    const float alpha = m_new > m_run ? fast_exp2((m_run - m_new) * c) : 1.0f;              \
                    l_run *= alpha;                                                                         \
                    _Pragma("unroll") for (int db = 0; db < DB; ++db)                                       \
                        _Pragma("unroll") for (int r = 0; r < 16; ++r) o[db][r] *= alpha;                   \
                    m_run = m_new;                                                                          \
                    RG_WEIGH(RG_NOTHING)                                                                    \
                }                                                                                           \
                l_run += psum;                                                                              \
            }
            // One round of a group.  Vector phase: the softmax of its tile I, while the other group is at the matrix cores; the copies of later tiles
            // go to places that the matrix phases before have read.  Matrix phase: the scores of tile I + 1, then O += P V of tile I.
            // SLOT: I modulo SLOTS.  What a matrix phase reads has landed by the end of a vector phase before it (SPLIT: V; SHARE: both, and
            // a whole round earlier, since the other group's copies of a tile count as well), or of the matrix phase before it (SPLIT: K).
#define RG_OF(SLOT) ((SLOT) % SLOTS)
#define RG_FULL_ROUND(I, SLOT, ALIVE)                                                                       \
            {                                                                                               \
                const int i_ = (I);                                                                         \
                if (INDEXED) next_rows(t0 + stride * (i_ + AHEAD + 1));                                  \
                unsigned off_k[LD_N], off_v[LD_N];                                                          \
                lane_offsets(off_k, k_chunk, row_off, in_fresh);                                            \
                lane_offsets(off_v, v_chunk, row_prev, in_fresh);                                           \
                constexpr unsigned slot_n = RG_OF((SLOT) + 1);                                              \
                const unsigned k_dst = copy_dst + RG_OF((SLOT) + AHEAD) * T::BYTES, v_dst = copy_dst + T::V_BASE + RG_OF((SLOT) + AHEAD - 1) * T::BYTES; \
                if (ALIVE) { RG_SOFTMAX(RG_MEMORY) }                                                        \
                else { _Pragma("unroll") for (int ch = 0; ch < 2 * LD_N; ++ch) { RG_COPY(ch) } }            \
                k_src += src_step;                                                                          \
                v_src += src_step;                                                                          \
                wait_lds_reads<0>();                                                                        \
                wait_async_copies<2 * LD_N>();                                                              \
                phase_barrier();                                                                            \
                if (ALIVE) {                                                                                \
                    __builtin_amdgcn_s_setprio(1);                                                          \
                    RG_S_STEPS(slot_n, SLOT, true)                                                          \
                    RG_PV_STEPS(SLOT)                                                                       \
                    __builtin_amdgcn_s_setprio(0);                                                          \
                }                                                                                           \
                if (!SHARE) wait_async_copies<LD_N>();                                                      \
                phase_barrier();                                                                            \
            }
#define RG_FULL_ROUNDS(ALIVE)                                                                               \
            for (int p = 0; p < turns; ++p, i += SLOTS) {                                                   \
                RG_FULL_ROUND(i, 1, ALIVE)                                                                  \
                if constexpr (SHARE) {                                                                      \
                    RG_FULL_ROUND(i + 1, 2, ALIVE)                                                          \
                    RG_FULL_ROUND(i + 2, 3, ALIVE)                                                          \
                }                                                                                           \
                RG_FULL_ROUND(i + SLOTS - 1, 0, ALIVE)                                                      \
            }
            float* refs = reinterpret_cast<float*>(lds + T::REF_BASE);
            for (int i = 0; i < rounds; ) {
                // Turns of SLOTS rounds, from one whose tile sits in slot 1 on, whose copies are of full tiles of one array and wanted, and none that
                // meets the masked tile.
                if (i % SLOTS == 1 && a.fast) {
                    const int lo = t0 + stride * (i + AHEAD - 1);   // the first tile copied (V), and past the last one that may be (K is a tile further on)
                    const bool in_fresh = lo < first1;
                    int hi = in_fresh ? first1 : lo < begin1 ? 0 : full_tiles;
                    hi = hi < t0 + stride * mine ? hi : t0 + stride * mine;
                    const int turn_tiles = stride * SLOTS;            // the last turn copies K of tile lo + turn_tiles * turns
                    const int turns = hi - lo > turn_tiles ? (hi - lo - 1) / turn_tiles : 0;
                    const char* k_src = tile_base(a.k0, a.k1, lo + stride);
                    const char* v_src = tile_base(a.v0, a.v1, lo);
                    const int64_t src_step = INDEXED && !in_fresh ? int64_t{0} : static_cast<int64_t>(stride * KT) * ld_bytes;
                    if (alive) { RG_FULL_ROUNDS(true) } else { RG_FULL_ROUNDS(false) }
                }
                if (i >= rounds) break;
                const int slot_ = i % SLOTS;
                if (INDEXED) next_rows(t0 + stride * (i + AHEAD + 1));
                issue(a.k0, a.k1, k_chunk, row_off, t0 + stride * (i + AHEAD), mine - (i + AHEAD), copy_dst + RG_OF(slot_ + AHEAD) * T::BYTES);
                issue(a.v0, a.v1, v_chunk, row_prev, t0 + stride * (i + AHEAD - 1), mine - (i + AHEAD - 1), copy_dst + T::V_BASE + RG_OF(slot_ + AHEAD - 1) * T::BYTES);
                if (i < mine && alive) {
                    RG_K_READ(0, RG_OF(slot_ + 1))
                    RG_K_READ(1, RG_OF(slot_ + 1))
                    __builtin_amdgcn_sched_barrier(0);
                    const int key0 = (t0 + stride * i) * KT;
                    if (key0 + KT > n_keys) {   // only the last tile of the key list can run past it
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int r = 0; r < 16; ++r)
                                if (key0 + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= n_keys) s[kb][r] = -INFINITY;
                    }
                    if (i == 0) {   // one reference per range, the maximum of its first tile (of finite scores)
                        if (!SHARE && !halves && grp == 1) {
                            m_run = refs[w4 * 32 + l32];
                        } else {
                            RG_MAX(mx)
                            m_run = fmaxf(m_floor, mx);
                        }
                    }
                    RG_SOFTMAX(RG_NOTHING)
                    if (!SHARE && i == 0 && grp == 0 && lh == 0) refs[w4 * 32 + l32] = m_run;
                }
                wait_lds_reads<0>();
                wait_async_copies<2 * LD_N>();
                phase_barrier();
                if (i < mine && alive) {
                    __builtin_amdgcn_s_setprio(1);
                    RG_S_STEPS(RG_OF(slot_ + 1), slot_, true)     // past the last tile: of stale rows, never used
                    RG_PV_STEPS(slot_)
                    __builtin_amdgcn_s_setprio(0);
                }
                if (!SHARE) wait_async_copies<LD_N>();
                phase_barrier();
                ++i;
            }
#undef RG_FULL_ROUNDS
#undef RG_OF
#undef RG_FULL_ROUND
#undef RG_SOFTMAX
#undef RG_MAX
#undef RG_MEMORY
#undef RG_COPY
#undef RG_NOTHING
#undef RG_WEIGH
#undef RG_PV_STEPS
#undef RG_SPREAD
#undef RG_S_STEPS
#undef RG_V_READ
#undef RG_K_READ
#undef RG_K_READ1
            if (grp == 0) phase_barrier();
            wait_async_copies<0>();              // nothing may still be writing LDS when it is used again or the workgroup ends
            __syncthreads();
        }

        // ---- SPLIT: the groups' results meet in LDS; group 0 finishes the first half of the d blocks, group 1 the others
        const bool whole = ranged ? tile_begin == 0 && tile_end == n_tiles : a.splits == 1;
        f32x4* ex = reinterpret_cast<f32x4*>(lds + w4 * T::EX_WAVE) + lane;
        float2* ml = reinterpret_cast<float2*>(lds + 4u * T::EX_WAVE) + w4 * 64 + lane;
        l_run = sum_across_halves(l_run);
        float m = m_run, w_own = 1.f, w_other = 0.f, l_tot = l_run;
#define RG_PART(DBI, G) f32x4{o[DBI][4 * (G)], o[DBI][4 * (G) + 1], o[DBI][4 * (G) + 2], o[DBI][4 * (G) + 3]}
#define RG_GIVE(DB0, DB1)                                                                                   \
        {                                                                                                   \
            _Pragma("unroll") for (int db = (DB0); db < (DB1); ++db)                                        \
                _Pragma("unroll") for (int g = 0; g < 4; ++g) ex[(db * 4 + g) * 64] = RG_PART(db, g);       \
        }
#define RG_FINISH(DB0, DB1)   /* O^T accumulator r of d-block db: d = db*32 + 8*(r/4) + 4*lh + r%4, query = l32 */ \
        {                                                                                                   \
            _Pragma("unroll") for (int db = (DB0); db < (DB1); ++db)                                        \
                _Pragma("unroll") for (int g = 0; g < 4; ++g) {                                             \
                    const int d = db * 32 + 8 * g + 4 * lh;                                                 \
                    f32x4 x = RG_PART(db, g);                                                               \
                    if (!SHARE) x = w_own * x + w_other * ex[(db * 4 + g) * 64];                            \
                    if (whole) {                                                                            \
                        bf16x4 pk;                                                                          \
                        _Pragma("unroll") for (int e = 0; e < 4; ++e) pk[e] = static_cast<__bf16>(x[e] * inv); \
                        *reinterpret_cast<bf16x4*>(a.out + static_cast<int64_t>(q_row) * a.ldo + head * D + d) = pk; \
                    } else {                                                                                \
                        *reinterpret_cast<f32x4*>(pp + d) = x;                                              \
                    }                                                                                       \
                }                                                                                           \
        }
        if (!SHARE) {
            ml[grp * 256] = float2{m_run, l_run};
            if (grp == 0) RG_GIVE(DB / 2, DB) else RG_GIVE(0, DB / 2)
            __syncthreads();
            const float2 other = ml[(grp ^ 1) * 256];
            m = fmaxf(m_run, other.x);
            w_own = fast_exp2((m_run - m) * c);
            w_other = fast_exp2((other.x - m) * c);
            l_tot = w_own * l_run + w_other * other.y;
        }
        if (q_row < a.n_q) {
            const float inv = 1.0f / l_tot;
            // partial result: unnormalised O, maximum (log2 domain, as the merge kernel expects) and sum
            const int64_t prow = ranged ? static_cast<int64_t>(slot) * QW + (q_row - q_tile * QW) : (static_cast<int64_t>(slot) * a.heads + head) * a.n_q_pad + q_row;
            float* pp = a.part + prow * (D + 4);
            if (SHARE) RG_FINISH(0, DB)
            else if (grp == 0) RG_FINISH(0, DB / 2)
            else RG_FINISH(DB / 2, DB)
            if (!whole && (SHARE || grp == 0) && lh == 0) { pp[D] = m * c; pp[D + 1] = l_tot; }
        }
#undef RG_FINISH
#undef RG_GIVE
#undef RG_PART
        left -= n;
        if (!ranged || left <= 0) break;
        __syncthreads();   // the results have been read before the next query tile's first copies
        slot |= 1;         // only the last query tile of a range can be partial from here on
        tile_begin = 0;
        tile_end = left < n_tiles ? left : n_tiles;
        if (++q_tile == a.q_tiles) { q_tile = a.q_full; ++head; }
    }
}

// Merges the split-KV partial results: out = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s.  RANGED: of the even ranges
// that met in a query tile (QW rows, tiles from q_full on; n_q counts the rows from there), in key order; query tiles
// that one range covered are finished already.
template <int D, int QW, bool RANGED, int MAXS>
__global__ void __launch_bounds__(kThreads)
attn_combine_kernel(const float* __restrict__ part, int splits, int heads, int n_q, int n_q_pad, bf16_t* __restrict__ out, int ldo,
                    int q_full, int q_rest, int n_tiles, int range) {
    // one thread per (query, head, 4 d's)
    constexpr int G = D / 4;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    const int64_t total = static_cast<int64_t>(n_q) * heads * G;
    if (gid >= total) return;
    const int g = static_cast<int>(gid % G);
    const int head = static_cast<int>((gid / G) % heads);
    const int qrow = static_cast<int>(gid / (static_cast<int64_t>(G) * heads));
    int w0 = 0, w0_slot = 0;
    if (RANGED) {
        const int first = (head * q_rest + qrow / QW) * n_tiles;      // this query tile's place in the list of key tiles
        w0 = first / range;
        splits = (first + n_tiles - 1) / range - w0 + 1;
        if (splits == 1) return;
        w0_slot = 2 * w0 + (w0 * range / n_tiles == first / n_tiles ? 0 : 1);   // later ranges start inside this query tile: slot 0
    }
    // every split's row is requested before the first value is used; a wave's loads of one split are contiguous
    float ms[MAXS], ls[MAXS];
    f32x4 val[MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) {
            const int64_t prow = RANGED ? static_cast<int64_t>(s == 0 ? w0_slot : 2 * (w0 + s)) * QW + qrow % QW : (static_cast<int64_t>(s) * heads + head) * n_q_pad + qrow;
            const float* pp = part + prow * (D + 4);
            const float2 ml = *reinterpret_cast<const float2*>(pp + D);
            ms[s] = ml.x; ls[s] = ml.y;
            val[s] = *reinterpret_cast<const f32x4*>(pp + 4 * g);
        }
    // No partial result is left out: one without keys, or whose scores are all -inf, has a sum of zero under a finite maximum and
    // adds nothing, and one whose sum is NaN (a NaN key, an overflowing score) has to make the row NaN as it does unsplit.
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) m = fmaxf(m, ms[s]);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) {
            const float w = fast_exp2(ms[s] - m);
            l += w * ls[s];
            acc[0] += w * val[s][0]; acc[1] += w * val[s][1]; acc[2] += w * val[s][2]; acc[3] += w * val[s][3];
        }
    const float inv = 1.0f / l;
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = static_cast<__bf16>(acc[e] * inv);
    *reinterpret_cast<bf16x4*>(out + static_cast<int64_t>(qrow + (RANGED ? q_full * QW : 0)) * ldo + head * D + 4 * g) = pk;
}

// The same sums as a function, for the kernel below: put() takes the g-th four values of a head's row, unless one range covered its query tile.  attn_combine_kernel keeps its own
// text, whose branches past the last split the compiler does not turn into selects: with up to 32 splits, 33 queries on 2596 keys, 9.15 us against 9.38 with this function and 13.4
// with loops that break.
struct Partials { const float* part; int splits, heads, n_q_pad, q_full, q_rest, n_tiles, range; };
template <int D, int QW, bool RANGED, int MAXS, typename Put>
__device__ __forceinline__ void merge_partials(const Partials& p, int qrow, int head, int g, Put put) {
    int splits = p.splits, w0 = 0, w0_slot = 0;
    if (RANGED) {
        const int first = (head * p.q_rest + qrow / QW) * p.n_tiles;      // this query tile's place in the list of key tiles
        w0 = first / p.range;
        splits = (first + p.n_tiles - 1) / p.range - w0 + 1;
        if (splits == 1) return;
        w0_slot = 2 * w0 + (w0 * p.range / p.n_tiles == first / p.n_tiles ? 0 : 1);   // later ranges start inside this query tile: slot 0
    }
    // every split's row is requested before the first value is used; a wave's loads of one split are contiguous
    float ms[MAXS], ls[MAXS];
    f32x4 val[MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) {
            const int64_t prow = RANGED ? static_cast<int64_t>(s == 0 ? w0_slot : 2 * (w0 + s)) * QW + qrow % QW : (static_cast<int64_t>(s) * p.heads + head) * p.n_q_pad + qrow;
            const float* pp = p.part + prow * (D + 4);
            const float2 ml = *reinterpret_cast<const float2*>(pp + D);
            ms[s] = ml.x; ls[s] = ml.y;
            val[s] = *reinterpret_cast<const f32x4*>(pp + 4 * g);
        }
    // No partial result is left out: one without keys, or whose scores are all -inf, has a sum of zero under a finite maximum and
    // adds nothing, and one whose sum is NaN (a NaN key, an overflowing score) has to make the row NaN as it does unsplit.
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) m = fmaxf(m, ms[s]);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
        if (s < splits) {
            const float w = fast_exp2(ms[s] - m);
            l += w * ls[s];
            acc[0] += w * val[s][0]; acc[1] += w * val[s][1]; acc[2] += w * val[s][2]; acc[3] += w * val[s][3];
        }
    const float inv = 1.0f / l;
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = static_cast<__bf16>(acc[e] * inv);
    put(pk);
}
// The merge and the row's E4M3 codes (quantize_rows_fp8_kernel, bit for bit) in one pass, a workgroup per row: the merged rows' way out and back and one launch fall away.
// A block's us, separate -> here (24 heads, 4608 keys): 100 rows 103 -> 99-105, 205 rows 121.6 -> 115-119, 820 rows 253.8 -> 249.5, 3000 rows 740 -> 740; 8 heads: 100 rows 55.4 -> 51.4,
// 820 rows 91.0 -> 88.6, 24 rows 50.4 -> 50.8.
constexpr int kCodesColumns = 4096, kCodesRanges = 8;
template <int D, int QW, bool RANGED>
__global__ void __launch_bounds__(kThreads)
attn_combine_codes_kernel(const float* __restrict__ part, int splits, int heads, int n_q_pad, int q_full, int q_rest, int n_tiles, int range,
                          bf16_t* __restrict__ out, int ldo, uint8_t* __restrict__ codes, float* __restrict__ scale, int keep_out) {
    const Partials p = {part, splits, heads, n_q_pad, q_full, q_rest, n_tiles, range};
    constexpr int G = D / 4, PIECES = kCodesColumns / 4 / kThreads;
    __shared__ float most[kThreads / 64];
    const int row = blockIdx.x, pieces = p.heads * G;
    float x[PIECES][4];
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
        const int piece = i * kThreads + threadIdx.x;
        if (piece < pieces) {
            const int head = piece / G, g = piece % G;
            bf16_t* to = out + static_cast<int64_t>(row) * ldo + 4 * piece;
            bf16x4 pk;
            bool merged = false;
            if (!RANGED || row >= q_full * QW)
                merge_partials<D, QW, RANGED, kCodesRanges>(p, row - (RANGED ? q_full * QW : 0), head, g, [&](bf16x4 sum) { pk = sum; merged = true; });
            if (!merged) pk = *reinterpret_cast<const bf16x4*>(to);
            else if (keep_out) *reinterpret_cast<bf16x4*>(to) = pk;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[i][e] = static_cast<float>(pk[e]);
                amax = __builtin_fmaxf(amax, __builtin_fabsf(x[i][e]));
            }
        }
    }
    amax = wave_max(amax);
    if ((threadIdx.x & 63) == 0) most[threadIdx.x >> 6] = amax;
    __syncthreads();
    amax = __builtin_fmaxf(__builtin_fmaxf(most[0], most[1]), __builtin_fmaxf(most[2], most[3]));
    const bool live = amax > 0.f;
    const float mult = live ? kE4M3Max / amax : 1.0f;
    if (threadIdx.x == 0) scale[row] = live ? amax / kE4M3Max : 1.0f;
    unsigned* to = reinterpret_cast<unsigned*>(codes + static_cast<int64_t>(row) * 4 * pieces);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
        const int piece = i * kThreads + threadIdx.x;
        if (piece < pieces) to[piece] = fp8_codes4(x[i], mult);
    }
}

// ---------------------------------------------------------------- how a call is dealt to workgroups
//
// NARROW: workgroups of four waves of 32 queries, two per CU, that run freely.  With head dimension 64 the softmax bounds, and groups that take turns at
// the matrix cores would leave the vector units idle instead.  SPLIT and SHARE (head dimension 128): see AttnTile, one workgroup per CU; there NARROW stays
// the fastest where few key tiles do not pay for their longer start and where the query tiles are a little more than a pass.  DEALT: few queries on not
// too many keys.
enum { FORM_SPLIT = 0, FORM_SHARE = 1, FORM_DEALT = 2, FORM_NARROW = 3 };
// what comparisons force (0: nothing): a form, as its number + 1, and which ranges of keys
struct Forced { int form, ranges; bool allows(int f) const { return form == 0 || form == f + 1; } };
int form_queries(int form) { return form == FORM_DEALT ? 32 : form == FORM_SHARE ? 256 : 128; }

// `splits` equal key ranges per query tile (in SPLIT workgroups an even number of them goes in pairs, a range to each wave group), or (range > 0)
// even ranges of `range` key tiles behind the first q_full query tiles of every head.  whole: those as tiles of 128 queries; SHARE
// workgroups take them in pairs and leave an odd last one to the ranges.
struct AttnPlan { int form, splits, range, range_wgs, q_full, whole; };

// What plan_ranges ranks numbers of equal key ranges by, in microseconds, where the unsplit query tiles leave CUs empty.  A key
// tile costs `alone` on a CU that holds four waves, `pair` and more where an XCD's 32 CUs hold up to twice that each, `pass` in a full pass of
// 64; then the merge launch, the partial rows' way out and back, and what more ranges cost the merge kernel.  Fitted to forced ranges of 1-32 over 105
// shapes, for rows named by an index list (which lie apart, so that a tile waits longer where nothing else fills the CU) to 409 calls: about 1 % behind
// the best range count on average.
template <int D>
double range_time(int source, int q_tiles, int heads, int n_q, int n_tiles, int s) {
    struct Cost { double fixed, alone, pair, more, pass, merge, mb, range, many; };
    constexpr Cost narrow[2] = {{3.9, 0.68, 0.95, -0.05, 0.64, 1.3, 0.58, 0.35, 1.2}, {4.5, 0.91, 1.24, 0.23, 0.93, 2.9, 0.60, 0.0, 0.0}};
    constexpr Cost wide = {6.1, 1.00, 1.47, 0.39, 1.60, 3.4, 0.33, 0.28, 1.2};
    const Cost& c = D == 64 ? narrow[source == SRC_INDEXED] : wide;
    const int per = (n_tiles + s - 1) / s;
    const int per_xcd = (heads * s + 7) / 8 * q_tiles, full = per_xcd / 64, rem = per_xcd % 64;
    double t = c.fixed + full * c.pass * (per + 2);
    if (rem > 0) t += per * (rem <= 32 ? c.alone : c.pair + c.more * (rem - 32) / 32.0);
    if (s > 1) t += c.merge + c.mb * (s * 4.0e-6 * n_q * heads * (D + 4)) + c.range * s + (s > 8 ? c.many : 0.0);
    return t;
}

// Key ranges of workgroups of four waves: what calls with head dimension 64 take, and wide E4M3 blocks (head dimension 128, keys in one array).  Those blocks' two
// quantisations turn another rounding of the attention's results by one bf16 ulp into whole code steps (1.8 % of a 3072-wide double-stream block's output, 0.7 % at width 1024),
// and the weights are rounded relative to their range's reference; so other key ranges would change that mode's results by that much.
template <int D>
AttnPlan plan_ranges(int source, int n_q, int n_keys, int heads, int force_splits, size_t part_bytes) {
    constexpr int QW = 128;
    const int q_tiles = (n_q + QW - 1) / QW;
    const int n_tiles = (n_keys + KT - 1) / KT;
    AttnPlan plan = {D == 128 ? FORM_SPLIT : FORM_NARROW, 1, 0, 0, q_tiles, q_tiles};
    const double slots = 512.0;
    const double wgs = static_cast<double>(q_tiles) * heads;
    double best = 0.0;
    const bool few = static_cast<int64_t>(q_tiles) * heads <= 256;   // at most one workgroup per CU before the split: a model of its own
    const size_t part_row_set = static_cast<size_t>(heads) * n_q * (D + 4) * sizeof(float);
    for (int s = 1; few && s <= kMaxSplits && (s == 1 || (s * 2 <= n_tiles && s * part_row_set <= part_bytes)); ++s) {
        const double t = range_time<D>(source, q_tiles, heads, n_q, n_tiles, s);
        if (s == 1 || t < (source == SRC_INDEXED ? 0.97 : 1.0) * best) { best = t; plan.splits = s; }   // no cost per range there: nearly equal goes to fewer
    }
    for (int s = 1; !few && s <= 8 && (s == 1 || s * 4 <= n_tiles); ++s) {
        const double load = wgs * s / slots;
        const double passes = load <= 1.0 ? 1.0 : 0.5 * (ceil(load) + load);   // a last, partly filled pass runs faster
        const double fill = wgs * s <= 256.0 ? 0.68 : 1.0;                      // a CU with one workgroup runs it faster
        double t = passes * ((n_tiles + s - 1) / s + 4) * 2.0 * fill;
        if (s > 1) t += 3.0 + 1.5 * static_cast<double>(s) * n_q * heads * (D + 4) * 8.0 / 4.0e6;
        if (s == 1 || t < best) { best = t; plan.splits = s; }
    }
    if (force_splits > 0 && force_splits * 2 <= n_tiles) plan.splits = force_splits;
    if (plan.splits > 1 && plan.splits * part_row_set > part_bytes) plan.splits = 1;
    // Even ranges, where equal ones leave the last pass of workgroups nearly empty: each of the last `slots` workgroups takes the same number of
    // consecutive key tiles of what whole passes of unsplit query tiles leave over.  At most eight ranges meet in a query tile.
    if (D == 128 && force_splits == 0) {
        const int whole = heads % 8 == 0 ? static_cast<int>(wgs / slots) : 0;    // other head counts: unsplit tiles would fill the XCDs unevenly
        const int q_full = static_cast<int>(whole * slots) / heads;
        const int64_t units = static_cast<int64_t>(heads) * (q_tiles - q_full) * n_tiles;
        int64_t range = (units + static_cast<int64_t>(slots) - 1) / static_cast<int64_t>(slots);
        const int64_t least = (n_tiles + 6) / 7 > 4 ? (n_tiles + 6) / 7 : 4;
        if (range < least) range = least;
        const int64_t range_wgs = (units + range - 1) / range;
        const size_t need = static_cast<size_t>(range_wgs) * 2 * QW * (D + 4) * sizeof(float);
        const double t = 1.9 * whole * (n_tiles + 4) + 2.3 * static_cast<double>(range) + 16.0;
        if (units > 0 && units < (1 << 30) && need <= part_bytes && t < 0.97 * (few ? 1.0 : 0.9) * best)
            plan = {FORM_SPLIT, 1, static_cast<int>(range), static_cast<int>(range_wgs), q_full, q_full};
    }
    return plan;
}

// Microseconds of a call with equal key ranges.  A pass is 32 workgroups on each of the 8 XCDs, one per CU (NARROW: 64); it costs a start and `units` of work per workgroup (key
// tiles; DEALT: blocks of 32 keys of a wave) at `full`, the last one at `part` + `fill` x its filling, or where it fills no more than half of itself `low` + `low_fill` x
// filling (only NARROW differs there: one workgroup per CU or two); then the merge launch, the partial rows' way out and back, what more ranges cost it, and the
// keys' and the queries' megabytes.  Fitted to 23000 forced plans of 2077 calls (16-9500 queries, 33-16000 keys, 8, 12, 16 and 24 heads, all three key sources), each timed on keys
// that no cache held, as those of a wide model's blocks are not, and on keys that the last level did: over 500 other calls the choice is 1.0 % behind the best of 10 to 30
// plans on average and 24 % at most.  Costs fitted to calls of 500 keys and more, and without NARROW among the forms, were 5.9 % behind and up to 1.27 times as slow as
// NARROW alone.  us, 24 heads, NARROW alone / those costs / now: 6098 x 567 66 / 80 / 68, 2777 x 513 39.5 / 47 / 38, 2700 x 2700 103 / 117 / 103, 1409 x 1409 54 / 62 / 40,
// 6000 x 2000 166 / 176 / 167; 713 x 122 8.8 / 14.2 / 9.8.
struct FormCost { double fixed, pass, full, part, fill, low, low_fill, merge, mb, range, keys, rows; };
constexpr FormCost kFormCosts[2][4] = {   // keys in one or two arrays, by index list; SPLIT, SHARE, DEALT, NARROW
    {{5.809, 1.96, 0.833, 0.592, 0.124, 0.592, 0.124, 3.194, 0.393, 0.032, 0.031, 0.365}, {7.184, 0.0, 1.6, 0.828, 0.595, 0.828, 0.595, 2.816, 0.384, 0.0, 0.0, 0.429},
     {1.926, 3.274, 1.237, 1.524, 0.0, 1.524, 0.0, 3.107, 0.34, 0.061, 0.092, 0.298}, {5.078, 0.0, 1.754, 1.302, 0.6, 1.028, 0.136, 2.83, 0.326, 0.047, 0.027, 0.241}},
    {{6.406, 4.106, 0.889, 0.677, 0.082, 0.677, 0.082, 3.65, 0.378, 0.0, 0.066, 0.415}, {8.651, 0.858, 1.686, 0.993, 0.521, 0.993, 0.521, 2.816, 0.403, 0.0, 0.0, 0.459},
     {1.987, 3.986, 1.543, 1.853, 0.0, 1.853, 0.0, 2.681, 0.353, 0.233, 0.067, 0.45}, {5.002, 0.0, 2.109, 1.901, 0.388, 1.424, 0.006, 2.804, 0.321, 0.063, 0.043, 0.268}}};
constexpr FormCost kDealtNarrow[2] = {   // head dimension 64, DEALT
    {3.03, 1.87, 0.85, 0.61, 0.10, 0.61, 0.10, 3.07, 0.62, 0.0, 0.0, 0.0}, {1.04, 4.36, 0.97, 0.97, 0.00, 0.97, 0.00, 3.01, 0.51, 0.0, 0.0, 0.0}};

template <int D>
double form_time(int form, bool indexed, int n_q, int heads, int n_tiles, int wgs) {   // wgs: workgroups per query tile
    const FormCost& c = D == 64 ? kDealtNarrow[indexed] : kFormCosts[indexed][form];
    const int q_tiles = (n_q + form_queries(form) - 1) / form_queries(form), slots = form == FORM_NARROW ? 64 : 32;
    const int per = (n_tiles + wgs - 1) / wgs;
    // DEALT: between the blocks of the busiest wave and of the average one
    const double units = form == FORM_DEALT ? 0.5 * ((2 * per + 7) / 8 + (D == 64 ? (2 * per + 7) / 8 : per / 4.0)) : per;
    const int per_xcd = (heads * wgs + 7) / 8 * q_tiles, full = per_xcd / slots, rem = per_xcd % slots;
    const double filling = static_cast<double>(rem) / slots;
    double t = c.fixed + c.pass * (full + (rem > 0)) + c.full * units * full + 4.0e-6 * heads * D * (c.keys * n_tiles * KT + c.rows * n_q);
    if (rem > 0) t += units * (2 * rem > slots ? c.part + c.fill * filling : c.low + c.low_fill * filling);
    if (wgs > 1) t += c.merge + c.mb * wgs * 4.0e-6 * n_q * heads * (D + 4) + c.range * wgs;
    return t;
}

// The same for even ranges on 256 workgroups (NARROW: 512) behind q_full query tiles of every head: `pass` and `tile` for whole passes of those, `again` for the
// share of ranges that run on into another query tile, `full` a key tile of the ranges where they fill a pass, else `part` x their filling.
struct EvenCost { double fixed, pass, again, tile, full, part, mb, keys; };
constexpr EvenCost kEvenCosts[2][4] = {
    {{14.255, 12.951, 2.717, 0.858, 0.896, 1.043, 0.519, 0.149}, {15.843, 16.556, 0.0, 1.637, 1.676, 1.73, 0.436, 0.007}, {}, {10.086, 6.764, 0.0, 1.894, 2.054, 1.995, 0.337, 0.06}},
    {{17.268, 18.649, 7.781, 0.94, 0.996, 1.194, 0.524, 0.189}, {18.092, 20.528, 2.193, 1.717, 1.764, 1.894, 0.469, 0.07}, {}, {11.37, 6.897, 0.0, 2.311, 2.562, 2.574, 0.315, 0.044}}};
double even_time(int form, bool indexed, int n_q, int heads, int n_tiles, int q_full, int range, int range_wgs) {
    const EvenCost& c = kEvenCosts[indexed][form];
    const double slots = form == FORM_NARROW ? 512.0 : 256.0, whole = heads * q_full / slots, filling = (range_wgs + 7) / 8 / (slots / 8.0);
    double t = c.fixed + whole * (c.pass + c.tile * n_tiles) + c.again * (range - 1) / n_tiles + range * (filling >= 1.0 ? c.full : c.part * filling);
    t += c.keys * 4.0e-6 * n_tiles * KT * heads * 128;
    return t + c.mb * 4.0e-6 * (n_q - q_full * form_queries(form)) * static_cast<double>(heads) * (128 + 4) * (static_cast<double>(n_tiles) / range + 1.0);
}

// Ranges that a second launch joins have to be faster by so much: among a block's launches that one waits longer than back to back (820 queries on 8704 keys, 24
// heads, in the step: 353 us in three ranges that the costs alone take, 347 unsplit; by themselves 100 and 97), and alone the choice is as good with it.
constexpr double kMergeMargin = 1.04;

// DEALT keeps the rows that an index list names in LDS
bool dealt_fits(int source, int n_tiles, int wgs) { return source != SRC_INDEXED || (n_tiles + wgs - 1) / wgs * KT <= kDealtKeys; }

// Head dimension 128: the fastest of the forms, equal or even ranges; no ranges at all (splits 0) where nothing fits what is forced.
AttnPlan plan_wide(int source, int n_q, int n_keys, int heads, size_t part_bytes, Forced forced) {
    constexpr int D = 128;
    const bool indexed = source == SRC_INDEXED;
    const int n_tiles = (n_keys + KT - 1) / KT, tiles128 = (n_q + 127) / 128;
    const size_t part_row_set = static_cast<size_t>(heads) * n_q * (D + 4) * sizeof(float);
    AttnPlan plan = {};
    double best = 0.0;
    for (int form = FORM_SPLIT; form <= FORM_NARROW; ++form) {
        if (!forced.allows(form) || forced.ranges > REGIONE_RANGES_EQUAL) continue;
        const int q_tiles = (n_q + form_queries(form) - 1) / form_queries(form);
        for (int wgs = 1; wgs <= (form == FORM_SPLIT ? kMaxSplits / 2 : kMaxSplits); ++wgs) {
            if (wgs > 1 && (wgs * 2 > n_tiles || wgs * part_row_set > part_bytes)) break;
            if (form == FORM_DEALT && !dealt_fits(source, n_tiles, wgs)) continue;
            const double t = form_time<D>(form, indexed, n_q, heads, n_tiles, wgs) * (wgs > 1 ? kMergeMargin : 1.0);
            if (plan.splits > 0 && t >= best) continue;
            best = t;
            plan = {form, form == FORM_SPLIT && n_tiles > 1 ? 2 * wgs : wgs, 0, 0, q_tiles, tiles128};
        }
    }
    for (int form = FORM_SPLIT; form <= FORM_NARROW; ++form) {
        if (!forced.allows(form) || forced.ranges == REGIONE_RANGES_EQUAL || form == FORM_DEALT) continue;
        const int slots = form == FORM_NARROW ? 512 : 256;
        for (int pass = 0; pass < 2; ++pass) {   // with and without whole passes of unsplit query tiles in front
            const int qw = form_queries(form), q_tiles = (n_q + qw - 1) / qw;
            const int whole = heads % 8 == 0 ? q_tiles * heads / slots : 0;
            if (pass > 0 && whole == 0) break;
            const int tiles = pass == 0 ? slots * whole / heads * (qw / 128) : 0;
            const int q_full = tiles / (qw / 128);
            if (forced.ranges > 0 && forced.ranges != (q_full > 0 ? REGIONE_RANGES_EVEN_BEHIND : REGIONE_RANGES_EVEN)) continue;
            const int64_t units = static_cast<int64_t>(heads) * (q_tiles - q_full) * n_tiles;
            if (units <= 0 || units >= (1 << 30)) continue;
            int64_t range = (units + slots - 1) / slots;
            const int64_t least = (n_tiles + kMaxSplits - 3) / (kMaxSplits - 2);     // as many ranges in a query tile as the merge kernel takes
            range = range < 2 ? 2 : range;
            range = range < least ? least : range;
            const int64_t range_wgs = (units + range - 1) / range;
            if (static_cast<size_t>(range_wgs) * 2 * qw * (D + 4) * sizeof(float) > part_bytes) continue;
            const double t = even_time(form, indexed, n_q, heads, n_tiles, q_full, static_cast<int>(range), static_cast<int>(range_wgs)) * kMergeMargin;
            if (plan.splits > 0 && t >= best) continue;
            best = t;
            plan = {form, 1, static_cast<int>(range), static_cast<int>(range_wgs), q_full, tiles};
        }
    }
    return plan;
}

// keep_ranges: see plan_ranges
AttnPlan plan_attention(const regione_ctx* ctx, int source, int n_q, int n_keys, int heads, int d, bool keep_ranges) {
    const int n_tiles = (n_keys + KT - 1) / KT, forced = ctx->attn_force_splits;
    const Forced asked = {ctx->attn_force_form, ctx->attn_force_ranges};
    if (d == 128 && !keep_ranges && forced == 0) {
        const AttnPlan plan = plan_wide(source, n_q, n_keys, heads, ctx->attn_part_bytes, asked);
        return plan.splits > 0 ? plan : plan_wide(source, n_q, n_keys, heads, ctx->attn_part_bytes, {0, 0});
    }
    AttnPlan plan = d == 64 ? plan_ranges<64>(source, n_q, n_keys, heads, forced, ctx->attn_range_bytes) : plan_ranges<128>(source, n_q, n_keys, heads, forced, ctx->attn_range_bytes);
    if (forced > 0) {   // that many equal ranges in the form asked for, if it has such workgroups
        const int form = asked.form - 1;
        if (form == FORM_DEALT ? dealt_fits(source, n_tiles, plan.splits) : d == 128 && form >= 0) plan.form = form;
        plan.q_full = (n_q + form_queries(plan.form) - 1) / form_queries(plan.form);
        return plan;
    }
    // the same ranges in the fastest form, or (head dimension 64) other ranges in DEALT workgroups
    if (d == 128) {
        plan.form = FORM_NARROW;
        if (plan.range > 0) return plan;
        double best = form_time<128>(FORM_NARROW, false, n_q, heads, n_tiles, plan.splits);
        for (int form = FORM_SPLIT; form <= FORM_SHARE; ++form) {
            const int pairs = form == FORM_SPLIT && plan.splits % 2 == 0 ? plan.splits / 2 : plan.splits;
            const double t = form_time<128>(form, false, n_q, heads, n_tiles, pairs);
            if (t >= best) continue;
            best = t;
            plan.form = form;
        }
    } else if (asked.allows(FORM_DEALT) && (asked.form > 0 || static_cast<int64_t>(plan.whole) * heads <= 256)) {
        double best = asked.form > 0 ? DBL_MAX : range_time<64>(source, plan.whole, heads, n_q, n_tiles, plan.splits);
        for (int wgs = 1; wgs <= kMaxSplits && (wgs == 1 || (wgs * 2 <= n_tiles && wgs * sizeof(float) * n_q * heads * (64 + 4) <= ctx->attn_part_bytes)); ++wgs) {
            const double t = form_time<64>(FORM_DEALT, source == SRC_INDEXED, n_q, heads, n_tiles, wgs);
            if (t >= best || !dealt_fits(source, n_tiles, wgs)) continue;
            best = t;
            plan.form = FORM_DEALT;
            plan.splits = wgs;
        }
    }
    plan.q_full = (n_q + form_queries(plan.form) - 1) / form_queries(plan.form);
    return plan;
}

template <int D>
int launch_attention(regione_ctx* ctx, AttnArgs a, bool keep_ranges, RowCodes* row_codes) {
    const int n_tiles = (a.n0 + a.n1 + KT - 1) / KT;
    const int source = a.idx1 ? SRC_INDEXED : a.n0 == 0 || a.n1 == 0 ? SRC_CONTIG : SRC_TWO;
    a.ld = a.n0 > 0 ? a.ldkv0 : a.ldkv1;
    // a lane's byte offset (inside a tile, or with an index list inside the cache) has to fit 32 bits
    a.fast = (a.n0 == 0 || a.n1 == 0 || a.ldkv0 == a.ldkv1) && ((a.idx1 ? static_cast<int64_t>(a.rows1) : KT) + 1) * a.ld * 2 < (int64_t{1} << 31);
    const AttnPlan plan = plan_attention(ctx, source, a.n_q, a.n0 + a.n1, a.heads, D, keep_ranges);
    const int qw = form_queries(plan.form);
    a.tiles_per_split = (n_tiles + plan.splits - 1) / plan.splits;
    a.halves = plan.form == FORM_SPLIT && plan.range == 0 && plan.splits % 2 == 0;
    a.splits = a.halves ? plan.splits / 2 : plan.splits;
    a.n_q_pad = a.n_q;
    a.part = ctx->attn_part;
    a.q_tiles = (a.n_q + qw - 1) / qw;
    a.q_full = plan.q_full;
    a.full_blocks = (a.heads * a.splits + 7) / 8 * plan.q_full * 8;
    a.range = plan.range;
    a.range_wgs = plan.range_wgs;
    const dim3 grid(static_cast<unsigned>(a.full_blocks + (a.range_wgs + 7) / 8 * 8));
    const bool indexed = source == SRC_INDEXED, ranged = a.range_wgs > 0;
    using Kernel = void (*)(AttnArgs);
    Kernel kernel;
    size_t lds_bytes;
    int which;
    if (plan.form == FORM_DEALT) {
        kernel = indexed ? attn_dealt_kernel<D, true> : attn_dealt_kernel<D, false>;
        lds_bytes = DealtTile<D>::LIST_BASE + (indexed ? kDealtKeys * sizeof(int32_t) : 0);
        which = 8 + indexed;
    } else if (plan.form == FORM_NARROW) {
        static constexpr Kernel kernels[3][2] = {{attn_narrow_kernel<D, SRC_CONTIG, false>, attn_narrow_kernel<D, SRC_CONTIG, D == 128>},
                                                 {attn_narrow_kernel<D, SRC_TWO, false>, attn_narrow_kernel<D, SRC_TWO, D == 128>},
                                                 {attn_narrow_kernel<D, SRC_INDEXED, false>, attn_narrow_kernel<D, SRC_INDEXED, D == 128>}};
        const int way = source == SRC_CONTIG && !a.fast ? SRC_TWO : source;
        kernel = kernels[way][ranged];
        lds_bytes = 2u * 2 * KT * D * sizeof(bf16_t);
        which = 10 + 2 * way + ranged;
    } else if constexpr (D == 128) {
        static constexpr Kernel kernels[8] = {attn_kvcache_kernel<D, false, false, false>, attn_kvcache_kernel<D, false, false, true>,
                                              attn_kvcache_kernel<D, false, true, false>, attn_kvcache_kernel<D, false, true, true>,
                                              attn_kvcache_kernel<D, true, false, false>, attn_kvcache_kernel<D, true, false, true>,
                                              attn_kvcache_kernel<D, true, true, false>, attn_kvcache_kernel<D, true, true, true>};
        const bool share = plan.form == FORM_SHARE;
        which = share * 4 + indexed * 2 + ranged;
        kernel = kernels[which];
        lds_bytes = share ? AttnTile<D, true>::LDS_BYTES : AttnTile<D, false>::LDS_BYTES;
    } else {
        RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention: no workgroups of form %d for head dimension %d", plan.form, D);
    }
    const uint32_t granted = 1u << (which + (D == 128 ? 0 : 16));
    if (!(ctx->lds_grant_mask & granted)) {   // more than 64 KiB of LDS has to be granted explicitly
        RG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes)));
        ctx->lds_grant_mask |= granted;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(plan.form == FORM_NARROW ? 256 : 512), lds_bytes, ctx->stream, a);
    RG_LAUNCH_CHECK();
    if (a.splits > 1 || ranged) {
        const int rows = a.n_q - (ranged ? a.q_full * qw : 0);
        const int64_t total = static_cast<int64_t>(rows) * a.heads * (D / 4);
        const dim3 merge_grid(static_cast<unsigned>((total + kThreads - 1) / kThreads));
        const bool many = (ranged ? (n_tiles - 1) / a.range + 2 : a.splits) > 8;
        if constexpr (D == 128) {
            if (row_codes && !many && a.heads * D <= kCodesColumns) {
                const auto merge = !ranged ? attn_combine_codes_kernel<D, 128, false> : qw == 256 ? attn_combine_codes_kernel<D, 256, true> : attn_combine_codes_kernel<D, 128, true>;
                hipLaunchKernelGGL(merge, dim3(static_cast<unsigned>(a.n_q)), dim3(kThreads), 0, ctx->stream, a.part, a.splits, a.heads, a.n_q_pad, a.q_full, a.q_tiles - a.q_full, n_tiles, a.range,
                                   a.out, a.ldo, row_codes->codes, row_codes->scale, row_codes->keep_out);
                RG_LAUNCH_CHECK();
                row_codes->done = true;
                return REGIONE_OK;
            }
            if (ranged) {
                const auto merge = qw == 256 ? (many ? attn_combine_kernel<D, 256, true, kMaxSplits> : attn_combine_kernel<D, 256, true, 8>)
                                             : (many ? attn_combine_kernel<D, 128, true, kMaxSplits> : attn_combine_kernel<D, 128, true, 8>);
                hipLaunchKernelGGL(merge, merge_grid, dim3(kThreads), 0, ctx->stream, a.part, 0, a.heads, rows, 0, a.out, a.ldo, a.q_full, a.q_tiles - a.q_full, n_tiles, a.range);
            }
        }
        if (!ranged)
            hipLaunchKernelGGL((many ? attn_combine_kernel<D, 128, false, kMaxSplits> : attn_combine_kernel<D, 128, false, 8>), merge_grid, dim3(kThreads), 0, ctx->stream,
                               a.part, a.splits, a.heads, rows, a.n_q_pad, a.out, a.ldo, 0, 0, 0, 0);
        RG_LAUNCH_CHECK();
    }
    return REGIONE_OK;
}

}  // namespace

extern "C" int regione_tune_attention(regione_ctx* ctx, int32_t key_splits) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_attention: null context");
    if (key_splits < 0 || key_splits > kMaxSplits) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_attention: key_splits=%d must be 0..32", key_splits);
    ctx->attn_force_splits = key_splits;
    return REGIONE_OK;
}

extern "C" int regione_tune_attention_form(regione_ctx* ctx, int32_t form, int32_t ranges) {
    static_assert(REGIONE_ATTN_TILES_128 == FORM_SPLIT + 1 && REGIONE_ATTN_TILES_256 == FORM_SHARE + 1 && REGIONE_ATTN_DEALT == FORM_DEALT + 1 && REGIONE_ATTN_FREE == FORM_NARROW + 1, "the same order");
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_attention_form: null context");
    if (form < 0 || form > REGIONE_ATTN_FREE || ranges < 0 || ranges > REGIONE_RANGES_EVEN_BEHIND) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_attention_form: form %d, ranges %d", form, ranges);
    ctx->attn_force_form = form;
    ctx->attn_force_ranges = ranges;
    return REGIONE_OK;
}

extern "C" int regione_attention_workgroups(regione_ctx* ctx, int32_t n_q, int32_t n_keys, int32_t heads, int32_t d, int32_t source, int32_t* form, int32_t* key_splits,
                                            int32_t* range_tiles) {
    if (!ctx || !form || !key_splits || !range_tiles) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_workgroups: null argument");
    if (n_q <= 0 || n_keys <= 0 || heads <= 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_workgroups: n_q=%d n_keys=%d heads=%d", n_q, n_keys, heads);
    if (ctx->f32 || (d != 64 && d != 128)) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention_workgroups: bf16 contexts and head dimensions of 64 or 128 (%d) only", d);
    if (source < REGIONE_KEYS_CONTIGUOUS || source > REGIONE_KEYS_WIDE_8BIT) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_workgroups: source %d", source);
    const bool wide8 = source == REGIONE_KEYS_WIDE_8BIT;
    const AttnPlan plan = plan_attention(ctx, wide8 ? SRC_CONTIG : source, n_q, n_keys, heads, d, wide8);
    *form = plan.form + 1;
    *key_splits = plan.splits;
    *range_tiles = plan.range;
    return REGIONE_OK;
}

extern "C" int regione_attention_plan(regione_ctx* ctx, int32_t n_q, int32_t n_keys, int32_t heads, int32_t d, int32_t source, int32_t* key_splits,
                                      int32_t* range_tiles, int32_t* whole_query_tiles) {
    if (!ctx || !key_splits || !range_tiles || !whole_query_tiles) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_plan: null argument");
    if (n_q <= 0 || n_keys <= 0 || heads <= 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_plan: n_q=%d n_keys=%d heads=%d", n_q, n_keys, heads);
    if (ctx->f32 || (d != 64 && d != 128)) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention_plan: bf16 contexts and head dimensions of 64 or 128 (%d) only", d);
    if (source != REGIONE_KEYS_CONTIGUOUS && source != REGIONE_KEYS_TWO && source != REGIONE_KEYS_INDEXED) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attention_plan: source %d", source);
    static_assert(REGIONE_KEYS_CONTIGUOUS == SRC_CONTIG && REGIONE_KEYS_TWO == SRC_TWO && REGIONE_KEYS_INDEXED == SRC_INDEXED, "the same order");
    const AttnPlan plan = plan_attention(ctx, source, n_q, n_keys, heads, d, false);
    *key_splits = plan.splits;
    *range_tiles = plan.range;
    *whole_query_tiles = plan.whole;
    return REGIONE_OK;
}

int rg_attention(regione_ctx* ctx, const void* q_any, int ldq, int n_q,
                 const void* k0_any, const void* v0_any, int ldkv0, int n0,
                 const void* k1_any, const void* v1_any, int ldkv1, int n1, const int32_t* idx1, int rows1,
                 int heads, int d, float scale, void* out_any, int ldo, bool keep_ranges, RowCodes* row_codes) {
    if (n_q <= 0) return REGIONE_OK;
    if (ctx->f32)
        return rg_attention_f32(ctx, static_cast<const float*>(q_any), ldq, n_q, static_cast<const float*>(k0_any), static_cast<const float*>(v0_any), ldkv0, n0,
                                static_cast<const float*>(k1_any), static_cast<const float*>(v1_any), ldkv1, n1, idx1, heads, d, scale, static_cast<float*>(out_any), ldo);
    const bf16_t* q = static_cast<const bf16_t*>(q_any);
    const bf16_t* k0 = static_cast<const bf16_t*>(k0_any); const bf16_t* v0 = static_cast<const bf16_t*>(v0_any);
    const bf16_t* k1 = static_cast<const bf16_t*>(k1_any); const bf16_t* v1 = static_cast<const bf16_t*>(v1_any);
    bf16_t* out = static_cast<bf16_t*>(out_any);
    if (n0 + n1 <= 0) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attention: %d queries but no key", n_q);
    if (d != 64 && d != 128) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attention: head dimension %d (64 or 128 supported)", d);
    if ((ldq & 7) || (ldo & 3) || (n0 > 0 && (ldkv0 & 7)) || (n1 > 0 && (ldkv1 & 7)))
        RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attention: row strides must keep 16-byte alignment");
    ProfScope prof(ctx, REGIONE_PROF_ATTENTION);
    AttnArgs a = {};
    a.q = q; a.ldq = ldq; a.n_q = n_q;
    a.k0 = k0; a.v0 = v0; a.ldkv0 = ldkv0; a.n0 = n0;
    a.k1 = k1; a.v1 = v1; a.ldkv1 = ldkv1; a.n1 = n1; a.idx1 = n1 > 0 ? idx1 : nullptr; a.rows1 = rows1;
    a.heads = heads;
    a.scale_log2e = (scale > 0.f ? scale : 1.0f / sqrtf(static_cast<float>(d))) * 1.4426950408889634f;
    a.out = out; a.ldo = ldo;
    if (d == 64) return launch_attention<64>(ctx, a, keep_ranges, row_codes);
    return launch_attention<128>(ctx, a, keep_ranges, row_codes);
}

extern "C" int regione_attn_kvcache(regione_ctx* ctx, const void* q, int32_t n_q,
                                    const void* k_fresh, const void* v_fresh, int32_t n_fresh,
                                    const void* k_cache, const void* v_cache, int32_t n_c,
                                    const int32_t* cache_index_opt, int32_t n_cache_index,
                                    int32_t heads, int32_t d, float scale, void* out) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: null context");
    if (n_q < 0 || n_fresh < 0 || n_c < 0 || heads <= 0 || n_cache_index < 0)
        RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: n_q=%d n_fresh=%d n_c=%d heads=%d", n_q, n_fresh, n_c, heads);
    if (d != 64 && d != 128) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "attn_kvcache: head dimension %d (64 or 128 supported)", d);
    if (n_q == 0) return REGIONE_OK;
    if (!q || !out) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: null q or out");
    if (n_fresh > 0 && (!k_fresh || !v_fresh)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: null fresh K/V");
    if (n_c > 0 && (!k_cache || !v_cache)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: null cache");
    const int n1 = cache_index_opt ? n_cache_index : n_c;
    if (cache_index_opt && n_c == 0 && n_cache_index > 0) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attn_kvcache: index list into an empty cache");
    if (n_fresh + n1 == 0) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "attn_kvcache: %d queries but no key", n_q);
    if (!rg_aligned16(q) || !rg_aligned16(out) || !rg_aligned16(k_fresh) || !rg_aligned16(v_fresh) || !rg_aligned16(k_cache) || !rg_aligned16(v_cache))
        RG_FAIL(REGIONE_ERR_INVALID_ARG, "attn_kvcache: tensors must be 16-byte aligned");
    const int ld = heads * d;
    return rg_attention(ctx, q, ld, n_q, k_fresh, v_fresh, ld, n_fresh, k_cache, v_cache, ld, n1, cache_index_opt, n_c, heads, d, scale, out, ld, false);
}
