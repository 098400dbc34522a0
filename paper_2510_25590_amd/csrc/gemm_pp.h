// GEMM kernel in which two groups of waves alternate between memory work and matrix-core work (gemm_pp_kernel below).
#pragma once
#include "gemm_epilogue.h"

namespace {

// Asynchronous global -> LDS copy: lane l writes 16 bytes at lds_base + 16*l from base + lane_off (bytes); counted in
// vmcnt.  Assembly, so that the compiler's wait-count pass does not wait for it before every later LDS read.
__device__ __forceinline__ void pp_copy16(unsigned lane_off, const void* base, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(lane_off), "s"(base), "s"(lds_base) : "memory", "m0");
}
// The same if I < n (wave-uniform): a copy that is not wanted keeps its place in the wave's count but moves nothing.  A
// branch around it instead costs tens of cycles per step (15-25 % of a narrow tile's time).
template <int I> __device__ __forceinline__ void pp_copy16_if(unsigned lane_off, const void* base, unsigned lds_base, int n) {
    asm volatile("s_cmp_gt_i32 %3, %4\n\ts_cselect_b64 exec, -1, 0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
                 :: "v"(lane_off), "s"(base), "s"(lds_base), "s"(n), "n"(I) : "memory", "m0", "scc");
}
template <int I0, int I1, int N> __device__ __forceinline__ void pp_copies_if(const unsigned (&lane_off)[N], const void* base, unsigned lds_base, int n) {
    if constexpr (I0 < I1) {
        pp_copy16_if<I0>(lane_off[I0], base, lds_base + I0 * 1024u, n);
        pp_copies_if<I0 + 1, I1, N>(lane_off, base, lds_base, n);
    }
}
// this wave's LDS reads are complete and at most N of its copies are still in flight
template <int N> __device__ __forceinline__ void pp_wait() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void pp_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// Partial sums travel between workgroups that may sit on different XCDs: 16-byte buffer accesses of device scope (the sc1
// bit of the cache policy), which neither stay in nor are served from an XCD's own L2.
constexpr int kDeviceScope = 16;
__device__ __forceinline__ auto pp_part_rsrc(float* base, int64_t floats) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, static_cast<int>(floats * 4), 0x00027000); }

// Units of work (tile, K split) are numbered so that each XCD (blockIdx.x % 8) owns a contiguous range of them: within it
// the row tiles of one column tile and K range follow each other and share the weights in that XCD's L2.
__device__ __forceinline__ bool pp_unit(int m_tiles, int n_tiles, int units_per_xcd, int group_rows, int splits, int& m_tile, int& n_tile, int& split) {
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int unit = xcd * units_per_xcd + local;
    if (local >= units_per_xcd || unit >= m_tiles * n_tiles * splits) return false;
    split = 0;
    if (splits == 1) {
        tile_coords(unit, m_tiles, n_tiles, group_rows, m_tile, n_tile);
    } else {
        m_tile = unit % m_tiles;
        const int rest = unit / m_tiles;
        n_tile = rest / splits;
        split = rest - n_tile * splits;
    }
    return true;
}
// Source offset (bytes inside a packed 32-column x 16-k weight block) of the 16 bytes that go to slot p of the block in LDS.
// Slot p holds column 16*g1 + 8*g0 + 4*jl + u, k half p >> 5, with the bits of p = (k half, jl, g0, g1 ^ jl, u): the
// sixteen columns that one fragment takes (see the epilogue's column order) then cover all 64 banks once.
__device__ __forceinline__ unsigned pp_w_source(unsigned p) {
    const unsigned jl = (p >> 4) & 1u, g0 = (p >> 3) & 1u, g1 = ((p >> 2) & 1u) ^ jl, u = p & 3u;
    return ((p >> 5) * 32u + 16u * g1 + 8u * g0 + 4u * jl + u) * 16u;
}
// LDS offset of lane `lane`'s 16 bytes of weight fragment jl of a 32-column x 32-k pair of blocks (1 KiB each, one after the other)
__device__ __forceinline__ unsigned pp_w_slot(unsigned lane, unsigned jl) {
    const unsigned kc = lane >> 4, u = lane & 3, g0 = (lane >> 2) & 1, g1 = (lane >> 3) & 1;
    return (kc >> 1) * 1024u + ((kc & 1) * 32u + jl * 16u + g0 * 8u + (g1 ^ jl) * 4u + u) * 16u;
}

// the largest divisor of F up to 8: fragments that are requested together when partial sums are added
constexpr int pp_group(int F) { int g = F < 8 ? F : 8; while (F % g) --g; return g; }

// The end of a tile: fragments [I0, I1) x CF of a wave.  K splits: every workgroup of a tile leaves its sums in `partial`
// (in register order: whole lines), and the one that arrives last adds all of them in split order (the same sums whoever
// is last) and goes on to the epilogue.  Nobody waits.  wave_slot: the wave's place among the tile's WAVES fragment sets.
template <int I0, int I1, int RF, int CF, int KIND, bool FP8>
__device__ __forceinline__ void pp_finish(f32x4 (&acc)[RF][CF], unsigned char* lds_raw, int wave_slot, int64_t part_floats, int tile, int split, int splits,
                                          float* __restrict__ partial, int* __restrict__ arrived, int M, int N, int m0, int n0w, const GemmEpilogue& ep) {
    const int lane = threadIdx.x & 63;
    if (splits > 1) {
        const auto rsrc = pp_part_rsrc(partial + static_cast<int64_t>(tile) * splits * part_floats, splits * part_floats);
        // (a resource of its own for the stores: with a scalar offset register the compiler does not keep the wait state that
        // a wide store needs before its data registers are overwritten, and the last lanes of each row of 16 stored the new value)
        const auto mine = pp_part_rsrc(partial + (static_cast<int64_t>(tile) * splits + split) * part_floats, part_floats);
        const unsigned part_off = static_cast<unsigned>(wave_slot * (RF * CF) * 64 + lane) * 16u;
        const unsigned part_bytes = static_cast<unsigned>(part_floats * 4);
#pragma unroll
        for (int i = I0; i < I1; ++i)
#pragma unroll
            for (int j = 0; j < CF; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), mine, part_off + (i * CF + j) * 1024u, 0, kDeviceScope);
        pp_wait<0>();              // the stores have reached the level all XCDs share ...
        __syncthreads();           // ... for every wave
        int* flag = reinterpret_cast<int*>(lds_raw);
        if (threadIdx.x == 0) *flag = __hip_atomic_fetch_add(arrived + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*flag != splits - 1) return;
        if (threadIdx.x == 0) __hip_atomic_store(arrived + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        // Fragments in groups of G, split after split; the next request (the last one repeats itself) is on its way while the sums of one are added.
        constexpr int F = (I1 - I0) * CF, G = pp_group(F);
        u32x4 v[2][G];
        auto request = [&](int b, int h, int s) __attribute__((always_inline)) {
            const int off = s * static_cast<int>(part_bytes) + h * 1024;
#pragma unroll
            for (int f = 0; f < G; ++f) v[b][f] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, part_off + (I0 * CF + f) * 1024u, off, kDeviceScope);
        };
        auto add = [&](int b, int h, int s) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < G; ++f) {
                f32x4& a = acc[I0 + (h + f) / CF][(h + f) % CF];
                const f32x4 x = __builtin_bit_cast(f32x4, v[b][f]);
                a = s == 0 ? x : a + x;
            }
        };
        request(0, 0, 0);
#pragma unroll
        for (int h = 0; h < F; h += G)
            for (int s = 0; s < splits; s += 2) {
                request(1, h, s + 1 < splits ? s + 1 : s);
                add(0, h, s);
                const bool more = s + 2 < splits;
                request(0, more || h + G >= F ? h : h + G, more ? s + 2 : 0);
                if (s + 1 < splits) add(1, h, s + 1);
            }
    }
    gemm_epilogue16<KIND, FP8, I0, I1, RF, CF>(acc, M, N, m0, n0w, ep);
}

// RF x CF fragments of 16 x 16 per wave, 2 x 4 waves: 32*RF rows x 64*CF columns per workgroup.
template <int RF, int CF> struct PpTile {
    static constexpr int ROWS = 32 * RF, COLS = 64 * CF, THREADS = 512;
    // 32-k halves of a K-step of 64 per phase: as many as make a phase of about 512 matrix-core cycles
    static constexpr int HP = (CF == 2 || RF == 4) ? 2 : 1;
    static constexpr int KB = 2 * HP;                              // 16-k blocks of the packed weights per phase
    static constexpr int W_SLOTS = HP == 2 ? 3 : 4;
    static constexpr unsigned A_STEP = ROWS * 128u;                // bytes of one K-step of the A tile
    static constexpr unsigned W_SLOT = (COLS / 32) * KB * 1024u;   // bytes of one phase of the W tile
    static constexpr unsigned W_BASE = 3u * A_STEP;
    static constexpr unsigned LDS_BYTES = W_BASE + W_SLOTS * W_SLOT;
    static constexpr int WC = (COLS / 32) * KB / 8;                // 1 KiB weight copies per wave and phase
    static constexpr int AC = (ROWS / 8 + 7) / 8;                  // 1 KiB A copies per wave and K-step
    static constexpr int A_WAVES = ROWS / 8 / AC;                  // waves that copy A rows (7 at 224 rows, else 8)
    static_assert(A_WAVES * AC * 8 == ROWS, "whole waves copy the A tile");
    static constexpr int64_t PART_FLOATS = static_cast<int64_t>(ROWS) * COLS;
};

template <int RF, int CF, int KIND, bool FP8>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_pp_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Wp,
               int M, int N, int K, int m_tiles, int n_tiles, int units_per_xcd, int group_rows,
               int splits, int steps_per_split, float* __restrict__ partial, int* __restrict__ arrived, GemmEpilogue ep) {
    using T = PpTile<RF, CF>;
    constexpr int HP = T::HP, KB = T::KB, WC = T::WC, AC = T::AC;
    static_assert(!FP8 || HP == 2, "the 8-bit instruction takes both 32-k halves of a step");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds_raw)));

    int n_tile, m_tile, split;
    if (!pp_unit(m_tiles, n_tiles, units_per_xcd, group_rows, splits, m_tile, n_tile, split)) return;
    const int m0_wg = m_tile * T::ROWS, n0 = n_tile * T::COLS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;

    const int ks_begin = split * steps_per_split;
    int n_steps = K / 64 - ks_begin;
    n_steps = n_steps < steps_per_split ? n_steps : steps_per_split;
    const int n_phases = n_steps * (2 / HP);

    // Copy sources.  A: a lane copies 16 bytes of one row; LDS rows are 128 bytes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7),
    // the swizzle applied on the global side (rows past M repeat the last row; their results are never stored).
    unsigned a_voff[AC];
#pragma unroll
    for (int i = 0; i < AC; ++i) {
        const int row = wave * 8 * AC + i * 8 + (lane >> 3);
        int r = m0_wg + row;
        r = r < M ? r : M - 1;
        a_voff[i] = static_cast<unsigned>(r - m0_wg) * static_cast<unsigned>(lda) * 2u + static_cast<unsigned>(((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const char* a_base = reinterpret_cast<const char*>(A + static_cast<int64_t>(m0_wg) * lda + static_cast<int64_t>(ks_begin) * 64);
    // W: a wave copies WC of the phase's 1 KiB blocks (32 columns x 16 k).
    const int n_blocks = (N + 31) >> 5;
    int nb = (n0 >> 5) + wave * WC / KB;
    nb = nb < n_blocks ? nb : n_blocks - 1;                        // blocks past N repeat the last block
    const char* w_base = reinterpret_cast<const char*>(Wp + (static_cast<int64_t>(nb) * (K >> 4) + static_cast<int64_t>(ks_begin) * 4 + wave * WC % KB) * 512);
    const unsigned w_voff = pp_w_source(lane);
    const unsigned a_dst = lds0 + static_cast<unsigned>(wave) * (AC * 1024u);
    const unsigned w_dst = lds0 + T::W_BASE + static_cast<unsigned>(wave) * (WC * 1024u);

    // fragment addresses: a lane of a fragment holds row (column) lane % 16 and eight k from 8 * (lane / 16) on
    unsigned a_off[2], w_off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        a_off[h] = static_cast<unsigned>(wm * (RF * 16) + l16) * 128u + static_cast<unsigned>(((4 * h + kc) ^ ((l16 >> 1) & 7)) << 4);
#pragma unroll
    for (int jl = 0; jl < 2; ++jl) w_off[jl] = T::W_BASE + static_cast<unsigned>(wn * (CF / 2)) * (KB * 1024u) + pp_w_slot(lane, jl);

    f32x4 acc[RF][CF];
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The copies of a phase are one packet: the W block set of the phase three (HP = 1) or two (HP = 2) phases ahead, and
    // its share of the A rows two K-steps ahead.  All buffers a packet writes were last read a full phase ago, by both
    // groups; a packet has landed before the phase that reads it when at most PENDING newer copies are in flight.
    // Packets past the end repeat the last step (their buffers are never read), so the counts are the same in every phase.
    int a_next = 0, w_next = 0;
    unsigned a_buf = 0, w_slot = 0;
    int a_live = (M - m0_wg - wave * (8 * AC) + 7) >> 3;           // rows past M are not copied, nor rows past the tile
    if (T::A_WAVES < 8 && wave >= T::A_WAVES) a_live = 0;
    constexpr int AE = (AC + 1) / 2;
    constexpr int PENDING = HP == 2 ? AC + WC : AC + 2 * WC;
#define PP_COPY_A(I0, I1)                                                                                   \
    {                                                                                                       \
        const char* src_ = a_base + static_cast<int64_t>(a_next < n_steps ? a_next : n_steps - 1) * 128;    \
        pp_copies_if<I0, I1>(a_voff, src_, a_dst + a_buf, a_live);                                          \
    }
#define PP_A_DONE() { ++a_next; a_buf = a_buf == 2 * T::A_STEP ? 0 : a_buf + T::A_STEP; }
#define PP_COPY_W()                                                                                         \
    {                                                                                                       \
        const char* src_ = w_base + static_cast<int64_t>(w_next < n_phases ? w_next : n_phases - 1) * (KB * 1024); \
        _Pragma("unroll") for (int c = 0; c < WC; ++c) pp_copy16(w_voff, src_ + c * 1024, w_dst + w_slot + c * 1024u); \
        ++w_next; w_slot = w_slot == (T::W_SLOTS - 1) * T::W_SLOT ? 0 : w_slot + T::W_SLOT;                 \
    }
#define PP_WAIT() { pp_wait<PENDING>(); __builtin_amdgcn_sched_barrier(0); }
    PP_COPY_A(0, AC) PP_A_DONE() PP_COPY_W()
    if (HP == 2) {
        PP_COPY_A(0, AC) PP_A_DONE() PP_COPY_W()
    } else {
        PP_COPY_A(0, AE) PP_COPY_W()
        PP_COPY_A(AE, AC) PP_A_DONE() PP_COPY_W()
    }
    PP_WAIT()
    pp_barrier();
    if (wm == 1) pp_barrier();     // the second group runs one half phase behind the first

    unsigned a_rd = 0, w_rd = 0;   // LDS offsets of the A step and W slot being read
    bf16x8 af[HP][RF], wf[HP][CF];
    // 16-row fragments of this wave that hold rows of the result: the last row tile skips the others (on this chip the matrix
    // cores' power sets the clock, so work on rows that do not exist would slow down the tiles that do)
    int live = (M - m0_wg - wm * (RF * 16) + 15) >> 4;
    live = live < 0 ? 0 : (live < RF ? live : RF);
#define PP_MEM(H, LIVE)                                                                                           \
    {                                                                                                       \
        _Pragma("unroll") for (int k = 0; k < HP; ++k) {                                                    \
            const unsigned char* as_ = lds_raw + (a_off[((H) + k) & 1] + a_rd);                             \
            _Pragma("unroll") for (int j = 0; j < CF; ++j)                                                  \
                wf[k][j] = *reinterpret_cast<const bf16x8*>(lds_raw + (w_off[j & 1] + w_rd) + (j >> 1) * (KB * 1024) + k * 2048); \
            _Pragma("unroll") for (int i = 0; i < RF; ++i) if (i < (LIVE)) af[k][i] = *reinterpret_cast<const bf16x8*>(as_ + i * 2048); \
        }                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
    }
#define PP_COMPUTE(LIVE)                                                                                       \
    {                                                                                                       \
        __builtin_amdgcn_s_setprio(1);                                                                      \
        if constexpr (FP8) {                                                                                \
            _Pragma("unroll") for (int i = 0; i < RF; ++i)                                                  \
                if (i < (LIVE)) _Pragma("unroll") for (int j = 0; j < CF; ++j)                              \
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(pp_pair(wf[0][j], wf[HP - 1][j]), pp_pair(af[0][i], af[HP - 1][i]), acc[i][j], 0, 0, 0, 0, 0, 0); \
        } else {                                                                                            \
            _Pragma("unroll") for (int k = 0; k < HP; ++k)                                                  \
                _Pragma("unroll") for (int i = 0; i < RF; ++i)                                              \
                    if (i < (LIVE)) _Pragma("unroll") for (int j = 0; j < CF; ++j)                          \
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[k][j], af[k][i], acc[i][j], 0, 0, 0); \
        }                                                                                                   \
        __builtin_amdgcn_s_setprio(0);                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
    }
#define PP_PHASE(H, LIVE)                                                                                       \
    {                                                                                                       \
        PP_MEM(H, LIVE)                                                                                      \
        if (HP == 2) { PP_COPY_A(0, AC) PP_A_DONE() }                                                       \
        else if ((H) == 0) { PP_COPY_A(0, AE) }                                                             \
        else { PP_COPY_A(AE, AC) PP_A_DONE() }                                                              \
        PP_COPY_W()                                                                                         \
        w_rd = w_rd == (T::W_SLOTS - 1) * T::W_SLOT ? 0 : w_rd + T::W_SLOT;                                 \
        PP_WAIT()                                                                                           \
        pp_barrier();                                                                                       \
        PP_COMPUTE(LIVE)                                                                                      \
        pp_barrier();                                                                                       \
    }
#define PP_LOOP(LIVE)                                                                                       \
    for (int s = 0; s < n_steps; ++s) {                                                                     \
        PP_PHASE(0, LIVE)                                                                                   \
        if (HP == 1) PP_PHASE(1, LIVE)                                                                      \
        a_rd = a_rd == 2 * T::A_STEP ? 0 : a_rd + T::A_STEP;                                                \
    }
    if (live == RF) { PP_LOOP(RF) } else { PP_LOOP(live) }
#undef PP_LOOP
#undef PP_PHASE
#undef PP_COMPUTE
#undef PP_MEM
#undef PP_WAIT
#undef PP_COPY_W
#undef PP_A_DONE
#undef PP_COPY_A
    if (wm == 0) pp_barrier();
    pp_wait<0>();                  // nothing may still be writing LDS when it is used again or the workgroup ends

    pp_finish<0, RF, RF, CF, KIND, FP8>(acc, lds_raw, wave, T::PART_FLOATS, n_tile * m_tiles + m_tile, split, splits, partial, arrived,
                                        M, N, m0_wg + wm * (RF * 16), n0 + wn * (16 * CF), ep);
}

// Where two groups hold partial sums of the same fragments they exchange halves of them through LDS (see KG_FINISH): rows [I0, I1) of a
// wave's fragments on their way out and in.
template <int I0, int I1, int RF, int CF> __device__ __forceinline__ void kg_put(const f32x4 (&acc)[RF][CF], f32x4* ex) {
#pragma unroll
    for (int i = I0; i < I1; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) ex[(i * CF + j) * 64] = acc[i][j];
}
template <int I0, int I1, int RF, int CF> __device__ __forceinline__ void kg_add(f32x4 (&acc)[RF][CF], const f32x4* ex) {
#pragma unroll
    for (int i = I0; i < I1; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[i][j] += ex[(i * CF + j) * 64];
}
// The end of a tile: rows [0, H) of the fragments are finished by group 0, the rest by group 1.  A macro: through a function that
// holds both groups' branches the accumulators end up in scratch memory.  Where the whole tile's sums do not fit into LDS (224 x 192) the groups
// put their halves there one after the other.
#define KG_FINISH(FP8)                                                                                      \
    {                                                                                                       \
        constexpr int H = (RF + 1) / 2;                                                                     \
        f32x4* ex = reinterpret_cast<f32x4*>(lds_raw) + static_cast<unsigned>(w4) * (T::EX_ROWS * CF * 64) + lane; \
        const int tile = n_tile * m_tiles + m_tile, m0 = m0_wg + wm * (RF * 16), n0w = n0 + wn * (16 * CF); \
        if constexpr (T::EX_ROWS == RF) {                                                                   \
            if (kg == 1) kg_put<0, H>(acc, ex); else kg_put<H, RF>(acc, ex);                                \
            __syncthreads();                                                                                \
            if (kg == 0) kg_add<0, H>(acc, ex); else kg_add<H, RF>(acc, ex);                                \
        } else {                                                                                            \
            if (kg == 1) kg_put<0, H>(acc, ex);                                                             \
            __syncthreads();                                                                                \
            if (kg == 0) kg_add<0, H>(acc, ex);                                                             \
            __syncthreads();                                                                                \
            if (kg == 0) kg_put<H, RF>(acc, ex - H * CF * 64);                                              \
            __syncthreads();                                                                                \
            if (kg == 1) kg_add<H, RF>(acc, ex - H * CF * 64);                                              \
        }                                                                                                   \
        if (splits > 1) __syncthreads();   /* the area is read before the arrival flag is written into it */ \
        if (kg == 0) pp_finish<0, H, RF, CF, KIND, FP8>(acc, lds_raw, w4, T::PART_FLOATS, tile, split, splits, partial, arrived, M, N, m0, n0w, ep); \
        else pp_finish<H, RF, RF, CF, KIND, FP8>(acc, lds_raw, w4, T::PART_FLOATS, tile, split, splits, partial, arrived, M, N, m0, n0w, ep); \
    }

// Narrow tiles: the two wave groups take the two 32-k halves of every K-step of the SAME tile, so that a wave of a 128-column
// tile still owns 64 columns (half the LDS bytes per MFMA of the form above) and a 96-column tile has whole waves; the
// groups' sums meet in LDS at the end.  WM x WN waves per group: 16*RF*WM rows x 16*CF*WN columns.
template <int RF, int CF, int WM> struct KgTile {
    static constexpr int WN = 4 / WM, ROWS = 16 * RF * WM, COLS = 16 * CF * WN, THREADS = 512;
    static constexpr int A_COPIES = ROWS / 8, COPIES = A_COPIES + COLS / 8, CW = (COPIES + 7) / 8;   // 1 KiB copies per K-step, per wave
    static constexpr unsigned STEP = COPIES * 1024u, W_BASE = A_COPIES * 1024u;
    static constexpr int NS = STEP > 40960u ? 3 : 4;                // K-steps in LDS
    static constexpr int EX_ROWS = ROWS * COLS * 4u <= 163840u ? RF : (RF + 1) / 2;   // fragment rows of a wave in the exchange at the end
    static constexpr unsigned ACC_BYTES = 4u * EX_ROWS * CF * 1024u;
    static constexpr unsigned LDS_BYTES = NS * STEP > ACC_BYTES ? NS * STEP : ACC_BYTES;
    static constexpr int64_t PART_FLOATS = static_cast<int64_t>(ROWS) * COLS;
    static_assert(COLS % 32 == 0 && ROWS % 32 == 0 && LDS_BYTES <= 163840u, "whole weight blocks, and what a CU has");
};

template <int RF, int CF, int WM, int KIND>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
gemm_kg_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Wp,
               int M, int N, int K, int m_tiles, int n_tiles, int units_per_xcd, int group_rows,
               int splits, int steps_per_split, float* __restrict__ partial, int* __restrict__ arrived, GemmEpilogue ep) {
    using T = KgTile<RF, CF, WM>;
    constexpr int CW = T::CW, NS = T::NS;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds_raw)));
    int n_tile, m_tile, split;
    if (!pp_unit(m_tiles, n_tiles, units_per_xcd, group_rows, splits, m_tile, n_tile, split)) return;
    const int m0_wg = m_tile * T::ROWS, n0 = n_tile * T::COLS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int kg = wave >> 2, w4 = wave & 3, wm = w4 / T::WN, wn = w4 % T::WN;

    const int ks_begin = split * steps_per_split;
    int n_steps = K / 64 - ks_begin;
    n_steps = n_steps < steps_per_split ? n_steps : steps_per_split;

    // The copies of a K-step (8 rows of A or one 32-column x 16-k weight block, 1 KiB each) are dealt out to the waves in
    // one list; its end is padded with repetitions of the last copy.
    const char* base[CW];
    unsigned voff[CW], stride[CW], dst[CW];
    const int n_blocks = (N + 31) >> 5;
#pragma unroll
    for (int i = 0; i < CW; ++i) {
        int c = wave * CW + i;
        c = c < T::COPIES ? c : T::COPIES - 1;
        dst[i] = lds0 + static_cast<unsigned>(c) * 1024u;
        if (c < T::A_COPIES) {
            const int row = c * 8 + (lane >> 3);
            int r = m0_wg + row;
            r = r < M ? r : M - 1;                                  // rows past M repeat the last row; never stored
            voff[i] = static_cast<unsigned>(r - m0_wg) * static_cast<unsigned>(lda) * 2u + static_cast<unsigned>(((lane & 7) ^ ((row >> 1) & 7)) << 4);
            base[i] = reinterpret_cast<const char*>(A + static_cast<int64_t>(m0_wg) * lda + static_cast<int64_t>(ks_begin) * 64);
            stride[i] = 128u;
        } else {
            const int f = c - T::A_COPIES;                          // block f / 4 of the tile, k-block f % 4 of the step
            int nb = (n0 >> 5) + (f >> 2);
            nb = nb < n_blocks ? nb : n_blocks - 1;                 // blocks past N repeat the last block
            voff[i] = pp_w_source(lane);
            base[i] = reinterpret_cast<const char*>(Wp + (static_cast<int64_t>(nb) * (K >> 4) + static_cast<int64_t>(ks_begin) * 4 + (f & 3)) * 512);
            stride[i] = 4096u;
        }
    }
    const unsigned a_off = static_cast<unsigned>(wm * (RF * 16) + l16) * 128u + static_cast<unsigned>(((4 * kg + kc) ^ ((l16 >> 1) & 7)) << 4);
    // weight fragment q of the tile's columns: fragment q % 2 of block q / 2 (4 KiB per block and step, k half kg in its half)
    unsigned w_off[2];
#pragma unroll
    for (int jl = 0; jl < 2; ++jl) w_off[jl] = T::W_BASE + static_cast<unsigned>(wn * (CF / 2)) * 4096u + kg * 2048u + pp_w_slot(lane, jl);
    static_assert(CF % 2 == 0, "a wave's columns are whole weight blocks");

    f32x4 acc[RF][CF];
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    int next = 0;
    unsigned buf = 0;
#define KG_COPY()                                                                                           \
    {                                                                                                       \
        const unsigned st_ = static_cast<unsigned>(next < n_steps ? next : n_steps - 1);                    \
        _Pragma("unroll") for (int i = 0; i < CW; ++i) pp_copy16(voff[i], base[i] + static_cast<uint64_t>(st_) * stride[i], dst[i] + buf); \
        ++next; buf = buf == (NS - 1) * T::STEP ? 0 : buf + T::STEP;                                        \
    }
#pragma unroll
    for (int p = 0; p < NS - 1; ++p) KG_COPY()
    pp_wait<(NS - 2) * CW>();
    pp_barrier();
    if (kg == 1) pp_barrier();     // the second group runs one half phase behind the first
    unsigned rd = 0;
    bf16x8 af[RF], wf[CF];
    int live = (M - m0_wg - wm * (RF * 16) + 15) >> 4;
    live = live < 0 ? 0 : (live < RF ? live : RF);
#define KG_LOOP(LIVE)                                                                                       \
    for (int s = 0; s < n_steps; ++s) {                                                                     \
        _Pragma("unroll") for (int j = 0; j < CF; ++j) wf[j] = *reinterpret_cast<const bf16x8*>(lds_raw + (w_off[j & 1] + rd) + (j >> 1) * 4096); \
        _Pragma("unroll") for (int i = 0; i < RF; ++i) if (i < (LIVE)) af[i] = *reinterpret_cast<const bf16x8*>(lds_raw + (a_off + rd) + i * 2048); \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        KG_COPY()                                                                                           \
        rd = rd == (NS - 1) * T::STEP ? 0 : rd + T::STEP;                                                   \
        pp_wait<(NS - 2) * CW>();                                                                           \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_barrier();                                                                                       \
        __builtin_amdgcn_s_setprio(1);                                                                      \
        _Pragma("unroll") for (int i = 0; i < RF; ++i)                                                      \
            if (i < (LIVE)) _Pragma("unroll") for (int j = 0; j < CF; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], af[i], acc[i][j], 0, 0, 0); \
        __builtin_amdgcn_s_setprio(0);                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_barrier();                                                                                       \
    }
    if (live == RF) { KG_LOOP(RF) } else { KG_LOOP(live) }
#undef KG_LOOP
#undef KG_COPY
    if (kg == 0) pp_barrier();
    pp_wait<0>();
    __syncthreads();
    KG_FINISH(false)
}

// E4M3 form of the narrow tiles: the instruction takes a whole K-step (128 values) at once, so the groups take turns: group
// g owns the steps g, g + 2, ..., copies them itself and reads them while the other group runs its MFMAs on the step before.
// A wave owns the rows and columns of a bf16 one (128 x 64 at 256 x 128: 96 KiB of fragment reads per step where two groups
// with rows of their own read 160, more than the LDS delivers during the step's MFMAs).
template <int RF, int CF, int WM> struct Kg8Tile {
    static constexpr int WN = 4 / WM, ROWS = 16 * RF * WM, COLS = 16 * CF * WN, THREADS = 512;
    static constexpr int AC = ROWS / 32, WC = COLS / 32;           // 1 KiB copies per wave of the group and step
    static constexpr unsigned STEP = (ROWS + COLS) * 128u, W_BASE = ROWS * 128u;
    static constexpr int LOOK = 5 * STEP <= 163840u ? 2 : 1;        // own steps that the copies run ahead
    static constexpr int NS = 2 * LOOK + 1;                         // steps in LDS
    static constexpr int EX_ROWS = ROWS * COLS * 4u <= 163840u ? RF : (RF + 1) / 2;   // fragment rows of a wave in the exchange at the end
    static constexpr unsigned ACC_BYTES = 4u * EX_ROWS * CF * 1024u;
    static constexpr unsigned LDS_BYTES = NS * STEP > ACC_BYTES ? NS * STEP : ACC_BYTES;
    static constexpr int64_t PART_FLOATS = static_cast<int64_t>(ROWS) * COLS;
    static_assert(COLS % 32 == 0 && ROWS % 32 == 0 && LDS_BYTES <= 163840u, "whole weight blocks, and what a CU has");
};

template <int RF, int CF, int WM, int KIND>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
gemm_kg8_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Wp,
                int M, int N, int K, int m_tiles, int n_tiles, int units_per_xcd, int group_rows,
                int splits, int steps_per_split, float* __restrict__ partial, int* __restrict__ arrived, GemmEpilogue ep) {
    using T = Kg8Tile<RF, CF, WM>;
    constexpr int AC = T::AC, WC = T::WC, LOOK = T::LOOK;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds_raw)));
    int n_tile, m_tile, split;
    if (!pp_unit(m_tiles, n_tiles, units_per_xcd, group_rows, splits, m_tile, n_tile, split)) return;
    const int m0_wg = m_tile * T::ROWS, n0 = n_tile * T::COLS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int kg = wave >> 2, w4 = wave & 3, wm = w4 / T::WN, wn = w4 % T::WN;

    const int ks_begin = split * steps_per_split;
    int n_steps = K / 64 - ks_begin;
    n_steps = n_steps < steps_per_split ? n_steps : steps_per_split;

    // Copy sources of a step: wave w of the group takes A rows [w * 8 * AC, + 8 * AC) and k-block w of every weight block of the tile.
    unsigned a_voff[AC];
#pragma unroll
    for (int i = 0; i < AC; ++i) {
        const int row = (w4 * AC + i) * 8 + (lane >> 3);
        int r = m0_wg + row;
        r = r < M ? r : M - 1;                                      // rows past M repeat the last row; never stored
        a_voff[i] = static_cast<unsigned>(r - m0_wg) * static_cast<unsigned>(lda) * 2u + static_cast<unsigned>(((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const int a_live = (M - m0_wg - w4 * (8 * AC) + 7) >> 3;        // rows past M are not copied
    const char* a_base = reinterpret_cast<const char*>(A + static_cast<int64_t>(m0_wg) * lda + static_cast<int64_t>(ks_begin) * 64);
    const int n_blocks = (N + 31) >> 5;
    const char* w_base = reinterpret_cast<const char*>(Wp + (static_cast<int64_t>(ks_begin) * 4 + w4) * 512);
    const int64_t w_block = static_cast<int64_t>(K >> 4) * 1024;    // bytes of a 32-column block
    const unsigned w_voff = pp_w_source(lane);
    const unsigned a_dst = lds0 + static_cast<unsigned>(w4) * (AC * 1024u), w_dst = lds0 + T::W_BASE + static_cast<unsigned>(w4) * 1024u;

    unsigned a_off[2], w_off[2];                                    // [k half], [fragment parity]
#pragma unroll
    for (int h = 0; h < 2; ++h)
        a_off[h] = static_cast<unsigned>(wm * (RF * 16) + l16) * 128u + static_cast<unsigned>(((4 * h + kc) ^ ((l16 >> 1) & 7)) << 4);
#pragma unroll
    for (int jl = 0; jl < 2; ++jl) w_off[jl] = T::W_BASE + static_cast<unsigned>(wn * (CF / 2)) * 4096u + pp_w_slot(lane, jl);
    static_assert(CF % 2 == 0, "a wave's columns are whole weight blocks");

    f32x4 acc[RF][CF];
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Step s sits in slot s % NS.  A group reads step s, then issues the copies of its step s + NS - 1 into the slot of step s - 1, which
    // the other group has finished reading one barrier ago; what it reads next has landed when LOOK - 1 packets are in flight.
    // Steps past the end repeat the last one (their slots are never multiplied).
    auto copy = [&](int step, unsigned slot) __attribute__((always_inline)) {
        const int st = step < n_steps ? step : n_steps - 1;
        pp_copies_if<0, AC>(a_voff, a_base + static_cast<int64_t>(st) * 128, a_dst + slot, a_live);
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            int nb = (n0 >> 5) + i;
            nb = nb < n_blocks ? nb : n_blocks - 1;                 // blocks past N repeat the last block
            pp_copy16(w_voff, w_base + nb * w_block + static_cast<int64_t>(st) * 4096, w_dst + slot + i * 4096u);
        }
    };
#pragma unroll
    for (int p = 0; p < LOOK; ++p) copy(kg + 2 * p, (kg + 2 * p) * T::STEP);
    if (kg == 1) pp_barrier();     // the second group runs one half phase behind the first
    pp_wait<(LOOK - 1) * (AC + WC)>();
    pp_barrier();
    unsigned rd = kg * T::STEP;
    bf16x8 af[2][RF], wf[2][CF];
    int live = (M - m0_wg - wm * (RF * 16) + 15) >> 4;
    live = live < 0 ? 0 : (live < RF ? live : RF);
#define KG8_LOOP(LIVE)                                                                                      \
    for (int s = kg; s < n_steps + kg; s += 2) {                                                            \
        _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                     \
            _Pragma("unroll") for (int j = 0; j < CF; ++j) wf[h][j] = *reinterpret_cast<const bf16x8*>(lds_raw + (w_off[j & 1] + rd) + (j >> 1) * 4096 + h * 2048); \
            _Pragma("unroll") for (int i = 0; i < RF; ++i) if (i < (LIVE)) af[h][i] = *reinterpret_cast<const bf16x8*>(lds_raw + (a_off[h] + rd) + i * 2048); \
        }                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        copy(s + 2 * LOOK, rd == 0 ? (T::NS - 1) * T::STEP : rd - T::STEP);                                 \
        rd += 2 * T::STEP;                                                                                  \
        rd = rd >= T::NS * T::STEP ? rd - T::NS * T::STEP : rd;                                             \
        pp_wait<LOOK * (AC + WC)>();                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_barrier();                                                                                       \
        if (s < n_steps) {                                                                                  \
            __builtin_amdgcn_s_setprio(1);                                                                  \
            _Pragma("unroll") for (int i = 0; i < RF; ++i)                                                  \
                if (i < (LIVE)) _Pragma("unroll") for (int j = 0; j < CF; ++j)                              \
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(pp_pair(wf[0][j], wf[1][j]), pp_pair(af[0][i], af[1][i]), acc[i][j], 0, 0, 0, 0, 0, 0); \
            __builtin_amdgcn_s_setprio(0);                                                                  \
        }                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_wait<(LOOK - 1) * (AC + WC)>();                                                                  \
        pp_barrier();                                                                                       \
    }
    if (live == RF) { KG8_LOOP(RF) } else { KG8_LOOP(live) }
#undef KG8_LOOP
    if (kg == 0) pp_barrier();
    pp_wait<0>();
    __syncthreads();
    KG_FINISH(true)
}

// E4M3 form of the wide tiles: 256 columns, a wave owns 16*RF rows x 64 columns, the two groups the upper and lower rows.  Only two
// steps fit into LDS at 256 x 256, which is enough because nothing is waited for before a whole phase has passed: a group
// copies its own rows, and the first group, whose phase begins first, all the weights.  The MFMAs of a step take 2048 cycles
// at 256 x 256, and the LDS as long for the step's 192 KiB of fragment reads and 64 KiB of copies.
template <int RF> struct Pp8Tile {
    static constexpr int CF = 4, ROWS = 32 * RF, COLS = 256, THREADS = 512;
    static constexpr int AC = (2 * RF + 3) / 4, WC = 8;             // 1 KiB copies per wave and step: of its group's rows, of the weights
    static constexpr unsigned STEP = (ROWS + COLS) * 128u, W_BASE = ROWS * 128u, LDS_BYTES = 2 * STEP;
    static constexpr int64_t PART_FLOATS = static_cast<int64_t>(ROWS) * COLS;
};

template <int RF, int KIND>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_pp8_kernel(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Wp,
                int M, int N, int K, int m_tiles, int n_tiles, int units_per_xcd, int group_rows,
                int splits, int steps_per_split, float* __restrict__ partial, int* __restrict__ arrived, GemmEpilogue ep) {
    using T = Pp8Tile<RF>;
    constexpr int CF = T::CF, AC = T::AC, WC = T::WC;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void*)(lds_raw)));
    int n_tile, m_tile, split;
    if (!pp_unit(m_tiles, n_tiles, units_per_xcd, group_rows, splits, m_tile, n_tile, split)) return;
    const int m0_wg = m_tile * T::ROWS, n0 = n_tile * T::COLS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;

    const int ks_begin = split * steps_per_split;
    int n_steps = K / 64 - ks_begin;
    n_steps = n_steps < steps_per_split ? n_steps : steps_per_split;

    // Copy sources of a step: wave wn of group wm takes rows [wn * 8 * AC, + 8 * AC) of the group's, and in the first group k-block wn of
    // every weight block of the tile.
    const int m0 = m0_wg + wm * (RF * 16);
    unsigned a_voff[AC];
#pragma unroll
    for (int i = 0; i < AC; ++i) {
        const int row = (wn * AC + i) * 8 + (lane >> 3);
        int r = m0 + row;
        r = r < M ? r : M - 1;                                      // rows past M repeat the last row; never stored
        a_voff[i] = static_cast<unsigned>(r - m0_wg) * static_cast<unsigned>(lda) * 2u + static_cast<unsigned>(((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    int a_live = (M - m0 - wn * (8 * AC) + 7) >> 3;                 // neither rows past M are copied nor rows past the group's
    a_live = a_live < 2 * RF - wn * AC ? a_live : 2 * RF - wn * AC;
    const char* a_base = reinterpret_cast<const char*>(A + static_cast<int64_t>(m0_wg) * lda + static_cast<int64_t>(ks_begin) * 64);
    const int n_blocks = (N + 31) >> 5;
    const char* w_base = reinterpret_cast<const char*>(Wp + (static_cast<int64_t>(ks_begin) * 4 + wn) * 512);
    const int64_t w_block = static_cast<int64_t>(K >> 4) * 1024;    // bytes of a 32-column block
    const unsigned w_voff = pp_w_source(lane);
    const unsigned a_dst = lds0 + static_cast<unsigned>(wm * (RF * 16)) * 128u + static_cast<unsigned>(wn) * (AC * 1024u);
    const unsigned w_dst = lds0 + T::W_BASE + static_cast<unsigned>(wn) * 1024u;
    const int w_live = wm == 0 ? WC : 0;

    unsigned a_off[2], w_off[2];                                    // [k half], [fragment parity]
#pragma unroll
    for (int h = 0; h < 2; ++h)
        a_off[h] = static_cast<unsigned>(wm * (RF * 16) + l16) * 128u + static_cast<unsigned>(((4 * h + kc) ^ ((l16 >> 1) & 7)) << 4);
#pragma unroll
    for (int jl = 0; jl < 2; ++jl) w_off[jl] = T::W_BASE + static_cast<unsigned>(wn * (CF / 2)) * 4096u + pp_w_slot(lane, jl);

    f32x4 acc[RF][CF];
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Step s sits in slot s % 2.  The copies of step s + 1 go into the slot of step s - 1, which both groups have finished reading: a group
    // its own rows one phase ago, the weights are written by the first group after the second group's last barrier.
    auto copy = [&](int step, unsigned slot) __attribute__((always_inline)) {
        const int st = step < n_steps ? step : n_steps - 1;         // steps past the end repeat the last one (their slot is never read)
        pp_copies_if<0, AC>(a_voff, a_base + static_cast<int64_t>(st) * 128, a_dst + slot, a_live);
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            int nb = (n0 >> 5) + i;
            nb = nb < n_blocks ? nb : n_blocks - 1;                 // blocks past N repeat the last block
            pp_copy16_if<0>(w_voff, w_base + nb * w_block + static_cast<int64_t>(st) * 4096, w_dst + slot + i * 4096u, w_live);
        }
    };
    copy(0, 0);
    pp_wait<0>();
    pp_barrier();
    if (wm == 1) pp_barrier();     // the second group runs one half phase behind the first
    unsigned rd = 0;
    bf16x8 af[2][RF], wf[2][CF];
    int live = (M - m0 + 15) >> 4;
    live = live < 0 ? 0 : (live < RF ? live : RF);
#define PP8_LOOP(LIVE)                                                                                      \
    for (int s = 0; s < n_steps; ++s) {                                                                     \
        _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                     \
            _Pragma("unroll") for (int j = 0; j < CF; ++j) wf[h][j] = *reinterpret_cast<const bf16x8*>(lds_raw + (w_off[j & 1] + rd) + (j >> 1) * 4096 + h * 2048); \
            _Pragma("unroll") for (int i = 0; i < RF; ++i) if (i < (LIVE)) af[h][i] = *reinterpret_cast<const bf16x8*>(lds_raw + (a_off[h] + rd) + i * 2048); \
        }                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        rd = T::STEP - rd;                                                                                  \
        copy(s + 1, rd);                                                                                    \
        pp_wait<AC + WC>();                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_barrier();                                                                                       \
        __builtin_amdgcn_s_setprio(1);                                                                      \
        _Pragma("unroll") for (int i = 0; i < RF; ++i)                                                      \
            if (i < (LIVE)) _Pragma("unroll") for (int j = 0; j < CF; ++j)                                  \
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(pp_pair(wf[0][j], wf[1][j]), pp_pair(af[0][i], af[1][i]), acc[i][j], 0, 0, 0, 0, 0, 0); \
        __builtin_amdgcn_s_setprio(0);                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                                  \
        pp_wait<0>();                                                                                       \
        pp_barrier();                                                                                       \
    }
    if (live == RF) { PP8_LOOP(RF) } else { PP8_LOOP(live) }
#undef PP8_LOOP
    if (wm == 0) pp_barrier();
    pp_finish<0, RF, RF, CF, KIND, true>(acc, lds_raw, wave, T::PART_FLOATS, n_tile * m_tiles + m_tile, split, splits, partial, arrived,
                                         M, N, m0, n0 + wn * (16 * CF), ep);
}

}  // namespace
