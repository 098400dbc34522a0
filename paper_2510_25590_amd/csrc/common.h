// Shared declarations of the library's translation units (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <stdarg.h>
#include <stdio.h>
#include "regione.h"
#include "regione_bench.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

constexpr int kMaxSplitTiles = 1024;   // tiles of one K-split GEMM launch

constexpr int kModSets = 16;           // sets of modulation vectors that a step forms at a time, in one launch

constexpr int kGemmPlanSlots = 64;
struct GemmPlanSlot { int m, n, k, kind, tile, splits; size_t part_bytes; };   // a remembered choice of GEMM tile and K splits

struct regione_ctx {
    hipStream_t stream;
    regione_dims dims;
    int device;
    int f32;       // compute dtype of the context is float32: the activation buffers below then hold 4-byte elements
    // workspace (device)
    int32_t* part_counts;  // scratch of the partition: per-block edited counts, then one decision bit per token
    int64_t part_counts_cap;   // its size in int32 entries
    int* part_arrived;             // arrival counter of the partition's workgroups (behind those of the GEMMs); zero between launches
    int32_t* n_edited_pinned;      // pinned host copy of the last edited-token count (host address)
    int32_t* n_edited_pinned_dev;  // the same memory as the device sees it
    int32_t count_ticket;          // last ticket handed to a partition whose count the host polls for (word 1 of the pinned memory)
    // activation buffers: elements of the compute dtype (bf16, or float32 in a float32 context); addressed in bytes
    char* u;       // [max_fresh, H]     normalised + modulated rows
    char* q;       // [max_fresh, H]
    char* kf;      // [max_fresh, H]     fresh keys when the cache is not used
    char* vf;      // [max_fresh, H]
    char* a;       // [max_fresh, H+M]   attention output (+ activated MLP part, single-stream)
    float* h1;     // [max_fresh, H]     residual stream between the two halves of a block
    char* m;       // [max_fresh, M]     activated MLP hidden rows
    float* attn_part;  // split-KV partial results
    size_t attn_part_bytes;
    size_t attn_range_bytes;   // how much of it plan_ranges counts on
    float* mod_ws;     // [2 + kModSets][6H] modulation vectors: of the two streams when a block call forms them itself, then those of a step's blocks
    // workspace of the 8-bit block (allocated by its first call): codes of one projection's input rows and their scales
    uint8_t* q8; size_t q8_bytes; float* q8_scale;
    float* gemm_part;  // split-K partial sums
    size_t gemm_part_bytes;
    int* gemm_arrived;     // [2][kMaxSplitTiles] arrival counters of K-split GEMMs' tiles, one set per lane; zero between launches
    // second lane for independent work inside one call (text and image rows of a double-stream block use different
    // weights, so their projections do not depend on each other): a stream of the default priority and two events,
    // created on first use; while a lane swap is active, `stream` and `gemm_part` name the lane's own stream and half
    hipStream_t side_stream;
    hipEvent_t ev_fork, ev_join;
    GemmPlanSlot gemm_plans[kGemmPlanSlots];
    int gemm_force_tn, gemm_force_splits;  // 0 = chosen per call
    int attn_force_splits, attn_force_form, attn_force_ranges;  // 0 = chosen per call
    // kernels that need more than 64 KiB of LDS have to be granted it once per device: one bit per kernel family and
    // instantiation that this context (one device) has already asked for
    uint32_t lds_grant_mask;
    // optional per-kernel-class timing with HIP events on the context's stream
    int prof_on;
    int prof_used;
    int prof_cap;
    hipEvent_t* prof_ev;   // 2 * prof_cap events: start/stop pairs
    int* prof_class;       // class of each pair
};

// Brackets the launches of one kernel class with an event pair when profiling is on.
struct ProfScope {
    regione_ctx* c; int slot;
    ProfScope(regione_ctx* ctx, int kernel_class) : c(ctx), slot(-1) {
        if (c && c->prof_on && c->prof_used < c->prof_cap) {
            slot = c->prof_used++;
            c->prof_class[slot] = kernel_class;
            (void)hipEventRecord(c->prof_ev[2 * slot], c->stream);
        }
    }
    ~ProfScope() { if (slot >= 0) (void)hipEventRecord(c->prof_ev[2 * slot + 1], c->stream); }
};

void regione_set_error(const char* fmt, ...);
#define RG_FAIL(code, ...) do { regione_set_error(__VA_ARGS__); return (code); } while (0)
#define RG_HIP(call) do { hipError_t e_ = (call); if (e_ != hipSuccess) { \
    regione_set_error("%s failed: %s", #call, hipGetErrorString(e_)); return REGIONE_ERR_HIP; } } while (0)
#define RG_LAUNCH_CHECK() RG_HIP(hipGetLastError())

// More than 64 KiB of LDS, a kernel's own and what its launch asks for together, has to be granted: once per kernel (`granted` is the kernel's) and device.
static inline int rg_grant_lds(const regione_ctx* ctx, const void* kernel, std::atomic<uint64_t>& granted, size_t launch_bytes) {
    const uint64_t bit = uint64_t{1} << (ctx->device & 63);
    if (granted.load(std::memory_order_relaxed) & bit) return REGIONE_OK;
    RG_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(launch_bytes)));
    granted.fetch_or(bit, std::memory_order_relaxed);
    return REGIONE_OK;
}

static inline bool rg_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- device helpers
__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    __bf16 h = static_cast<__bf16>(f);  // round to nearest even (v_cvt_pk_bf16_f32 on gfx950)
    return __builtin_bit_cast(bf16_t, h);
}

// ---- internal launchers (each enqueues on ctx->stream and returns an error code)
enum { EPI_PLAIN = 0, EPI_QKV = 1, EPI_RESID = 2, EPI_VELOCITY = 3 };

struct GemmEpilogue {
    int kind;            // EPI_*
    int vec_ok;          // set by rg_gemm: the wide (8 columns per lane) epilogue may be used
    int keep_sums;       // host only: this product stores K and V (see rg_layernorm_mod)
    const float* bias;   // [N] or null
    int act;             // REGIONE_ACT_* (applied to columns >= act_from)
    int act_from;
    // EPI_PLAIN: y[row*ldy + col] (bf16 or f32)
    void* y; int ldy; int y_f32;
    // EPI_QKV: columns [0,H) -> q[row*ldq+col]; [H,2H) -> k[slot(row)*ldkv + col-H]; [2H,3H) -> v[...];
    //          columns >= 3H -> y[row*ldy + y_col0 + col-3H] (single-stream MLP part)
    bf16_t* q; int ldq; bf16_t* k; bf16_t* v; int ldkv; const int32_t* slot; int slot_offset; int hidden; int y_col0;
    int slot_period, slot_branch_rows;   // slot_period > 0: rows [b * slot_period, + slot_period) are branch b; the slot list repeats, each branch's rows sit slot_branch_rows further
    // EPI_RESID: y[row*ldy+col] = resid[row*ldr+col] + gate[col]*(acc+bias)
    const void* resid; int ldr; int resid_f32; const float* gate;
    // 8-bit GEMM only: the float32 sums are multiplied by row_scale[row] * col_scale[col] before anything else
    const float* row_scale; const float* col_scale;
    // EPI_VELOCITY (the head's product finishes the step: Eq.9 fresh branch, Eq.4, merge):
    //   v = storage-rounded(acc + bias); y (if non-null) = v; vel_ca = v; vel_xe -= vel_dt * v; vel_xfull[vel_index[row]] = vel_xe
    void* vel_ca; void* vel_xe; void* vel_xfull; const int32_t* vel_index; float vel_dt;
};

// Row of the key/value destination of output row `row`: its cache slot when a slot list is given.
__device__ __forceinline__ int32_t epilogue_slot(const GemmEpilogue& ep, int row) {
    if (!ep.slot) return row;
    if (ep.slot_period == 0) return ep.slot[row] + ep.slot_offset;
    const int branch = row / ep.slot_period;
    return ep.slot[row - branch * ep.slot_period] + ep.slot_offset + branch * ep.slot_branch_rows;
}

// a, w_packed (and the epilogue's q, k, v, y, resid where they are activations) are bf16, or float32 in a float32 context
int rg_gemm(regione_ctx* ctx, const void* a, int lda, const void* w_packed, int m, int n, int k, const GemmEpilogue& ep);
// y = x W^T + b with the velocity step (EPI_VELOCITY) as its epilogue (bf16 contexts); merge (optional): rows to write to their places in the same launch,
// *merged tells whether they were
struct RowMerge { const void* src; void* dst; const int32_t* index; int rows, pieces; };   // dst[index[i]] = src[i], rows of `pieces` 16-byte pieces
int rg_gemm_velocity(regione_ctx* ctx, const void* a, int lda, const void* w_packed, int m, int n, int k, const GemmEpilogue& ep, const RowMerge* merge, bool* merged);
// the velocity step and the merges of latent and hidden rows behind a head's product (float32 contexts); v: the product, c_a may be the same tensor
int rg_velocity_merge(regione_ctx* ctx, const void* v, void* c_a, void* x_e, void* x_full, const int32_t* index, float dt, int n, int c, int dtype, const RowMerge& merge);
// rows h_full[index[i]] to h_rows[i], their LayerNorm + modulation to u[i], and latent rows x_t[index[i]] (x_pieces 16-byte pieces) to x_e[i]: one launch where
// gather_layernorm_ok (rows of more than 1024 values, everything 16-byte aligned)
bool rg_gather_layernorm_ok(const void* h_full, const void* h_rows, const void* u, const float* shift, const float* scale, const void* x_t, const void* x_e, int hidden, int64_t x_row_bytes);
// slots (optional): the slot list of regione_fresh_slots, [0, n_txt) and index[i] + n_txt, in the same launch
int rg_gather_layernorm(regione_ctx* ctx, const void* h_full, int h_f32, const int32_t* index, int n, int hidden, const float* shift, const float* scale, void* h_rows, void* u,
                        const void* x_t, void* x_e, int x_pieces, int32_t* slots, int n_txt);
int rg_gather_pair_slots(regione_ctx* ctx, const void* src_a, int32_t row_elems_a, int32_t dtype_a, void* dst_a, const void* src_b, int32_t row_elems_b, int32_t dtype_b, void* dst_b,
                         const int32_t* index, const int32_t* n_dev, int64_t n_max, int32_t* slots, int n_txt);
// modulation vectors of several blocks in one launch: y = silu(x) W^T + b for each entry, W [n, k] row-major bf16; go (optional): nothing is done where *go is zero on the GPU
struct VecBatch { const float* x[kModSets]; const bf16_t* w[kModSets]; const float* b[kModSets]; float* y[kModSets]; int n[kModSets]; int first_wg[kModSets + 1]; int count; };
static inline bool rg_vec_columns_ok(int k) { return k % 8 == 0 && k <= 16384; }      // whole 16-byte pieces, and the vector as float32 within 64 KiB of LDS
int rg_vec_linear_batch(regione_ctx* ctx, VecBatch& batch, int k, const int32_t* go);
// One product: norm: of layernorm_mod(a), rows a of k values (a_f32: float32).
struct GemmCall { const void* a; int lda, norm, a_f32; const float* shift; const float* scale; const void* w; int m, n, k; GemmEpilogue ep; };
// Two products of the same shape but for their rows (the text and the image rows of a block, each with weights of their own) in one launch, with the results of two calls bit for
// bit; rg_gemm_pairs tells where that pays (nothing else may be passed to rg_gemm_pair).
bool rg_gemm_pairs(const regione_ctx* ctx, const GemmCall& a, const GemmCall& b);
bool rg_gemm_pairs_f32(const GemmCall& a, const GemmCall& b);
int rg_gemm_pair(regione_ctx* ctx, const GemmCall& a, const GemmCall& b);
int rg_gemm_pair_f32(regione_ctx* ctx, const GemmCall& a, const GemmCall& b);
// the product of layernorm_mod(h) (h: rows of k values, bf16 or float32); u: workspace [m, k] of the compute dtype
int rg_layernorm_gemm(regione_ctx* ctx, const void* h, int h_f32, const float* shift, const float* scale, void* u, const void* w_packed, int m, int n, int k, const GemmEpilogue& ep);
// the product of layernorm_mod(h) in one launch where that pays; *done tells
int rg_layernorm_gemm_f32(regione_ctx* ctx, const float* h, const float* shift, const float* scale, const float* w, int m, int n, int k, const GemmEpilogue& ep, bool* done);
int rg_gemm_f32(regione_ctx* ctx, const float* a, int lda, const float* w, int m, int n, int k, const GemmEpilogue& ep);
// E4M3 operands (k counts 8-bit elements, a multiple of 128; lda in bytes, a multiple of 16); ep.row_scale / col_scale set
// LayerNorm + modulation with the E4M3 row quantisation of its float32 result: codes [n, hidden], one scale per row
int rg_layernorm_mod_fp8(regione_ctx* ctx, const void* h, int h_f32, int n, int hidden, const float* shift, const float* scale,
                         uint8_t* q, float* row_scale);
int rg_gemm_fp8(regione_ctx* ctx, const uint8_t* a, int lda, const uint8_t* w_packed, int m, int n, int k, const GemmEpilogue& ep);
// u: compute dtype.  keep_sums: a wave per row whatever its length.  Blocks ask for it ahead of the projection whose K and V they store, and that projection takes its tile by kPlanKept:
// so the same input rows give the same stored bits as before there were LayerNorms of several waves.  An E4M3 block that reads such rows turns other last bits (0.04 % of the cache one bf16
// rounding off) into 1.1 % of its output, more than the 1e-2 that two versions' outputs may differ by.  That holds block by block, not for what a stack of blocks hands on: the block's other
// products and its second LayerNorm are as fast as anywhere, and the rows that the next block gets differ in last bits.  Which cache an E4M3 block will read is not known here, so
// every storing bf16 forward pays: 8704 rows of 3072 42 us for 28, of 2.4 ms.
int rg_layernorm_mod(regione_ctx* ctx, const void* h, int h_f32, int n, int hidden, const float* shift, const float* scale, void* u, bool keep_sums = false);
int rg_qk_norm_rope(regione_ctx* ctx, bf16_t* q, int ldq, bf16_t* k, int ldkv, const int32_t* kv_slot,
                    const int32_t* pos_slot, int pos0, int slot_offset, int slot_period, int slot_branch_rows, int n, int heads, int d,
                    const float* q_norm, const float* k_norm, const float* table, int table_rows);
// E4M3 codes of the attention's result rows (heads * d columns) and their scales, formed by the launch that merges key ranges where there is one; keep_out: the rows are wanted, too.
// done tells whether they were formed.
struct RowCodes { uint8_t* codes; float* scale; bool keep_out, done; };
int rg_attention(regione_ctx* ctx, const void* q, int ldq, int n_q,
                 const void* k0, const void* v0, int ldkv0, int n0,
                 const void* k1, const void* v1, int ldkv1, int n1, const int32_t* idx1, int rows1,   // rows1: rows of the array that idx1 picks from
                 int heads, int d, float scale, void* out, int ldo, bool keep_ranges, RowCodes* row_codes = nullptr);       // keep_ranges: for wide E4M3 blocks, see plan_ranges
int rg_attention_f32(regione_ctx* ctx, const float* q, int ldq, int n_q,
                     const float* k0, const float* v0, int ldkv0, int n0,
                     const float* k1, const float* v1, int ldkv1, int n1, const int32_t* idx1,
                     int heads, int d, float scale, float* out, int ldo);
int rg_pack_weight_f32(regione_ctx* ctx, const float* w, int n, int k, float* w_packed);
// regione_partition whose host count arrives through a ticketed pinned word instead of a stream synchronisation
// (rg_partition_queue), which rg_partition_count waits for
int rg_partition_queue(regione_ctx* ctx, const void* x_t, const void* v, const void* x_ref,
                       int64_t n_tokens, int32_t c, int32_t dtype, float sigma_t, float eta,
                       float* score_opt, uint8_t* mask, int32_t* e_index, int32_t* u_index, int32_t* n_edited_dev);
int rg_partition_count(regione_ctx* ctx, int32_t* n_edited_host);
// the static-scratch lookup of regione_partition_static, done ahead of time by regione_create
int rg_partition_static_warm(void);
// int32 entries of scratch memory the partition needs for max_tokens tokens
int64_t rg_partition_scratch_ints(int64_t max_tokens);
