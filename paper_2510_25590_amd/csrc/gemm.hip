// bf16 and E4M3 GEMMs on the CDNA4 matrix cores for the block's dense projections (QKV, attention output, MLP up/down;
// section "Region-Aware Generation": the DiT runs on [X^P, X^E] only): which tile a product gets, and the entry points.
//
//   C[m, n] = sum_k A[m, k] * W[n, k]      A: activations [M, K] row-major, W: weights, PACKED by regione_pack_weight
//
// The packed layout: block (n/32, k/16) is 64 lanes x 16 bytes, lane l holding W[32*(n/32) + l%32][16*(k/16) + 8*(l/32) .. +8].
// The tile kernels (gemm_pp.h) copy such blocks whole into LDS and read the columns of a fragment from there; the kernel
// for few rows and for results of at most 64 columns (gemm_small.h) reads them as they lie.
#include "gemm_epilogue.h"
#include "gemm_small.h"
#include "gemm_tiles.h"

namespace {

constexpr int BK = 64;        // k elements per step
constexpr int kThreads = 256;

// [n, k] row-major -> fragment-major packed layout (rows past n are zero)
__global__ void __launch_bounds__(kThreads)
pack_weight_kernel(const bf16_t* __restrict__ w, int n, int k, bf16_t* __restrict__ wp) {
    const int64_t chunks = static_cast<int64_t>((n + 31) >> 5) * (k >> 4) * 64;   // 16-byte chunks of the packed array
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; c < chunks; c += stride) {
        const int lane = static_cast<int>(c & 63);
        const int64_t blk = c >> 6;
        const int kb = static_cast<int>(blk % (k >> 4));
        const int nb = static_cast<int>(blk / (k >> 4));
        const int row = nb * 32 + (lane & 31), col = kb * 16 + 8 * (lane >> 5);
        uint4 x = make_uint4(0, 0, 0, 0);
        if (row < n) x = *reinterpret_cast<const uint4*>(w + static_cast<int64_t>(row) * k + col);
        *reinterpret_cast<uint4*>(wp + c * 8) = x;
    }
}

// ---- which tile and how many K splits
//
// A plan's time is estimated from what bounds its K-steps on this chip (cycles per step of 64 k and workgroup):
//   matrix cores : ROWS * COLS / 32 (both wave groups' MFMAs, 16 cycles each on four SIMDs) and what the barriers cost;
//   operand feed : 29.6 per KiB copied into LDS (the CU's address path; the L2 delivers what it asks for);
//   latency      : two steps of copies in flight;
// at 2.2 GHz, times a factor of the tile that takes in its start, its epilogue and what the matrix cores' power takes from the clock; not below the time that the
// weights take from HBM.  A K split adds its partial sums' way out and back (padded tiles).
// All constants are fitted to every tile and K split of 267 shapes (32-9400 rows, 1024-21504 columns, k 1024-15360, weights of 3072-wide models uncached).  Against
// the best of all plans the choice loses 0.6 % on average over these and over 143 others, 7 % at most on those (fitted together, so that no constant is a rate by itself: what a round or
// its results cost beside the steps went into the tiles' factors); the constants before, fitted without the two widest tiles of gemm_kg_kernel,
// lost 2.0 % with them.  us, then / now: 2048 x 9216 x 3072 103.3 / 95.8, 1640 x 12288 x 3072 103.5 / 98.9, 1382 x 3072 x 15360 116.7 / 109.9, 205 x 21504 x 3072 43.8 / 41.6.
struct TileShape { int code, rows, cols, lds_kb, form; double factor[2]; };   // form: kTilesFp8 only; factor: kTiles only, of kPlan and of kPlanSmall
constexpr TileShape kTiles[] = {{222, 64, 64, 64, 0, {1.089, 0.865}}, {224, 64, 128, 96, 0, {1.156, 0.725}}, {242, 128, 64, 96, 0, {1.056, 1.022}}, {244, 128, 128, 128, 0, {1.059, 0.932}},
                                {274, 224, 128, 132, 0, {1.054, 1.141}}, {284, 256, 128, 144, 0, {1.381, 1.103}}, {426, 128, 96, 112, 0, {1.058, 0.939}}, {436, 192, 96, 144, 0, {1.114, 1.093}},
                                {446, 256, 96, 132, 0, {0.985, 1.053}}, {44, 128, 256, 144, 0, {1.028, 0.989}}, {64, 192, 256, 136, 0, {1.143, 1.057}}, {74, 224, 256, 148, 0, {1.065, 1.013}},
                                {84, 256, 256, 160, 0, {1.011, 0.971}}, {266, 192, 192, 144, 0, {1.021, 1.015}}, {276, 224, 192, 156, 0, {1.012, 1.269}}};
struct GemmPlan { int tile; int splits; };

// cycles: per KiB copied, barriers and least time of a step by form (narrow, wide), once more for narrow ones; MHz; us per round; TB/s of weights and results; K splits
struct PlanConstants { double feed, over_n, over_w, least_n, least_w, add_n, clock, round, hbm, out, split, split_unit, split_tile, two; int factors; bool wide_half_steps; };   // factors: which of a tile's, -1: none
constexpr PlanConstants kPlan = {29.55, 174.9, 93.0, 546.2, 310.6, 59.5, 23.2, 0.14, 7.18e6, 128.0e6, 1.44, 0.132, 0.0267, 4.13, 0, true};
// Fewer than 1024 columns or less K: the fit above saw none of these.  Fitted to every tile and K split of 750 such products (100-20000 rows, 65-16000 columns, k 64-12800, weights cached),
// 1.0 % behind the best plan on average there and 1.3 % over 180 others, where kPlan is 3.2 % behind (47 % at most) and kPlanKept 3.6 %.
// us, kPlanKept / kPlan / now: 1458 x 512 x 2560 13.2 / 15.5 / 13.2, 10085 x 1792 x 256 20.8 / 24.2 / 20.8, 9358 x 1024 x 256 12.3 / 13.8 / 12.3; the other way 4832 x 960 x 3840 42.7 / 38.9 / 42.7.
constexpr PlanConstants kPlanSmall = {27.49, 310.0, 1.0, 159.5, 267.7, 41.3, 448.9, 0.0, 1e12, 1e12, 0.552, 0.4445, 0.0059, 3.208, 1, true};
// The constants before those, without the factors and the two widest tiles of gemm_kg_kernel, for the projection of a storing forward (see rg_layernorm_mod); the one choice that still takes
// 256 x 128 tiles at 1024 columns and K and more.  us, kPlanKept / kPlan: 2048 x 9216 x 3072 103.3 / 95.8, of 4608 and 8704 rows the same tiles.
constexpr PlanConstants kPlanKept = {28.0, 120.0, 60.0, 450.0, 500.0, 53.0, 455.0, 6.9, 5.5e6, 8.0e6, 1.8, 0.19, 0.0116, 2.35, -1, false};
double plan_time_bf16(const PlanConstants& c, const TileShape& t, int m, int n, int steps, int splits) {
    if (!c.wide_half_steps && (t.code == 266 || t.code == 276)) return 1e30;
    const int m_tiles = (m + t.rows - 1) / t.rows, n_tiles = (n + t.cols - 1) / t.cols;
    const long units = static_cast<long>(m_tiles) * n_tiles * splits;
    const int per = (steps + splits - 1) / splits;
    const bool narrow = t.code >= 200;
    const double mfma = t.rows * t.cols / 32.0, feed = c.feed * (t.rows + t.cols) / 8.0, least = narrow ? c.least_n : c.least_w;
    double step = mfma + (narrow ? c.over_n : c.over_w);
    if (feed > step) step = feed;
    if (step < least) step = least;
    if (narrow) step += c.add_n;
    const double active = units < 256 ? units / 256.0 : 1.0, live = static_cast<double>(m) / (static_cast<double>(m_tiles) * t.rows);
    const double mhz = 2200.0 - c.clock * (mfma / step * active * live);
    const long slots = t.lds_kb <= 80 ? 512 : 256;
    const long full = units / slots, rem = units % slots;
    const double one = per * step / mhz * (c.factors < 0 ? 1.0 : t.factor[c.factors]);
    auto round_time = [&](long u) { return one * (slots > 256 && u > 256 ? c.two : 1.0) + c.round; };
    double us = full * round_time(slots) + (rem > 0 ? round_time(rem) : 0.0);
    const double hbm = static_cast<double>(n) * steps * 128.0 / c.hbm + c.round;     // the weights once from HBM
    if (us < hbm) us = hbm;
    us += static_cast<double>(m) * n * 2.0 / c.out;
    if (splits > 1) {
        const double tile_kb = t.rows * t.cols * 4.0 / 1e3;
        us += c.split + c.split_unit * units * tile_kb / 1e3 + c.split_tile * splits * tile_kb;
    }
    return us;
}

// The E4M3 tiles by kernel: rows of their own for each group, a ring of three or four phases (gemm_pp_kernel); the same with
// a ring of two steps (gemm_pp8_kernel); groups that take turns at the steps (gemm_kg8_kernel).
enum { F8_PP = 0, F8_PP8 = 1, F8_KG8 = 2 };
constexpr TileShape kTilesFp8[] = {{42, 128, 128, 96, F8_PP},    {62, 192, 128, 120, F8_PP},  {82, 256, 128, 144, F8_PP},   {44, 128, 256, 144, F8_PP},
                                   {54, 160, 256, 104, F8_PP8},  {64, 192, 256, 112, F8_PP8}, {74, 224, 256, 120, F8_PP8},  {84, 256, 256, 128, F8_PP8},
                                   {222, 64, 64, 80, F8_KG8},    {224, 64, 128, 120, F8_KG8}, {274, 224, 128, 132, F8_KG8}, {426, 128, 96, 140, F8_KG8},
                                   {446, 256, 96, 132, F8_KG8}};

// The same estimate for E4M3 (a step is 128 values of K).  The MFMAs of a tile's step take as many cycles as in bf16 for twice the work, so
// that the LDS bounds most tiles: 128 bytes a cycle for the fragments that all waves read and for the copies.  The constants are
// fitted to every tile and K split, warm and with cold caches, over 201 shapes (1-19456 rows, 65-21504 columns, k 256-15360): the
// choice is 0.45 % behind the best plan on average and 9 % at most.  With the bf16 constants, and none but tiles of 32 columns
// per wave and 128 x 256, it was 13 % behind the kernel before at 8704 rows.
// us (warm caches; K 3072 unless stated), kernel before / bf16 constants / now: 8704 x 12288 298 / 330 / 287, 8704 x 9216 236 / 269 / 216,
// 8704 x 3072 of K 12288 312 / 316 / 253, 6000 x 12288 204 / 257 / 213, 820 x 12288 46 / 45 / 38, 820 x 3072 of K 12288 54 / 45 / 39,
// 12 x 9216 13 / 16 / 10; over 130 shapes now 1.21 times the kernel before (1.27 with cold caches), 0.95 and 0.89 at the least.
double plan_time_fp8(const TileShape& t, int m, int n, int steps, int splits) {
    const int m_tiles = (m + t.rows - 1) / t.rows, n_tiles = (n + t.cols - 1) / t.cols;
    const long units = static_cast<long>(m_tiles) * n_tiles * splits;
    const int per = (steps + splits - 1) / splits;
    const double barriers[] = {160.0, 55.0, 310.0}, latency[] = {900.0, 1970.0, 0.0}, fixed[] = {3.7, 7.3, 4.4};
    const double mfma = t.rows * t.cols / 32.0;
    const double fragment_rows = (t.form == F8_KG8 ? 4 : 8) * 16.0 * (t.code / 10 % 10 + t.code % 10);
    double step = mfma + barriers[t.form];
    const double lds = 1.066 * (fragment_rows + t.rows + t.cols);
    if (step < lds) step = lds;
    if (step < latency[t.form]) step = latency[t.form];
    const double active = units < 256 ? units / 256.0 : 1.0, live = static_cast<double>(m) / (static_cast<double>(m_tiles) * t.rows);
    const double mhz = 2200.0 - 450.0 * (mfma / step * active * live);
    const double tile_mb = t.rows * t.cols * 4.0 / 1e6;
    const long slots = t.lds_kb <= 80 ? 512 : 256;
    const long full = units / slots, rem = units % slots;
    const double one = per * step / mhz, fix = fixed[t.form] + 22.0 * tile_mb;
    auto round_time = [&](long u) { return one * (slots > 256 && u > 256 ? 2.65 : 1.0) + fix; };
    double us = full * round_time(slots) + (rem > 0 ? round_time(rem) : 0.0);
    const double hbm = static_cast<double>(n) * steps * 128.0 / 5.4e6 + fix;      // the weights once from HBM
    if (us < hbm) us = hbm;
    us += 2.5 + static_cast<double>(m) * n * 2.0 / 14.4e6;
    if (splits > 1) us += 1.2 + 0.26 * units * tile_mb + 9.5 * splits * tile_mb;
    return us;
}

template <size_t N, typename Time>
GemmPlan plan_over(const TileShape (&tiles)[N], Time time, size_t part_bytes, int m, int n, int steps) {
    GemmPlan best = {tiles[0].code, 1};
    double best_t = 1e30;
    for (const TileShape& t : tiles) {
        const long count = static_cast<long>((m + t.rows - 1) / t.rows) * ((n + t.cols - 1) / t.cols);
        for (int s : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16}) {
            if (s > 1) {
                if (count * s > 640 || steps / s < 3) break;
                if (count > kMaxSplitTiles || static_cast<size_t>(count) * s * t.rows * t.cols * sizeof(float) > part_bytes) break;
                const int per = (steps + s - 1) / s;
                if ((steps + per - 1) / per != s) continue;       // another split count in disguise
            }
            const double us = time(t, m, n, steps, s);
            if (us < best_t) { best_t = us; best = {t.code, s}; }
        }
    }
    return best;
}
enum { PLAN_BF16 = 0, PLAN_FP8 = 1, PLAN_KEPT = 2 };
GemmPlan choose_plan(int m, int n, int k, int kind, size_t part_bytes) {
    if (kind == PLAN_FP8) return plan_over(kTilesFp8, plan_time_fp8, part_bytes, m, n, k / BK);
    const PlanConstants& c = kind == PLAN_KEPT ? kPlanKept : n < 1024 || k < 1024 ? kPlanSmall : kPlan;
    return plan_over(kTiles, [&](const TileShape& t, int m_, int n_, int steps, int splits) { return plan_time_bf16(c, t, m_, n_, steps, splits); }, part_bytes, m, n, k / BK);
}

// The plan of a product, remembered per context (a direct-mapped table: a forward repeats a handful of shapes, and trying all
// plans takes the host about as long as a small product takes the GPU).
GemmPlan plan_gemm(regione_ctx* ctx, int m, int n, int k, int kind) {
    if (ctx->gemm_force_tn > 0) {
        const int by_size[7] = {0, 222, 244, 426, 44, 74, 84}, by_size_fp8[7] = {0, 42, 44, 62, 82, 42, 44};
        const int tile = ctx->gemm_force_tn <= 6 ? (kind == PLAN_FP8 ? by_size_fp8 : by_size)[ctx->gemm_force_tn] : ctx->gemm_force_tn;
        return {tile, ctx->gemm_force_splits > 0 ? ctx->gemm_force_splits : 1};
    }
    if (ctx->gemm_force_splits > 0) return {choose_plan(m, n, k, kind, ctx->gemm_part_bytes).tile, ctx->gemm_force_splits};
    const uint32_t h = (static_cast<uint32_t>(m) * 2654435761u) ^ (static_cast<uint32_t>(n) * 2246822519u) ^ (static_cast<uint32_t>(k) * 3266489917u);
    GemmPlanSlot& slot = ctx->gemm_plans[(h >> 16) % kGemmPlanSlots];
    if (slot.m == m && slot.n == n && slot.k == k && slot.kind == kind && slot.part_bytes == ctx->gemm_part_bytes) return {slot.tile, slot.splits};
    const GemmPlan p = choose_plan(m, n, k, kind, ctx->gemm_part_bytes);
    slot = {m, n, k, kind, p.tile, p.splits, ctx->gemm_part_bytes};
    return p;
}

// Which products the kernel of 16-row tiles takes (gemm_small.h), and in tiles of how many columns; 0: the tile kernels.  Its workgroups hold a CU each, and
// every row tile reads all weights from L2 again: it wins where one round of 256 workgroups does.  Times in us, tile kernels -> 32 / 64 columns, where
// a call by itself takes 4.4: rows x columns x K 544 x 256 x 1024 6.9 -> 5.7 / 4.4, 64 x 3072 x 1024 6.9 -> 5.8 / 4.7, 100 x 3072 x 1024 7.0 -> 7.8 / 7.0 (336
// workgroups), 820 x 768 x 256 4.6 -> 7.2 / 5.3.  Long K costs it chains of loads, most of all on weights that no cache holds: the tile kernels' time over this
// kernel's, mean of 580 products of up to 2400 rows, cached / uncached weights: 32 columns, K 2048 1.46 / 1.43, 3072 1.38 / 1.21, 4096 1.31 / 1.08, 5120 1.17 / 0.95; 64
// columns, K 1280 1.26 / 1.21, 1792 1.24 / 1.09, 2304 1.16 / 0.99, 3072 1.09 / 0.92; the last lengths are those of narrow models, whose weights the caches hold.
// Narrow results (at most 64 columns: the velocity head) all go there: 820 x 64 x 3072 13.3 -> 6.4 / 8.0 against a kernel of 32 x 32 tiles, 2560 rows 14.4 -> 11.7
// / 8.1, 8704 rows 44 -> 28 / 23.
// With K <= 256 a second round pays.  After a LayerNorm (k <= 1024), whose launch goes away too, one round is the limit all the same, since every workgroup normalises
// its rows again: us per block with up to two rounds -> one, tile kernels and LayerNorm before: width 256, 400 rows 37.0 -> 33.7 (41.4), single-stream 150 rows 22.0 -> 20.4 (26.3);
// width 768, single-stream 50 rows 33.2 -> 30.0 (32.4); width 1024, 100 rows 52.5 -> 48.0 (54.0), single-stream 34 rows 34.9 -> 32.7 (33.4).
constexpr int kNarrowColumns = 64;
int small_columns(int m, int n, int k, bool after_ln) {
    const int64_t row_tiles = (m + 15) / 16, wgs32 = row_tiles * ((n + 31) / 32), wgs64 = row_tiles * ((n + 63) / 64);
    if (row_tiles > 65535) return 0;
    if (n <= kNarrowColumns) return wgs32 <= 256 ? 32 : 64;
    if (k > 5120) return 0;
    if (wgs32 <= 256) return 32;
    const int64_t most = k <= 256 && !after_ln ? 512 : 256;
    return k <= 3072 && wgs64 <= most ? 64 : 0;
}
// ... unless a comparison forces a plan of the tile kernels
int small_columns(const regione_ctx* ctx, int m, int n, int k, bool after_ln = false) {
    return ctx->gemm_force_tn == 0 && ctx->gemm_force_splits == 0 ? small_columns(m, n, k, after_ln) : 0;
}

// the wide epilogue needs every eight-column group whole (n % 8, checked by the caller) and every touched row 16-byte aligned
bool wide_epilogue_ok(const GemmEpilogue& ep, int n) {
    if (ep.kind == EPI_PLAIN) return (ep.ldy % 8 == 0) && rg_aligned16(ep.y) && (ep.act_from % 8 == 0);
    if (ep.kind == EPI_QKV) return (ep.hidden % 8 == 0) && (ep.ldq % 8 == 0) && (ep.ldkv % 8 == 0) && rg_aligned16(ep.q) && rg_aligned16(ep.k) && rg_aligned16(ep.v) &&
                                   (n <= 3 * ep.hidden || ((ep.ldy % 8 == 0) && (ep.y_col0 % 8 == 0) && rg_aligned16(ep.y)));
    if (ep.kind == EPI_RESID) return (ep.ldy % 8 == 0) && (ep.ldr % 8 == 0) && rg_aligned16(ep.y) && rg_aligned16(ep.resid);
    if (ep.kind == EPI_VELOCITY) return (ep.ldy % 8 == 0) && rg_aligned16(ep.y) && rg_aligned16(ep.vel_ca) && rg_aligned16(ep.vel_xe) && rg_aligned16(ep.vel_xfull);
    return false;
}

}  // namespace

static int gemm_tile(regione_ctx* ctx, const GemmPlan& p, const bf16_t* a, int lda, const bf16_t* wp, int m, int n, int k, const GemmEpilogue& ep) {
    if (p.tile == 266 || p.tile == 276) return rg_gemm_tile_kg(ctx, p.tile, a, lda, wp, m, n, k, p.splits, ep);
    if (p.tile >= 400) return rg_gemm_tile_96(ctx, p.tile, a, lda, wp, m, n, k, p.splits, ep);
    if (p.tile >= 200) return rg_gemm_tile_128(ctx, p.tile, a, lda, wp, m, n, k, p.splits, ep);
    return rg_gemm_tile_wide(ctx, p.tile, a, lda, wp, m, n, k, p.splits, ep);
}

int rg_gemm_fp8(regione_ctx* ctx, const uint8_t* a, int lda, const uint8_t* wp, int m, int n, int k, const GemmEpilogue& ep_in) {
    if (m <= 0 || n <= 0) return REGIONE_OK;
    if (k <= 0 || (k % (2 * BK)) || (lda & 15)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm_fp8: k=%d must be a positive multiple of 128 and lda=%d of 16", k, lda);
    if (!rg_aligned16(a) || !rg_aligned16(wp)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_fp8: operands must be 16-byte aligned");
    if (!ep_in.row_scale || !ep_in.col_scale) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_fp8: both scales are needed");
    if (ep_in.kind != EPI_PLAIN && ep_in.kind != EPI_QKV && ep_in.kind != EPI_RESID) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_fp8: epilogue kind %d", ep_in.kind);
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    GemmEpilogue ep = ep_in;
    ep.vec_ok = (n % 8 == 0) && rg_aligned16(ep.col_scale) && wide_epilogue_ok(ep, n);
    // the kernels count pairs of E4M3 values: the same bytes as half as many 16-bit elements
    const GemmPlan p = plan_gemm(ctx, m, n, k / 2, PLAN_FP8);
    return rg_gemm_tile_fp8(ctx, p.tile, reinterpret_cast<const bf16_t*>(a), lda / 2, reinterpret_cast<const bf16_t*>(wp), m, n, k / 2, p.splits, ep);
}

int rg_gemm_velocity(regione_ctx* ctx, const void* a_any, int lda, const void* wp_any, int m, int n, int k, const GemmEpilogue& ep_in, const RowMerge* merge, bool* merged) {
    if (merged) *merged = false;
    if (m <= 0 || n <= 0) return REGIONE_OK;
    if (ctx->f32) RG_FAIL(REGIONE_ERR_UNSUPPORTED, "gemm: the fused velocity step is a bf16-context path");
    if (k <= 0 || (k % BK) || (lda & 7)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm: k=%d must be a positive multiple of 64 and lda=%d of 8", k, lda);
    if (!rg_aligned16(a_any) || !rg_aligned16(wp_any)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: operands must be 16-byte aligned");
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    GemmEpilogue ep = ep_in;
    ep.kind = EPI_VELOCITY;
    ep.vec_ok = (n % 8 == 0) && wide_epilogue_ok(ep, n);
    const bf16_t* a = static_cast<const bf16_t*>(a_any);
    const bf16_t* wp = static_cast<const bf16_t*>(wp_any);
    if (const int columns = small_columns(ctx, m, n, k)) {
        const int row_tiles = (m + kSmallRows - 1) / kSmallRows;
        if (!merge || row_tiles + 2048 > 65535 || static_cast<int64_t>(merge->rows) * merge->pieces > INT32_MAX) return gemm_small(ctx, a, lda, wp, m, n, k, columns, ep);
        *merged = true;
        return columns == 32 ? launch_small_merge<2>(ctx, a, lda, wp, m, n, k, ep, *merge) : launch_small_merge<4>(ctx, a, lda, wp, m, n, k, ep, *merge);
    }
    // The plan of the product alone: the sums are then those of rg_gemm bit for bit.  Tile 222 with one K split for all such heads took
    // (us, kernel before the two-group ones / 222 / now; hidden 3072): 820 x 128 14.1 / 19.3 / 10.6, 36 x 256 11.4 / 16.7 / 9.0, 8704 x 1024 122 / 139 / 60.
    // Odd widths (see the epilogue): 8704 x 65 22 / 28 / 27, 8704 x 100 23.5 / - / 27, 4096 x 65 16.5 / - / 17.3, 2048 x 66 15.4 / - / 12.4.
    return gemm_tile(ctx, plan_gemm(ctx, m, n, k, PLAN_BF16), a, lda, wp, m, n, k, ep);
}

int rg_gemm(regione_ctx* ctx, const void* a_any, int lda, const void* wp_any, int m, int n, int k, const GemmEpilogue& ep_in) {
    if (m <= 0 || n <= 0) return REGIONE_OK;
    if (ctx->f32) return rg_gemm_f32(ctx, static_cast<const float*>(a_any), lda, static_cast<const float*>(wp_any), m, n, k, ep_in);
    const bf16_t* a = static_cast<const bf16_t*>(a_any);
    const bf16_t* wp = static_cast<const bf16_t*>(wp_any);
    if (k <= 0 || (k % BK) || (lda & 7)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm: k=%d must be a positive multiple of 64 and lda=%d of 8", k, lda);
    if (!rg_aligned16(a) || !rg_aligned16(wp)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: operands must be 16-byte aligned");
    if (ep_in.kind != EPI_PLAIN && ep_in.kind != EPI_QKV && ep_in.kind != EPI_RESID) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm: bad epilogue kind %d", ep_in.kind);
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    GemmEpilogue ep = ep_in;
    ep.vec_ok = (n % 8 == 0) && wide_epilogue_ok(ep, n);
    if (const int columns = small_columns(ctx, m, n, k)) return gemm_small(ctx, a, lda, wp, m, n, k, columns, ep);
    return gemm_tile(ctx, plan_gemm(ctx, m, n, k, ep.keep_sums ? PLAN_KEPT : PLAN_BF16), a, lda, wp, m, n, k, ep);
}

int rg_layernorm_gemm(regione_ctx* ctx, const void* h, int h_f32, const float* shift, const float* scale, void* u, const void* wp, int m, int n, int k, const GemmEpilogue& ep_in) {
    if (m <= 0 || n <= 0) return REGIONE_OK;
    if (ctx->f32 && h_f32) {
        bool done = false;
        if (int rc = rg_layernorm_gemm_f32(ctx, static_cast<const float*>(h), shift, scale, static_cast<const float*>(wp), m, n, k, ep_in, &done)) return rc;
        if (done) return REGIONE_OK;
    }
    const int columns = !ctx->f32 && k <= 1024 && (k % BK) == 0 && rg_aligned16(h) && rg_aligned16(wp) && rg_aligned16(shift) && rg_aligned16(scale) ? small_columns(ctx, m, n, k, true) : 0;
    if (columns && (ep_in.kind == EPI_PLAIN || ep_in.kind == EPI_QKV)) {
        ProfScope prof(ctx, REGIONE_PROF_GEMM);
        GemmEpilogue ep = ep_in;
        ep.vec_ok = (n % 8 == 0) && wide_epilogue_ok(ep, n);
        return gemm_small_ln(ctx, h, h_f32, shift, scale, static_cast<const bf16_t*>(wp), m, n, k, columns, ep);
    }
    if (int rc = rg_layernorm_mod(ctx, h, h_f32, m, k, shift, scale, u, ep_in.keep_sums != 0)) return rc;
    return rg_gemm(ctx, u, k, wp, m, n, k, ep_in);
}

// the columns of a workgroup for the row tiles of both products; 0: not a pair of small ones
static int pair_columns(const regione_ctx* ctx, const GemmCall& a, const GemmCall& b) {
    return small_columns(ctx, 16 * ((a.m + 15) / 16 + (b.m + 15) / 16), a.n, a.k, a.norm != 0);
}

bool rg_gemm_pairs(const regione_ctx* ctx, const GemmCall& a, const GemmCall& b) {
    if (a.m <= 0 || b.m <= 0 || a.n != b.n || a.k != b.k || a.norm != b.norm || a.a_f32 != b.a_f32 || a.ep.kind != b.ep.kind || a.n <= kNarrowColumns) return false;
    if (a.ep.kind != EPI_PLAIN && a.ep.kind != EPI_QKV && (a.ep.kind != EPI_RESID || a.norm)) return false;
    // what either product would be refused for is left to its own call
    const int unit = ctx->f32 ? 3 : 7;
    for (const GemmCall* c : {&a, &b})
        if ((c->lda & unit) || !rg_aligned16(c->a) || !rg_aligned16(c->w) || !rg_aligned16(c->shift) || !rg_aligned16(c->scale)) return false;
    if (ctx->f32) return rg_gemm_pairs_f32(a, b);
    // The rule of one product (small_columns) for the row tiles of both: each alone is then one of the small ones, too, and its sums are taken in the same order.
    return a.k > 0 && a.k % BK == 0 && (!a.norm || a.k <= kLnColumns) && pair_columns(ctx, a, b) != 0;
}

int rg_gemm_pair(regione_ctx* ctx, const GemmCall& a, const GemmCall& b) {
    ProfScope prof(ctx, REGIONE_PROF_GEMM);
    if (ctx->f32) return rg_gemm_pair_f32(ctx, a, b);
    GemmEpilogue ep_a = a.ep, ep_b = b.ep;
    ep_a.vec_ok = (a.n % 8 == 0) && wide_epilogue_ok(ep_a, a.n);
    ep_b.vec_ok = (b.n % 8 == 0) && wide_epilogue_ok(ep_b, b.n);
    return pair_columns(ctx, a, b) == 32 ? launch_small_pair_kind<2>(ctx, a, b, ep_a, ep_b) : launch_small_pair_kind<4>(ctx, a, b, ep_a, ep_b);
}

extern "C" int64_t regione_packed_weight_elems(int32_t n, int32_t k) {
    if (n <= 0 || k <= 0) return 0;
    return static_cast<int64_t>((n + 31) / 32) * 32 * k;
}

extern "C" int regione_pack_weight(regione_ctx* ctx, const void* w, int32_t n, int32_t k, void* w_packed) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "pack_weight: null context");
    if (n <= 0 || k <= 0 || (k % BK)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "pack_weight: n=%d, k=%d (k must be a multiple of 64)", n, k);
    if (!w || !w_packed || !rg_aligned16(w) || !rg_aligned16(w_packed)) RG_FAIL(REGIONE_ERR_INVALID_ARG, "pack_weight: null or unaligned tensor");
    if (w == w_packed) RG_FAIL(REGIONE_ERR_INVALID_ARG, "pack_weight: cannot pack in place");
    if (ctx->f32) return rg_pack_weight_f32(ctx, static_cast<const float*>(w), n, k, static_cast<float*>(w_packed));
    const int64_t chunks = regione_packed_weight_elems(n, k) / 8;
    int64_t blocks = (chunks + kThreads - 1) / kThreads;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(pack_weight_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, ctx->stream,
                       static_cast<const bf16_t*>(w), n, k, static_cast<bf16_t*>(w_packed));
    RG_LAUNCH_CHECK();
    return REGIONE_OK;
}

extern "C" int regione_tune_gemm(regione_ctx* ctx, int32_t wave_tile_blocks, int32_t k_splits) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_gemm: null context");
    bool known = wave_tile_blocks >= 0 && wave_tile_blocks <= 6;
    for (const TileShape& t : kTiles) known = known || t.code == wave_tile_blocks;
    for (const TileShape& t : kTilesFp8) known = known || t.code == wave_tile_blocks;
    if (!known || k_splits < 0 || k_splits > 16) RG_FAIL(REGIONE_ERR_INVALID_ARG, "tune_gemm: tile %d is none of 0..6 and no tile code, or k_splits=%d is not in 0..16", wave_tile_blocks, k_splits);
    ctx->gemm_force_tn = wave_tile_blocks;
    ctx->gemm_force_splits = k_splits;
    return REGIONE_OK;
}

extern "C" int regione_gemm_plan_host(int32_t m, int32_t n, int32_t k, int32_t kind, int64_t workspace_bytes, int32_t* tile, int32_t* k_splits) {
    if (!tile || !k_splits) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_plan: null argument");
    if (m <= 0 || n <= 0 || k <= 0 || workspace_bytes < 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_plan: m=%d n=%d k=%d", m, n, k);
    if (kind != REGIONE_GEMM_BF16 && kind != REGIONE_GEMM_E4M3 && kind != REGIONE_GEMM_BF16_STORED) RG_FAIL(REGIONE_ERR_INVALID_ARG, "gemm_plan: kind %d", kind);
    const bool fp8 = kind == REGIONE_GEMM_E4M3;
    if (k % (fp8 ? 2 * BK : BK)) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "gemm_plan: k=%d must be a multiple of %d", k, fp8 ? 2 * BK : BK);
    GemmPlan p = {0, 1};
    const int plan = fp8 ? PLAN_FP8 : kind == REGIONE_GEMM_BF16_STORED ? PLAN_KEPT : PLAN_BF16;
    if (fp8 || !small_columns(m, n, k, false)) p = choose_plan(m, n, fp8 ? k / 2 : k, plan, static_cast<size_t>(workspace_bytes));
    *tile = p.tile;
    *k_splits = p.splits;
    return REGIONE_OK;
}

extern "C" int regione_linear(regione_ctx* ctx, const void* x, const void* w_packed, const float* b_opt,
                              int32_t m, int32_t n, int32_t k, int32_t act, int32_t out_dtype, void* y) {
    if (!ctx) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear: null context");
    if (m < 0 || n <= 0 || k <= 0) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear: m=%d n=%d k=%d", m, n, k);
    if (act != REGIONE_ACT_NONE && act != REGIONE_ACT_GELU_TANH) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear: bad act %d", act);
    if (out_dtype != REGIONE_BF16 && out_dtype != REGIONE_FP32) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear: bad out_dtype %d", out_dtype);
    if (k % BK) RG_FAIL(REGIONE_ERR_BAD_SHAPE, "linear: k=%d must be a multiple of 64", k);
    if (m == 0) return REGIONE_OK;
    if (!x || !w_packed || !y) RG_FAIL(REGIONE_ERR_INVALID_ARG, "linear: null tensor");
    GemmEpilogue ep = {};
    ep.kind = EPI_PLAIN; ep.bias = b_opt; ep.act = act; ep.act_from = 0;
    ep.y = y; ep.ldy = n; ep.y_f32 = out_dtype == REGIONE_FP32;
    return rg_gemm(ctx, x, k, w_packed, m, n, k, ep);
}
