// C-ABI entry points: host-side argument checks, workspace layout, launch sequences.
#include "internal.hpp"
#include <string.h>
#include <mutex>

namespace ab {

ab_trace_fn g_trace_fn = nullptr;
void *g_trace_user = nullptr;

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int round_up(int x, int a) { return (x + a - 1) / a * a; }

static int pick_tile(int64_t M, int N)
{
    for (int tile = TILE_BIG; tile > TILE_SMALL; --tile) {
        const int edge = tile_edge(tile);
        if (N % edge != 0) continue;
        if (((M + edge - 1) / edge) * (N / edge) >= 512) return tile;
    }
    return TILE_SMALL;
}

// Products of at most so many 32 x 32 tiles go to gemm_slim.hip: two rounds of its work-groups on 256 CUs (an LDS ring of
// 128 KB leaves one a CU).  Whole calls, 64 x 64 tiles against slim ones, four layers of 1024 in bf16: 256 rows (256 tiles)
// 52.4 -> 28.2 us, 512 rows (512) 53.4 -> 40.6, 960 rows (960) 50.6 -> 63.7; three layers of 256 in fp32: 1920 rows (480)
// 33.4 -> 26.0, 3840 rows (960) 30.7 -> 37.9.
static const int64_t kSlimTiles = 512;
static bool slim(int64_t M, int N) { return (M + 31) / 32 * (N / 32) <= kSlimTiles; }

// fp32 products of at least so many 128 x 128 (or 128 x 64) tiles go to gemm_split.hip, smaller ones (and all 32 x 32 tiles
// above) to the fp32 instruction, whose smaller tiles fill the chip.  Whole calls, 32 layers of statistics, fp32 -> split:
// 256-256 with 9000 rows (142 tiles) 31.2 -> 30.4 us, 16000 (248) 36.7 -> 32.0, 60000 88 -> 56, 4.2 M 4625 -> 2690;
// 128-128 with 16000 rows (124 tiles) 22.7 -> 23.5, 30000 (234) 27.0 -> 24.1; 64-64 with 16000 (124) 17.8 -> 18.6, 30000
// (234) 19.3 -> 19.1, 60000 21.8 -> 20.6; 256-128-64 with 16000 34.8 -> 39.4, 30000 47.2 -> 42.7.
static const int64_t kSplitTiles = 192;

// bf16 products of at least so many 256 x 256 tiles go to gemm_big.hip and gemm_span.hip, smaller ones to the generic tiles, which fill
// more CUs but have one slab requested ahead.  Up to 1024 columns a product of less than a round goes in parts of its tiles, so
// the line lies low; where a pass has this product alone, lowest.  Whole calls, 50 layers of statistics, generic / 256 x 256, us, by tiles:
//   one product: 1024-1024 16 tiles 28.6 / 22.1, 56 32.9 / 23.1; 768-768 12 24.7 / 19.1 (with 255 candidates 24.5 / 20.7); 1024-256 12 28.2 / 21.9
//     (28.0 / 23.7); 256-256 24 15.4 / 14.6 (15.5 / 15.4), 48 16.5 / 14.7 (16.6 / 15.6); 128-1024 32 13.5 / 13.2 (13.6 / 14.0), 56 14.8 / 13.7; 128-256 42 (13.7 / 14.0), 55 (14.7 / 14.0)
//   several: 512-512-512 32 26.0 / 26.2 (26.1 / 27.4), 40 29.7 / 26.4; 768-768-768 30 32.4 / 31.4 (32.3 / 33.2), 36 37.3 / 31.5; 1024 four
//     times 32 49.7 / 58.0, 40 57.5 / 58.0 (57.5 / 59.5), 48 60.4 / 58.1; 256-256-256 32 21.0 / 22.4, 48 23.2 / 22.8 (23.3 / 23.4)
// Not the generating kernel for inputs that the streaming one does not take (K = 64 or above 1024): it has no parts, a work-group takes a
// whole tile and generates before it multiplies.  One product: 2048-256 12 tiles 47.7 / 62.4, 60 58.8 / 66.6, 64 67.1 / 66.7; 1280-512 12 33.7 /
// 43.7, 60 40.0 / 44.0; 2048-1024 12 51.6 / 63.1; 4096-256 30 85.7 / 117.7; 64-256 40 12.7 / 14.0, 60 13.2 / 14.0, 64 14.3 / 14.0; several:
// 1280-512-256 44 43.0 / 55.1, 2048-1024-1024 44 63.4 / 81.1.
// Nor low for a product behind one on generic tiles: that one takes longer then, outside the time of its wavefronts (256-640-256, 40
// scenarios, 17.7 -> 20.6 us with the same wave cycles, L2 misses and bytes written; the cause is not known).  256-512-512 (the first product on
// generic tiles) 36 tiles 24.7 / 26.4, 62 28.0 / 30.3; 256-640-256 36 32.0 / 37.8; 256-1024-1024 44 30.2 / 32.9; with the first product on large
// ones 256-768-256 36 35.1 / 29.4, 256-1024-512 44 36.6 / 30.8.  Where generic tiles of more than 64 columns come behind a product of more than 512, the line lies
// higher: 512-768-192 36 28.4 / 30.3, 60 31.4 / 32.6; 576-1024-256 36 30.4 / 33.0; 768-768-192 36 32.6 / 32.3, 52 36.5 / 35.0; 768-1024-1024-192 the second
// 44 50.9 / 53.2, 52 57.5 / 53.7; 768-1280-1024-192 52 62.7 / 64.6; but 512-512-192 36 27.0 / 27.1, 52 30.9 / 28.7, 1024-512-192 44 37.7 / 32.4.
static const int64_t kBigTiles = 64;

static ab_status check_desc(const ab_model_desc *d)
{
    if (!d) return AB_ERR_NULL;
    if (d->compute_dtype != AB_F32 && d->compute_dtype != AB_BF16) return AB_ERR_DTYPE;
    if (d->n_layers <= 0 || d->n_stats <= 0 || d->n_stats > AB_MAX_STATS) return AB_ERR_SHAPE;
    if (d->n_scalars < 0 || d->n_scalars > AB_MAX_SCALARS) return AB_ERR_SHAPE;
    if (d->n_hidden < 0 || d->n_hidden > AB_MAX_HIDDEN) return AB_ERR_SHAPE;
    if (d->n_hidden == 0 && d->tensor_encoder) return AB_ERR_UNSUPPORTED;   // the linear scorer takes flat statistics only
    for (int k = 0; k < d->n_hidden; ++k) {
        if (d->hidden[k] <= 0) return AB_ERR_SHAPE;
        if (d->hidden[k] % 64 != 0 || d->hidden[k] > 4096) return AB_ERR_UNSUPPORTED;
    }
    for (int k = 0; k < d->n_stats; ++k)
        if (d->enc_stat[k].kind != AB_ENC_LINEAR && d->enc_stat[k].kind != AB_ENC_LOG) return AB_ERR_SHAPE;
    for (int k = 0; k < d->n_scalars; ++k)
        if (d->enc_scalar[k].kind != AB_ENC_LINEAR && d->enc_scalar[k].kind != AB_ENC_LOG) return AB_ERR_SHAPE;
    if (d->n_outputs < 0 || d->n_outputs > AB_MAX_OUTPUTS) return AB_ERR_SHAPE;
    if (d->loss_kind != AB_LOSS_MSE && d->loss_kind != AB_LOSS_L2NORM) return AB_ERR_SHAPE;
    if (d->tensor_encoder < 0 || d->tensor_encoder > 2) return AB_ERR_SHAPE;
    if (d->tensor_encoder) {
        if (d->enc_hidden[0] <= 0 || d->enc_hidden[1] <= 0) return AB_ERR_SHAPE;
        if (d->n_stats > AB_MAX_ENCODER_STATS) return AB_ERR_UNSUPPORTED;
        if (d->tensor_encoder == 1 && (d->enc_hidden[0] != 128 || d->enc_hidden[1] != 128)) return AB_ERR_UNSUPPORTED;
        if (d->tensor_encoder == 2 && (d->enc_hidden[0] != 32 || d->enc_hidden[1] != 64)) return AB_ERR_UNSUPPORTED;
        if (d->compute_dtype != AB_BF16) return AB_ERR_UNSUPPORTED;
    } else if ((int64_t)d->n_layers * d->n_stats > (1 << 20)) {
        return AB_ERR_UNSUPPORTED;
    }
    return AB_OK;
}

enum { BIG_TILE = 1, BIG_SPAN = 2 };    // gemm_big.hip; gemm_span.hip (row tiles that span scenarios)

struct ScorePlan {
    int dtype, Fs, F, Kp, D, base;
    int H[AB_MAX_HIDDEN];
    int tile[AB_MAX_HIDDEN];      // tile of hidden GEMM k (k >= 1)
    int split[AB_MAX_HIDDEN];     // hidden GEMM k runs on gemm_split.hip with so many column groups, or 0
    int big[AB_MAX_HIDDEN];       // hidden GEMM k runs on a 256x256 bf16 kernel: BIG_TILE, BIG_SPAN, or 0
    int tile_a;                   // tile of the scenario-term GEMM
    int nt_last;
    int64_t chunk_scen, chunk_rows;
    size_t off_xs, off_w1s, off_aterm, off_bterm, off_cfgv, off_wout, off_xrow, off_partial, off_act0, off_act1, total;
    // second pass for the chosen candidate's prediction vector: one row per scenario, kVChunk scenarios at a time
    int64_t v_chunk;
    int v_tile[AB_MAX_HIDDEN];
    size_t off_vx, off_vact0, off_vact1, off_vlast;
};

static const int64_t kTargetChunkRows = 1 << 20;
static const int64_t kVChunk = 4096;

static int64_t big_tiles(const ScorePlan &p, int k) { return (p.chunk_rows + 255) / 256 * (p.H[k] / 256); }

// The 256 x 256 kernel of hidden product k, or 0; `after`: product k - 1 goes to one.
static int big_kernel(const ScorePlan &p, int32_t C, int k, bool after)
{
    const int K = p.H[k - 1], N = p.H[k];
    if (p.dtype != AB_BF16 || N % 256 != 0) return 0;
    int64_t least = kBigTiles;
    if (N <= 1024 && (k == 1 ? gemm_big_streams_gen(K) : after)) {
        if (p.D == 2) least = K >= 512 ? 12 : K < 192 && C % 4 ? 48 : 40;
        else least = K < 512 ? kBigTiles : K < 1024 ? 36 : K == 1024 ? 44 : 52;
        if (N > 512 && least < kBigTiles && k + 1 < p.D && p.H[k + 1] > 64 && !big_kernel(p, C, k + 1, true))
            least = K >= 768 && K <= 1024 ? 52 : kBigTiles;
    }
    if (big_tiles(p, k) < least) return 0;
    if (k > 1 || C % 256 == 0) return BIG_TILE;              // (its generating kernel has one scenario per row tile)
    return gemm_span_shape(C, K, N) ? BIG_SPAN : 0;
}

static ab_status plan_scoring(const ab_model_desc *d, int64_t S, int32_t C, ScorePlan *p)
{
    memset(p, 0, sizeof(*p));
    p->dtype = d->compute_dtype;
    p->base = d->tensor_encoder == 2 ? 3 : d->tensor_encoder ? 2 : 0;
    p->Fs = (d->tensor_encoder ? d->enc_hidden[1] : d->n_layers * d->n_stats) + d->n_scalars;
    p->F = p->Fs + 2;
    p->Kp = round_up(p->Fs, 64);
    p->D = d->n_hidden;
    int hmax = 0;
    for (int k = 0; k < p->D; ++k) { p->H[k] = d->hidden[k]; if (p->H[k] > hmax) hmax = p->H[k]; }
    if ((int64_t)C * p->H[0] >= (1LL << 31)) return AB_ERR_UNSUPPORTED;
    int64_t cs = kTargetChunkRows / C;
    if (cs < 1) cs = 1;
    if (cs > S) cs = S > 0 ? S : 1;
    const int64_t cap = ((1LL << 31) - 1) / p->H[0];
    if (cs > cap) cs = cap;
    p->chunk_scen = cs;
    p->chunk_rows = cs * C;
    p->tile_a = slim(S, p->H[0]) ? TILE_SLIM : pick_tile(S, p->H[0]);
    for (int k = 1; k < p->D; ++k) {
        p->tile[k] = pick_tile(p->chunk_rows, p->H[k]);
        p->big[k] = big_kernel(*p, C, k, p->big[k - 1] != 0);
    }
    p->nt_last = 1;
    int nt_room = 1;              // (the generic tiles' below kBigTiles, so that the size does not fall where the large kernels begin; from
                                  //  kBigTiles on it does, as at the lines between the generic tiles: ab_workspace_bytes says so)
    if (p->D >= 2) {
        const int kl = p->D - 1, generic = p->H[kl] / tile_edge(p->tile[kl]);
        p->nt_last = p->big[kl] ? p->H[kl] / 256 : generic;
        nt_room = p->big[kl] && big_tiles(*p, kl) >= kBigTiles ? p->nt_last : generic;
    }
    const size_t es = elem_size(p->dtype);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    p->off_xs = take((size_t)(S > 0 ? S : 1) * p->Kp * es);
    p->off_w1s = take((size_t)p->H[0] * p->Kp * es);
    p->off_aterm = take((size_t)(S > 0 ? S : 1) * p->H[0] * 4);
    p->off_bterm = take((size_t)C * p->H[0] * 4);
    p->off_cfgv = take(((size_t)2 * p->H[0] + 2 * (size_t)C) * 4);
    p->off_wout = take((size_t)(p->H[p->D - 1] + 1) * 4);     // folded output weights, then the folded bias
    p->off_xrow = take((size_t)p->chunk_rows * 2 * 4);          // per-scenario grids: (phi(S_p), phi(S_c)) of a chunk's rows
    p->off_partial = take((size_t)p->chunk_rows * nt_room * 4);
    p->off_act0 = p->off_act1 = 0;
    if (p->D >= 3) p->off_act0 = take((size_t)p->chunk_rows * hmax * es);
    if (p->D >= 4) p->off_act1 = take((size_t)p->chunk_rows * hmax * es);
    p->v_chunk = S < kVChunk ? (S > 0 ? S : 1) : kVChunk;
    for (int k = 1; k < p->D; ++k) p->v_tile[k] = slim(p->v_chunk, p->H[k]) ? TILE_SLIM : pick_tile(p->v_chunk, p->H[k]);
    p->off_vx = take((size_t)p->v_chunk * 2 * 4);
    p->off_vact0 = p->off_vact1 = p->off_vlast = 0;
    if (p->D >= 2) p->off_vlast = take((size_t)p->v_chunk * p->H[p->D - 1] * 4);
    if (p->D >= 3) p->off_vact0 = take((size_t)p->v_chunk * hmax * es);
    if (p->D >= 4) p->off_vact1 = take((size_t)p->v_chunk * hmax * es);
    p->total = off;
    // Small products go to gemm_slim.hip.  Its score epilogue leaves twice the partial sums; they go where the scenario
    // rows and the packed first layer were, done with by then, so that no call needs a larger workspace than before.
    for (int k = 1; k < p->D; ++k) {
        if (p->big[k] || !slim(p->chunk_rows, p->H[k])) continue;
        if (k == p->D - 1) {
            if ((size_t)p->chunk_rows * (p->H[k] / 32) * 4 > p->off_aterm - p->off_xs) continue;
            p->nt_last = p->H[k] / 32;
            p->off_partial = p->off_xs;
        }
        p->tile[k] = TILE_SLIM;
    }
    // fp32 products of enough work: bf16 matrix cores with split operands (gemm_split.hip).  A work-group takes one column
    // tile; of the last product several where the room for the partial sums does not hold one value a tile: in as few groups as
    // come within a twentieth of the fewest rounds on the chip's 512 places for work-groups.  All tiles one group's / so, us a
    // call: 64-4096 with 8192 rows 126 / 35 (59 on the fp32 instruction), 133120 rows 461 / 402, 128-2048 with 16384 106 / 54; in
    // the most groups / so, 64-4096 with 65536 rows 216 / 202, 532480 rows 1631 / 1505.
    for (int k = 1; k < p->D; ++k) {
        const int bn = p->H[k] % 128 == 0 ? 128 : 64, n_tiles = p->H[k] / bn;
        const int64_t m_tiles = (p->chunk_rows + 127) / 128;
        if (p->dtype != AB_F32 || p->tile[k] == TILE_SLIM || m_tiles * n_tiles < kSplitTiles) continue;
        p->split[k] = n_tiles;
        if (k == p->D - 1) {
            if (p->nt_last < n_tiles) {
                auto rounds = [&](int groups) { return (m_tiles * groups + 511) / 512 * (n_tiles / groups); };
                int64_t fewest = rounds(1);
                for (int n = 2; n <= p->nt_last; ++n)
                    if (n_tiles % n == 0 && rounds(n) < fewest) fewest = rounds(n);
                int n = 1;
                while (n_tiles % n != 0 || rounds(n) * 20 > fewest * 21) ++n;
                p->split[k] = n;
            }
            p->nt_last = p->split[k];
        }
    }
    return AB_OK;
}

#define AB_HIP(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return AB_ERR_DEVICE; } while (0)

// Flat statistics of few scenarios: transform and the scenario term's product in the first launch (scenario_term_kernel), every
// column tile transforming its scenarios' statistics anew; with more of them that costs more than the launch that goes away.
// Joined / apart, us a call: bf16, 512 units, 16 scenarios (32 tiles of 16 x 16) 13.1 / 17.3 with 304 columns, 27.9 / 30.4 with 2086;
// 100 scenarios (224 tiles) 21.8 / 26.5 and 38.2 / 40.8; 160 (320) 25.4 / 27.8 and 45.7 / 41.8; 300 (608) 28.1 / 27.7 and 53 / 43;
// 1024 units, 388 columns, 64 scenarios (256) 31.6 / 34.7, 160 (640) 37.3 / 35.2.
// fp32, 64 units, 52 columns, one scenario 11.0 / 17.0, 8000 (500 tiles of 32 x 32) 54.2 / 61.3 with 388; 256 units, 388 columns, 2000
// scenarios (504) 101.6 / 106.3; 2104 columns, one 18.8 / 25.3, 17 32.1 / 28.8;
// 64 units, 20 scenarios (2) 757 columns 19.1 / 19.6, 907 21.6 / 20.9; 256 units, 20 (8) 907 23.4 / 22.8, 64 (16) 32.0 / 32.1
// Long rows in bf16: the joined launch gains what packing W1 took, so by units, and loses by the logarithms of a whole row in each
// column tile, the more where they are not the hardware's (n not a multiple of four, or no room for eight columns behind them).
// Those: 64 units 1507 columns 15.7 / 15.6, 2107 17.5 / 16.1, 4096 22.1 / 17.7; 512 units, one scenario 1807 18.0 / 18.0, 3007
// 20.9 / 19.9, 20 scenarios 3007 23.9 / 22.4, 33 29.9 / 30.1, 64 4096 31.8 / 33.8; 768 units, one 3007 21.6 / 22.1; 1024 units
// 4096 24.2 / 28.2.  The hardware's: 64 units, one scenario 2284 14.9 / 15.2, 3004 16.6 / 16.0, two 3304 16.8 / 17.8, 3604
// 17.4 / 17.1; 512 units 3604 18.4 / 19.7.
static int term_columns(const ab_model_desc *d, int64_t S)
{
    const int H = d->hidden[0], n_stat = d->n_layers * d->n_stats;
    if (encode_quad_columns(n_stat, round_up(n_stat + d->n_scalars, 64))) return H >= 512 ? 4096 : S == 1 ? 2400 : 3400;
    return H < 512 ? 1500 : H < 768 && S <= 32 ? 1700 : 4096;
}

bool term_in_first_launch(const ab_model_desc *d, int64_t S)
{
    if (d->tensor_encoder || d->n_hidden < 1) return false;
    const int H = d->hidden[0], Fs = d->n_layers * d->n_stats + d->n_scalars;
    const int64_t tiles16 = (S + 15) / 16 * (H / 16), tiles32 = (S + 31) / 32 * (H / 32);
    if (d->compute_dtype == AB_BF16 || S <= 16)
        return Fs <= (d->compute_dtype == AB_BF16 ? term_columns(d, S) : 4096) && (tiles16 <= 256 || (tiles16 <= 448 && Fs <= 400));
    return Fs <= (tiles32 < 16 ? 850 : 1024) && tiles32 <= 512;
}

// The candidate term as a table [C, H]: only the generic tiles and the scorer with one hidden layer read it (a per-scenario grid
// comes in factored form there too).  Its blocks run slower beside the scenario term's than beside the transform's (fewer fit a
// CU), so a large one keeps the first launch without the product.  Joined / apart, us a call, one scenario (x candidates) and one
// hidden layer: bf16 192 x 2560 12.9 / 14.4, 512 x 1280 16.5 / 16.6, 512 x 2560 22.7 / 19.7, 1024 x 4096 50.4 / 34.7; fp32 1024 x 1280
// 21.1 / 22.9, 512 x 4096 25.1 / 25.0, 1024 x 4096 41.0 / 35.6.
static bool needs_table(const ScorePlan &p, int per_scenario)
{
    return !per_scenario && (p.D == 1 || (!p.big[1] && !p.split[1] && p.tile[1] != TILE_SLIM));
}
static bool joined_opening(const ab_model_desc *d, const ScorePlan &p, int64_t S, int32_t C, int per_scenario)
{
    const int64_t most = p.dtype == AB_BF16 ? 1 << 19 : 3 << 19;
    return term_in_first_launch(d, S) && !(needs_table(p, per_scenario) && (int64_t)C * p.H[0] > most);
}

// The weights of the products on gemm_split.hip in their parts (6 bytes each), laid out by the pass's first launch where the workspace has room that
// the pass does not use by then: the candidate table's, the candidate rows' where the grid is shared, the second pass's (not the chosen
// pairs', which the selection of each chunk writes).  at[k]: offset in the workspace, or 0; tile[k]: columns of the tiles that they are laid out for.  Whole calls, split in each work-group / so, us: 256-256
// 38400 rows 43.9 / 41.3, 614400 392 / 366; 128-128 32768 19.2 / 17.5, 2.4 M 435 / 402; 64-64 38400 18.1 / 17.4, 2.4 M 172 / 161.
// Tiles of 256 columns (eight wavefronts, half the splitting of activations): where the product is the last one (as it stores, the larger
// work-group is slower: 256 three times, 38400 rows 82.8 -> 93.2 us), its groups allow them and a tile has 16 slabs or more.  128 columns / 256, us: 256-256
// 139200 rows 104.4 / 101.6, 1.7 M 1010 / 985; 512-512 204800 473 / 455; 128-128-256 139200 112.4 / 113.0, 204800 141.8 / 144.0; 64-256
// 139200 41.2 / 44.3, 1.7 M 316 / 357.
struct PartsPlan { size_t at[AB_MAX_HIDDEN]; int tile[AB_MAX_HIDDEN]; };
static void plan_parts(const ScorePlan &p, int32_t C, int per_scenario, PartsPlan *out)
{
    memset(out, 0, sizeof(*out));
    struct { size_t at, left; } room[3] = {{p.off_bterm, needs_table(p, per_scenario) ? 0 : (size_t)C * p.H[0] * 4},
                                           {p.off_xrow, per_scenario ? 0 : (size_t)p.chunk_rows * 8}, {p.off_vlast, p.total - p.off_vlast}};
    int n = 0;
    for (int k = 1; k < p.D && n < kMostSplitWeights; ++k) {
        if (!p.split[k]) continue;
        const size_t bytes = (size_t)p.H[k] * p.H[k - 1] * 6;               // (a multiple of 256)
        for (auto &r : room) {
            if (r.left < bytes) continue;
            const bool wide = k == p.D - 1 && p.H[k - 1] >= 256 && p.H[k] % 256 == 0 && p.H[k] / 256 % p.split[k] == 0;
            out->tile[k] = wide ? 256 : p.H[k] % 128 == 0 ? 128 : 64;
            out->at[k] = r.at;
            r.at += bytes;
            r.left -= bytes;
            ++n;
            break;
        }
    }
}

// For which column tiles hidden product k's weights lie in their parts (for tests); 0: they do not.
int scoring_parts_tile(const ab_model_desc *d, int64_t S, int32_t C, int per_scenario, int k)
{
    ScorePlan p;
    PartsPlan parts;
    if (plan_scoring(d, S, C, &p) != AB_OK) return -1;
    plan_parts(p, C, per_scenario, &parts);
    return parts.tile[k];
}

// Whether a pass opens with the joined launch (for tests).
bool scoring_joined_opening(const ab_model_desc *d, int64_t S, int32_t C, int per_scenario)
{
    ScorePlan p;
    return plan_scoring(d, S, C, &p) == AB_OK && joined_opening(d, p, S, C, per_scenario);
}

// Which kernel hidden product k (k >= 1) of a pass takes (for tests): BIG_TILE, BIG_SPAN, or 0 for the smaller tiles.
int scoring_big_kernel(const ab_model_desc *d, int64_t S, int32_t C, int k)
{
    ScorePlan p;
    return plan_scoring(d, S, C, &p) == AB_OK ? p.big[k] : -1;
}

// Into how many parts the tiles of the last round of hidden product k go on so many CUs (for tests); 0: not on a streaming kernel.
int scoring_parts_of_tiles(const ab_model_desc *d, int64_t S, int32_t C, int k, int cus)
{
    ScorePlan p;
    if (plan_scoring(d, S, C, &p) != AB_OK) return -1;
    return !p.big[k] || (k == 1 && !gemm_big_streams_gen(p.H[0])) ? 0 : stream_parts(p.chunk_rows, p.H[k], cus);
}

// How many column groups hidden product k takes on gemm_split.hip (for tests); 0: not there.
int scoring_split_groups(const ab_model_desc *d, int64_t S, int32_t C, int k)
{
    ScorePlan p;
    return plan_scoring(d, S, C, &p) == AB_OK ? p.split[k] : -1;
}

static inline bool misaligned(const void *p, size_t a) { return ((uintptr_t)p % a) != 0; }

// defined in update.hip
size_t update_workspace_bytes(const ab_model_desc *d, int64_t B);
hipError_t launch_replay_mix(const float *x_new, const float *t_new, int64_t n_new, const float *x_old,
                             const float *t_old, int64_t n_old, const int32_t *pick, int64_t B, int32_t F,
                             int32_t n_out, float *x_out, float *t_out, hipStream_t st);
ab_status online_update(const ab_model_desc *d, ab_params *params, const float *x_raw, const float *target,
                        int64_t B, float lr, float beta1, float beta2, float eps, float *loss_out,
                        void *workspace, size_t ws_bytes, int first_trainable, hipStream_t st);

}  // namespace ab

using namespace ab;

extern "C" {

int32_t ab_version(void) { return 110; }

void ab_set_trace(ab_trace_fn fn, void *user) { g_trace_fn = fn; g_trace_user = user; }

const char *ab_status_string(ab_status s)
{
    switch (s) {
    case AB_OK: return "ok";
    case AB_ERR_NULL: return "a required pointer is NULL";
    case AB_ERR_SHAPE: return "a size is non-positive or inconsistent";
    case AB_ERR_DTYPE: return "unknown compute dtype";
    case AB_ERR_ALIGN: return "a pointer misses its required alignment";
    case AB_ERR_WORKSPACE: return "workspace missing or too small";
    case AB_ERR_UNSUPPORTED: return "description not supported by this library";
    case AB_ERR_DEVICE: return "HIP reported an error";
    default: return "unknown status";
    }
}

size_t ab_workspace_bytes(const ab_model_desc *desc, int64_t S, int32_t C, int64_t B)
{
    if (check_desc(desc) != AB_OK || S < 0 || C < 0 || B < 0) return 0;
    size_t need = 0;
    if (C > 0 && desc->n_hidden == 0) {
        need = 256;                        // the linear scorer runs in one launch and uses no workspace
    } else if (C > 0) {
        ScorePlan p;
        if (plan_scoring(desc, S, C, &p) != AB_OK) return 0;
        need = p.total;
    }
    if (B > 0) {
        const size_t u = update_workspace_bytes(desc, B);
        if (u == 0) return 0;
        if (u > need) need = u;
    }
    return need;
}

}  // extern "C"

// Scoring with the workspace given by address: the body of both scoring entry points.
static ab_status score_candidates_in(const ab_model_desc *desc, const ab_params *params,
                                     const ab_stats *stats, const ab_grid *grid,
                                     float *scores, int32_t *best_idx, float *best_score, float *v_best,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    ab_status rc = check_desc(desc);
    if (rc != AB_OK) return rc;
    if (!params || !stats || !grid) return AB_ERR_NULL;
    if (stats->S == 0) return AB_OK;      // nothing to score: valid no-op, no pointer is looked at
    if (!scores && !best_idx) return AB_ERR_NULL;
    if (best_score && !best_idx) return AB_ERR_NULL;
    if (v_best && !best_idx) return AB_ERR_NULL;
    if (stats->S < 0 || grid->P <= 0 || grid->Q <= 0) return AB_ERR_SHAPE;
    if ((int64_t)grid->P * grid->Q > (1 << 24)) return AB_ERR_SHAPE;
    if (!grid->partition_bytes || !grid->credit_mult) return AB_ERR_NULL;
    if (grid->per_scenario != 0 && grid->per_scenario != 1) return AB_ERR_SHAPE;
    if (misaligned(grid->partition_bytes, 4) || misaligned(grid->credit_mult, 4)) return AB_ERR_ALIGN;
    const int64_t S = stats->S;
    const int32_t C = grid->P * grid->Q;
    if (S > 0 && (!stats->dyn || (desc->n_scalars > 0 && !stats->scalars))) return AB_ERR_NULL;
    if (stats->layers_of && !desc->tensor_encoder) return AB_ERR_UNSUPPORTED;   // the flat layout has one width
    if (misaligned(stats->layers_of, 4)) return AB_ERR_ALIGN;
    if (desc->n_hidden == 0) {
        // no hidden layer: V = W x + b, one launch, no workspace
        if (!params->W[0] || !params->b[0]) return AB_ERR_NULL;
        if (misaligned(params->W[0], 16) || misaligned(params->b[0], 4)) return AB_ERR_ALIGN;
        if (misaligned(stats->dyn, 4) || misaligned(stats->scalars, 4) || misaligned(scores, 4) ||
            misaligned(best_idx, 4) || misaligned(best_score, 4) || misaligned(v_best, 4)) return AB_ERR_ALIGN;
        hipStream_t st0 = (hipStream_t)stream;
        const double Fs0 = (double)desc->n_layers * desc->n_stats + desc->n_scalars;
        TraceScope ts("score_linear", (double)S * (Fs0 * 4.0 + (scores ? C * 4.0 : 0.0) + 8.0), 1, st0);
        AB_HIP(launch_score_linear(desc->compute_dtype, desc, params, stats->dyn, stats->scalars, grid, S, scores,
                                   best_idx, best_score, v_best, st0));
        return AB_OK;
    }
    ScorePlan p;
    rc = plan_scoring(desc, S, C, &p);
    if (rc != AB_OK) return rc;
    const int n_layers_total = p.base + p.D + 1;
    for (int k = 0; k < n_layers_total; ++k) {
        if (!params->W[k] || !params->b[k]) return AB_ERR_NULL;
        if (misaligned(params->W[k], 16) || misaligned(params->b[k], 4)) return AB_ERR_ALIGN;
    }
    if (misaligned(stats->dyn, 4) || misaligned(stats->scalars, 4) || misaligned(scores, 4) ||
        misaligned(best_idx, 4) || misaligned(best_score, 4) || misaligned(v_best, 4)) return AB_ERR_ALIGN;
    if (!workspace || workspace_bytes < p.total) return AB_ERR_WORKSPACE;
    if (misaligned(workspace, 256)) return AB_ERR_ALIGN;
    if (S == 0) return AB_OK;

    hipStream_t st = (hipStream_t)stream;
    if (!v_best && score_tiny_supported(desc, S, C)) {
        // the paper's own operating point (a job, tens of candidates, a small scorer): one launch does everything
        double fl = (double)p.H[0] * p.Fs * 2.0 * S;
        for (int k = 0; k < p.D; ++k) fl += 2.0 * S * C * p.H[k] * (k ? p.H[k - 1] : 3);
        TraceScope ts("score_tiny", fl, 0, st);
        AB_HIP(launch_score_tiny(p.dtype, desc, params, stats->dyn, stats->scalars, grid->partition_bytes,
                                 grid->credit_mult, grid->P, grid->Q, grid->per_scenario, S, scores, best_idx,
                                 best_score, st));
        return AB_OK;
    }
    unsigned char *ws = (unsigned char *)workspace;
    void *xs = ws + p.off_xs, *w1s = ws + p.off_w1s;
    float *a_term = (float *)(ws + p.off_aterm);
    const bool table = needs_table(p, grid->per_scenario);
    float *b_term = table ? (float *)(ws + p.off_bterm) : nullptr;
    float *w_out_f = (float *)(ws + p.off_wout), *partial = (float *)(ws + p.off_partial);
    float *cfg_vec = (float *)(ws + p.off_cfgv);
    float *xp_row = (float *)(ws + p.off_xrow), *xc_row = xp_row + p.chunk_rows;
    const int per_scenario = grid->per_scenario;
    PartsPlan parts;
    plan_parts(p, C, per_scenario, &parts);
    SplitWeightsArgs split_weights{};
    for (int k = 1; k < p.D; ++k)
        if (parts.at[k])
            split_weights.w[split_weights.n++] = SplitWeights{(const float *)params->W[p.base + k], (i32x4 *)(ws + parts.at[k]), p.H[k], p.H[k - 1], parts.tile[k]};
    const double parts_bytes = 80.0 * split_weights_items(split_weights);
    void *act[2] = {ws + p.off_act0, ws + p.off_act1};
    const int dt = p.dtype;

    // 1. scenario rows: transformed statistics (or pooled tensor embedding) + scalars, K-padded
    const double es = (double)elem_size(dt);
    bool prep_done = false, term_done = false;
    bool grid_done = false;             // a per-scenario grid's rows: in the first launch if all scenarios are one chunk
    if (desc->tensor_encoder) {
        // the encoder, and in its launch, where they fit, the scalars' columns and the layer-1 preparation (step 2); every pass
        // reports the same stages, so those come empty then
        const EncoderSide side{stats->scalars, params->W[p.base], params->b[p.base], p.F, p.Fs, p.H[0], w1s, grid, b_term, cfg_vec,
                               params->W[p.base + p.D], params->b[p.base + p.D], p.H[p.D - 1], w_out_f};
        if (desc->tensor_encoder == 2) {
            // per scenario and layer: two gate products (256 x 96 and 256 x 128) and the K -> 32 embedding
            TraceScope ts("lstm_encoder", (double)S * desc->n_layers * 2.0 * (256.0 * 224.0 + 32.0 * desc->n_stats), 0, st);
            AB_HIP(launch_lstm_encoder(desc, stats->dyn, params->W[0], params->b[0], params->W[1], params->b[1],
                                       params->W[2], params->b[2], xs, p.Kp, S, stats->layers_of, side, &prep_done, st));
        } else {
            TraceScope ts("tensor_encoder", (double)S * desc->n_layers * 2.0 * (desc->n_stats * 128.0 + 128.0 * 128.0),
                          0, st);
            AB_HIP(launch_tensor_encoder(desc, stats->dyn, params->W[0], params->b[0], params->W[1],
                                         params->b[1], xs, p.Kp, S, stats->layers_of, side, &prep_done, st));
        }
        if (prep_done) {
            { TraceScope ts("encode_stats", 0.0, 1, st); }
            { TraceScope ts("prep_layer1", 0.0, 1, st); }
        } else {
            TraceScope ts("encode_stats", (double)S * (desc->n_scalars * 4.0 + (p.Kp - desc->enc_hidden[1]) * es), 1, st);
            AB_HIP(launch_encode_stats(dt, desc, stats->dyn, stats->scalars, xs, S, p.Kp, desc->enc_hidden[1], 0, st));
        }
    } else if (joined_opening(desc, p, S, C, per_scenario)) {
        // few scenarios: transform, preparation (step 2) and scenario term (step 3) in one launch, reported as the product that
        // it is; every pass reports the same stages, so the transform's comes empty
        { TraceScope ts("encode_and_prep", 0.0, 1, st); }
        TraceScope ts("gemm_scenario_term", 2.0 * S * p.H[0] * p.Kp, 0, st);
        AB_HIP(launch_scenario_term(dt, desc, stats->dyn, stats->scalars, S, params->W[p.base], params->b[p.base], p.F, p.Fs, p.H[0], p.Kp,
                                    a_term, grid, b_term, cfg_vec, params->W[p.base + p.D], params->b[p.base + p.D], p.H[p.D - 1],
                                    w_out_f, per_scenario && p.chunk_scen >= S ? xp_row : nullptr, xc_row, split_weights, st));
        prep_done = term_done = true;
        grid_done = p.chunk_scen >= S;
    } else {
        // flat statistics: transform and layer-1 preparation (step 2) share one launch where the layout allows
        const double prep_bytes = (double)p.H[0] * (p.F * es + p.Kp * es) + (table ? (double)C * p.H[0] * 4.0 : 0.0) +
                                  (per_scenario && p.chunk_scen >= S ? (double)S * C * 8.0 : 0.0) + parts_bytes;
        TraceScope ts("encode_and_prep", (double)S * (p.Fs * 4.0 + p.Kp * es) + prep_bytes, 1, st);
        AB_HIP(launch_encode_and_prep(dt, desc, stats->dyn, stats->scalars, xs, S, p.Kp, params->W[p.base],
                                      params->b[p.base], p.F, p.Fs, p.H[0], w1s, grid, b_term, cfg_vec,
                                      params->W[p.base + p.D], params->b[p.base + p.D], p.H[p.D - 1], w_out_f,
                                      per_scenario && p.chunk_scen >= S ? xp_row : nullptr, xc_row, split_weights, &prep_done, st));
        grid_done = prep_done && p.chunk_scen >= S;
        if (!prep_done) AB_HIP(launch_encode_stats(dt, desc, stats->dyn, stats->scalars, xs, S, p.Kp, 0, 1, st));
    }
    // 2. layer-1 split: packed statistics columns of W1, candidate term B[c], fp32 output weights
    if (!prep_done) {
        TraceScope ts("prep_layer1", (double)p.H[0] * (p.F * es + p.Kp * es) + (table ? (double)C * p.H[0] * 4.0 : 0.0) + parts_bytes, 1, st);
        AB_HIP(launch_prep_layer1(dt, desc, params->W[p.base], params->b[p.base], p.F, p.Fs, p.H[0], p.Kp, w1s,
                                  grid, b_term, cfg_vec, params->W[p.base + p.D], params->b[p.base + p.D],
                                  p.H[p.D - 1], w_out_f, split_weights, st));
    }
    // 3. scenario term A[s] = x_s W1_s^T + b1 (fp32 out)
    if (!term_done) {
        GemmArgs g;
        memset(&g, 0, sizeof(g));
        g.A = xs; g.lda = p.Kp; g.B = w1s; g.ldb = p.Kp;
        g.M = S; g.N = p.H[0]; g.K = p.Kp;
        g.out = a_term; g.ldo = p.H[0]; g.out_f32 = 1;
        g.bias = params->b[p.base];
        TraceScope ts("gemm_scenario_term", 2.0 * S * p.H[0] * p.Kp, 0, st);
        AB_HIP(launch_gemm(dt, p.tile_a, AMODE_LOAD, EPI_STORE, g, st));
    }
    // the chosen candidate's pair for step 5: written by the selection where its room holds all scenarios (a launch of its
    // own; 300 scenarios of 256 candidates with V, a call: 115.8 us with that launch, 114.3 so)
    float *xp_sel = (float *)(ws + p.off_vx), *xc_sel = xp_sel + p.v_chunk;
    const bool pairs_done = S <= p.v_chunk;
    auto chosen_at = [&](int64_t s0, float *xp, float *xc) {
        const int64_t own = per_scenario ? s0 : 0;
        return ChosenArgs{grid->partition_bytes + own * grid->P, grid->credit_mult + own * grid->Q, grid->P, grid->Q, per_scenario,
                          desc->enc_partition, desc->enc_credit, xp, xc};
    };
    // 4. candidate rows, a chunk of scenarios at a time
    for (int64_t s0 = 0; s0 < S; s0 += p.chunk_scen) {
        const int64_t ns = (S - s0 < p.chunk_scen) ? S - s0 : p.chunk_scen;
        const int64_t rows = ns * C;
        const float *a_chunk = a_term + s0 * p.H[0];
        int nt = 1;
        if (per_scenario && !grid_done) {
            TraceScope ts("grid_rows", (double)rows * 8.0, 1, st);
            AB_HIP(launch_grid_rows(desc, grid->partition_bytes + s0 * grid->P, grid->credit_mult + s0 * grid->Q,
                                    grid->P, grid->Q, xp_row, xc_row, rows, st));
        }
        if (p.D == 1) {
            TraceScope ts("score_single_hidden", 3.0 * rows * p.H[0], 0, st);
            AB_HIP(launch_score_single_hidden(a_chunk, b_term, w_out_f, partial, rows, C, p.H[0], cfg_vec,
                                              cfg_vec + p.H[0], per_scenario ? xp_row : nullptr,
                                              per_scenario ? xc_row : nullptr, st));
        } else {
            for (int k = 1; k < p.D; ++k) {
                GemmArgs g;
                memset(&g, 0, sizeof(g));
                if (k == 1) {
                    g.a_term = a_chunk; g.b_term = b_term; g.ldt = p.H[0]; g.C = C;
                    g.wp = cfg_vec; g.wc = cfg_vec + p.H[0]; g.xp = cfg_vec + 2 * p.H[0]; g.xc = cfg_vec + 2 * p.H[0] + C;
                    if (per_scenario) { g.xp = xp_row; g.xc = xc_row; g.x_per_row = 1; }
                    g.xp_runs4 = grid->Q % 4 == 0;          // (row = s C + p Q + q and 4 | Q: four adjacent rows, one p)
                }
                else { g.A = act[k & 1]; g.lda = p.H[k - 1]; }
                g.B = params->W[p.base + k]; g.ldb = p.H[k - 1];
                g.M = rows; g.N = p.H[k]; g.K = p.H[k - 1];
                g.bias = params->b[p.base + k]; g.relu = 1;
                const bool last = (k == p.D - 1);
                if (last) { g.w_out = w_out_f; g.partial = partial; nt = p.nt_last; }
                else { g.out = act[(k + 1) & 1]; g.ldo = p.H[k]; }
                TraceScope ts(k == 1 ? (last ? "gemm_hidden_first_last" : "gemm_hidden_first")
                                     : (last ? "gemm_hidden_last" : "gemm_hidden_mid"),
                              2.0 * rows * p.H[k] * p.H[k - 1], 0, st);
                const int amode = k == 1 ? AMODE_GEN : AMODE_LOAD, epi = last ? EPI_SCORE : EPI_STORE;
                if (parts.at[k]) g.B_parts = ws + parts.at[k];
                if (p.split[k])
                    AB_HIP(launch_gemm_split(amode, epi, g, p.split[k], parts.tile[k], st));
                else if (p.big[k] == BIG_SPAN)
                    AB_HIP(launch_gemm_span(epi, g, st));
                else if (p.big[k] && gemm_big_supported(dt, amode, epi, g))
                    AB_HIP(launch_gemm_big(amode, epi, g, st));
                else if (p.big[k])
                    return AB_ERR_UNSUPPORTED;     // cannot happen: the plan checked the same conditions
                else    // the generic tiles take a per-scenario grid's operand in its factored form
                    AB_HIP(launch_gemm(dt, p.tile[k], amode == AMODE_GEN && per_scenario ? AMODE_GENV : amode, epi, g, st));
            }
        }
        const ChosenArgs pair = chosen_at(s0, xp_sel + s0, xc_sel + s0);
        TraceScope ts("finish_select", (double)rows * (nt * 4.0 + (scores ? 4.0 : 0.0)) + ns * 8.0, 1, st);
        AB_HIP(launch_finish_select(partial, nt, C, w_out_f + p.H[p.D - 1],
                                    scores ? scores + s0 * C : nullptr, C,
                                    best_idx ? best_idx + s0 : nullptr,
                                    best_score ? best_score + s0 : nullptr, ns, C, v_best && pairs_done ? &pair : nullptr, st));
    }
    // 5. the chosen candidate's prediction vector: the hidden chain once more on one row per scenario (the row's
    // candidate values are those of best_idx), then the output layer unit by unit
    if (v_best) {
        const int n_out = desc->n_outputs > 0 ? desc->n_outputs : 1;
        float *h_last = (float *)(ws + p.off_vlast);
        void *vact[2] = {ws + p.off_vact0, ws + p.off_vact1};
        for (int64_t s0 = 0; s0 < S; s0 += p.v_chunk) {
            const int64_t ns = (S - s0 < p.v_chunk) ? S - s0 : p.v_chunk;
            if (!pairs_done) {
                TraceScope ts("chosen_pair", (double)ns * 20.0, 1, st);
                AB_HIP(launch_chosen_pair(chosen_at(s0, xp_sel, xc_sel), best_idx + s0, ns, st));
            }
            for (int k = 1; k < p.D; ++k) {
                GemmArgs g;
                memset(&g, 0, sizeof(g));
                if (k == 1) {
                    g.a_term = a_term + s0 * p.H[0]; g.ldt = p.H[0]; g.C = 1;
                    g.wp = cfg_vec; g.wc = cfg_vec + p.H[0]; g.xp = xp_sel; g.xc = xc_sel; g.x_per_row = 1;
                } else { g.A = vact[k & 1]; g.lda = p.H[k - 1]; }
                g.B = params->W[p.base + k]; g.ldb = p.H[k - 1];
                g.M = ns; g.N = p.H[k]; g.K = p.H[k - 1];
                g.bias = params->b[p.base + k]; g.relu = 1;
                if (k == p.D - 1) { g.out = h_last; g.ldo = p.H[k]; g.out_f32 = 1; }
                else { g.out = vact[(k + 1) & 1]; g.ldo = p.H[k]; }
                TraceScope ts("gemm_chosen_rows", 2.0 * ns * p.H[k] * p.H[k - 1], 0, st);
                AB_HIP(launch_gemm(dt, p.v_tile[k], k == 1 ? AMODE_GENV : AMODE_LOAD, EPI_STORE, g, st));
            }
            TraceScope ts("output_v", (double)ns * (p.H[p.D - 1] * 4.0 + n_out * 4.0), 1, st);
            AB_HIP(launch_output_v(dt, p.D >= 2 ? h_last : nullptr, a_term + s0 * p.H[0], cfg_vec, cfg_vec + p.H[0],
                                   xp_sel, xc_sel, params->W[p.base + p.D], params->b[p.base + p.D], p.H[p.D - 1],
                                   n_out, best_idx + s0, v_best + s0 * n_out, ns, st));
        }
    }
    return AB_OK;
}

// Workspace of ab_score_candidates_static: lives in the code object, one copy per device.  The name is a
// host-side stand-in only; the device address is looked up once per device and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[AB_STATIC_SCRATCH_BYTES];
static const int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

static ab_status static_scratch(void **out)
{
    int dev = -1;
    AB_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return AB_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        AB_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return AB_ERR_DEVICE;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return AB_OK;
}

extern "C" {

ab_status ab_score_candidates(const ab_model_desc *desc, const ab_params *params,
                              const ab_stats *stats, const ab_grid *grid,
                              float *scores, int32_t *best_idx, float *best_score,
                              void *workspace, size_t workspace_bytes, void *stream)
{
    return score_candidates_in(desc, params, stats, grid, scores, best_idx, best_score, nullptr,
                               workspace, workspace_bytes, stream);
}

ab_status ab_score_candidates_v(const ab_model_desc *desc, const ab_params *params,
                                const ab_stats *stats, const ab_grid *grid,
                                float *scores, int32_t *best_idx, float *best_score, float *v_best,
                                void *workspace, size_t workspace_bytes, void *stream)
{
    return score_candidates_in(desc, params, stats, grid, scores, best_idx, best_score, v_best,
                               workspace, workspace_bytes, stream);
}

size_t ab_static_scratch_bytes(void) { return AB_STATIC_SCRATCH_BYTES; }

ab_status ab_score_candidates_static(const ab_model_desc *desc, const ab_params *params,
                                     const ab_stats *stats, const ab_grid *grid,
                                     float *scores, int32_t *best_idx, float *best_score, void *stream)
{
    ab_status rc = check_desc(desc);
    if (rc != AB_OK) return rc;
    if (!params || !stats || !grid) return AB_ERR_NULL;
    if (desc->n_hidden > 0 && stats->S > 0 && grid->P > 0 && grid->Q > 0 && (int64_t)grid->P * grid->Q <= (1 << 24)) {
        // refuse what does not fit before anything else is looked at
        ScorePlan p;
        rc = plan_scoring(desc, stats->S, grid->P * grid->Q, &p);
        if (rc != AB_OK) return rc;
        if (p.total > AB_STATIC_SCRATCH_BYTES) return AB_ERR_WORKSPACE;
    }
    void *ptr = nullptr;
    rc = static_scratch(&ptr);
    if (rc != AB_OK) return rc;
    return score_candidates_in(desc, params, stats, grid, scores, best_idx, best_score, nullptr,
                               ptr, AB_STATIC_SCRATCH_BYTES, stream);
}

ab_status ab_select_best(const float *scores, int64_t S, int32_t C, int64_t row_stride,
                         int32_t *best_idx, float *best_score, void *stream)
{
    if (!scores || !best_idx) return AB_ERR_NULL;
    if (S < 0 || C <= 0 || row_stride < C) return AB_ERR_SHAPE;
    if (misaligned(scores, 4) || misaligned(best_idx, 4) || misaligned(best_score, 4)) return AB_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    for (int64_t s0 = 0; s0 < S; s0 += (1 << 30)) {
        const int64_t ns = (S - s0 < (1 << 30)) ? S - s0 : (1 << 30);
        TraceScope ts("select_best", (double)ns * (C * 4.0 + 8.0), 1, st);
        AB_HIP(launch_finish_select(scores + s0 * row_stride, 1, row_stride, nullptr, nullptr, 0,
                                    best_idx + s0, best_score ? best_score + s0 : nullptr, ns, C, nullptr, st));
    }
    return AB_OK;
}

ab_status ab_trigger(const float *scores, int64_t S, int32_t C, int64_t row_stride,
                     const int32_t *current_idx, const float *observed,
                     float gain_threshold, float error_threshold,
                     int32_t *best_idx, float *gain, uint8_t *reconfigure, uint8_t *adapt, void *stream)
{
    if (!scores || !current_idx || !best_idx || !reconfigure) return AB_ERR_NULL;
    if (adapt && !observed) return AB_ERR_NULL;
    if (S < 0 || C <= 0 || row_stride < C) return AB_ERR_SHAPE;
    if (misaligned(scores, 4) || misaligned(current_idx, 4) || misaligned(observed, 4) ||
        misaligned(best_idx, 4) || misaligned(gain, 4)) return AB_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    for (int64_t s0 = 0; s0 < S; s0 += (1 << 30)) {
        const int64_t ns = (S - s0 < (1 << 30)) ? S - s0 : (1 << 30);
        TraceScope ts("trigger", (double)ns * (C * 4.0 + 16.0), 1, st);
        AB_HIP(launch_trigger(scores + s0 * row_stride, ns, C, row_stride, current_idx + s0,
                              observed ? observed + s0 : nullptr, gain_threshold, error_threshold,
                              best_idx + s0, gain ? gain + s0 : nullptr, reconfigure + s0,
                              adapt ? adapt + s0 : nullptr, st));
    }
    return AB_OK;
}

ab_status ab_online_update(const ab_model_desc *desc, ab_params *params,
                           const float *x_raw, const float *target, int64_t B,
                           float lr, float beta1, float beta2, float eps,
                           float *loss_out, void *workspace, size_t workspace_bytes, void *stream)
{
    ab_status rc = check_desc(desc);
    if (rc != AB_OK) return rc;
    if (desc->tensor_encoder) return AB_ERR_UNSUPPORTED;
    if (!params || !x_raw || !target) return AB_ERR_NULL;
    if (B <= 0) return AB_ERR_SHAPE;
    return online_update(desc, params, x_raw, target, B, lr, beta1, beta2, eps, loss_out,
                         workspace, workspace_bytes, 0, (hipStream_t)stream);
}

ab_status ab_online_update_tail(const ab_model_desc *desc, ab_params *params,
                                const float *x_raw, const float *target, int64_t B, int32_t first_trainable,
                                float lr, float beta1, float beta2, float eps,
                                float *loss_out, void *workspace, size_t workspace_bytes, void *stream)
{
    ab_status rc = check_desc(desc);
    if (rc != AB_OK) return rc;
    if (desc->tensor_encoder) return AB_ERR_UNSUPPORTED;
    if (!params || !x_raw || !target) return AB_ERR_NULL;
    if (B <= 0 || first_trainable < 0 || first_trainable > desc->n_hidden) return AB_ERR_SHAPE;
    return online_update(desc, params, x_raw, target, B, lr, beta1, beta2, eps, loss_out,
                         workspace, workspace_bytes, first_trainable, (hipStream_t)stream);
}

ab_status ab_replay_mix(const float *x_new, const float *target_new, int64_t n_new,
                        const float *x_old, const float *target_old, int64_t n_old,
                        const int32_t *pick, int64_t B, int32_t F, int32_t n_outputs,
                        float *x_out, float *target_out, void *stream)
{
    if (n_new < 0 || n_old < 0 || B < 0 || F <= 0 || n_outputs < 1 || n_outputs > AB_MAX_OUTPUTS) return AB_ERR_SHAPE;
    if (B == 0) return AB_OK;
    if (!pick || !x_out || !target_out) return AB_ERR_NULL;
    if ((n_new > 0 && (!x_new || !target_new)) || (n_old > 0 && (!x_old || !target_old))) return AB_ERR_NULL;
    if (n_new > 0x7fffffffLL || n_old > 0x7fffffffLL || (B + 3) / 4 > 0x7fffffffLL) return AB_ERR_UNSUPPORTED;
    if (misaligned(x_new, 4) || misaligned(x_old, 4) || misaligned(x_out, 4) || misaligned(pick, 4) ||
        misaligned(target_new, 4) || misaligned(target_old, 4) || misaligned(target_out, 4)) return AB_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    TraceScope ts("replay_mix", (double)B * (F + n_outputs) * 8.0 + (double)B * 4.0, 1, st);
    AB_HIP(launch_replay_mix(x_new, target_new, n_new, x_old, target_old, n_old, pick, B, F, n_outputs, x_out,
                             target_out, st));
    return AB_OK;
}

}  // extern "C"
