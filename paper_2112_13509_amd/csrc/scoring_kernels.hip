// Streaming kernels around the matrix-core GEMMs of the scoring path: feature transform, layer-1
// candidate term, weight packing, the shared per-tensor encoder, score assembly and argmax.
#include "internal.hpp"
#include <type_traits>
#include <string.h>

namespace ab {

// ------------------------------------------------------------------------------------------------
// Feature transform (Section 3.3 "Meta network optimizer": runtime statistics are turned into the
// network's input vector).  One thread produces two adjacent columns of one scenario's row.
//   xs[s, col0 + j]            j in [0, n_stat)            <- phi_stat(dyn[s, j])      (flat model only)
//   xs[s, col0 + n_stat + j]   j in [0, n_scal)            <- phi_scal(scal[s, j])
//   xs[s, ...up to ld)                                      <- 0   (K padding for the GEMM)
// ------------------------------------------------------------------------------------------------
struct EncodeArgs {
    const float *dyn; const float *scal;
    void *xs; int64_t S; int32_t ld;
    int32_t col0, n_stat, n_stats_per_layer, n_scal;
    ab_enc enc_stat[AB_MAX_STATS];
    ab_enc enc_scal[AB_MAX_SCALARS];
};

template <typename T>
__global__ __launch_bounds__(256) void encode_stats_kernel(const EncodeArgs a)
{
    const int pairs = (a.ld - a.col0) >> 1;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t s = gid / pairs;
    if (s >= a.S) return;
    const int j0 = (int)(gid - s * pairs) * 2;
    float v[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int j = j0 + e;
        float x = 0.f;
        if (j < a.n_stat) {
            x = phi(a.dyn[s * a.n_stat + j], a.enc_stat[j % a.n_stats_per_layer]);
        } else if (j < a.n_stat + a.n_scal) {
            const int q = j - a.n_stat;
            x = phi(a.scal[s * a.n_scal + q], a.enc_scal[q]);
        }
        v[e] = x;
    }
    const int64_t o = s * a.ld + a.col0 + j0;
    if constexpr (sizeof(T) == 2) ((uint32_t *)a.xs)[o >> 1] = pack_bf16x2(v[0], v[1]);
    else ((f32x2 *)a.xs)[o >> 1] = f32x2{v[0], v[1]};
}

// The same transform, four adjacent columns per thread (16-byte loads, 8- or 16-byte stores), for rows
// whose statistics part is a multiple of four columns and 16-byte aligned.  A work-group takes `rpb`
// rows; lane -> (row, quad) by a multiply-high with magic = floor(2^32 / q4) + 1 (exact while
// index * q4 < 2^32), likewise column -> statistic index.  The transform constants sit in LDS so that a
// lane can pick its own.  With bf16 as compute type the logarithm is the hardware's log2 (1 ulp, far
// below what the rounding to bf16 keeps) times ln 2.
template <typename T>
__device__ __forceinline__ float phi_tab(float x, const f32x4 *tab, int i)
{
    float lg;
    if constexpr (sizeof(T) == 2) lg = __builtin_amdgcn_logf(x) * 0.69314718056f;
    else lg = logf(x);
    const f32x4 t = tab[i];                        // (kind, shift, scale, -)
    return ((t.x != 0.f ? lg : x) - t.y) * t.z;
}

template <typename T>
__device__ __forceinline__ void store_quad(void *xs, int64_t o, const float (&v)[4])
{
    if constexpr (sizeof(T) == 2) {
        typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
        *(u32x2 *)((uint16_t *)xs + o) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else {
        *(f32x4 *)((float *)xs + o) = f32x4{v[0], v[1], v[2], v[3]};
    }
}

struct QuadSplit { int q4s, q4t; uint32_t magic_q4s, magic_q4t, magic_k; int rpb; };

template <typename T, int NT = 256>                        // NT threads
__device__ __forceinline__ void encode_stats_quad_block(const EncodeArgs &a, const QuadSplit &g, unsigned block)
{
    __shared__ f32x4 tab[AB_MAX_STATS + AB_MAX_SCALARS];     // statistics first, then the scalars
    if (threadIdx.x < AB_MAX_STATS + AB_MAX_SCALARS) {
        const int i = threadIdx.x;
        const ab_enc *e = i < AB_MAX_STATS ? &a.enc_stat[i] : &a.enc_scal[i - AB_MAX_STATS];
        tab[i] = f32x4{e->kind == AB_ENC_LOG ? 1.f : 0.f, e->shift, e->scale, 0.f};
    }
    __syncthreads();
    const int64_t row0 = (int64_t)block * g.rpb;
    const int rows = (int)((a.S - row0 < g.rpb) ? a.S - row0 : g.rpb);

    // the statistics columns: q4s quads a row, a thread's four loads issued before the first value is used
    const uint32_t n_a = (uint32_t)rows * (uint32_t)g.q4s;
    for (uint32_t base = 0; base < n_a; base += 4 * NT) {
        f32x4 x[4];
        uint32_t r[4];
        int col[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = base + u * NT + threadIdx.x;
            r[u] = __umulhi(i, g.magic_q4s);
            col[u] = (int)(i - r[u] * (uint32_t)g.q4s) * 4;
            if (i < n_a) x[u] = __builtin_nontemporal_load((const f32x4 *)(a.dyn + (row0 + r[u]) * a.n_stat + col[u]));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (base + u * NT + threadIdx.x >= n_a) break;
            int k = a.n_stats_per_layer == 1
                        ? 0 : col[u] - (int)__umulhi((uint32_t)col[u], g.magic_k) * a.n_stats_per_layer;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = phi_tab<T>(x[u][e], tab, k);
                k = (k + 1 == a.n_stats_per_layer) ? 0 : k + 1;
            }
            store_quad<T>(a.xs, (row0 + r[u]) * a.ld + a.col0 + col[u], v);
        }
    }

    // the scalars and the zero padding behind them: q4t quads a row
    const uint32_t n_b = (uint32_t)rows * (uint32_t)g.q4t;
    for (uint32_t i = threadIdx.x; i < n_b; i += NT) {
        const uint32_t r = __umulhi(i, g.magic_q4t);
        const int q0 = (int)(i - r * (uint32_t)g.q4t) * 4;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = q0 + e;
            v[e] = q < a.n_scal ? phi_tab<T>(a.scal[(row0 + r) * a.n_scal + q], tab, AB_MAX_STATS + q) : 0.f;
        }
        store_quad<T>(a.xs, (row0 + r) * a.ld + a.col0 + a.n_stat + q0, v);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void encode_stats_quad_kernel(const EncodeArgs a, const QuadSplit g)
{
    encode_stats_quad_block<T>(a, g, blockIdx.x);
}

// ------------------------------------------------------------------------------------------------
// Layer-1 preparation.  The first dense layer acts on [statistics | S_p | S_c]; its statistics
// columns are shared by all candidates of a scenario and its two configuration columns by all
// scenarios, so W1 x + b1 = A[s] + B[c] with A[s] = W1_s x_s + b1 (the bias rides in the A[s] GEMM's
// epilogue) and B[c] = wp * phi(S_p) + wc * phi(S_c).  This kernel packs the statistics columns of W1
// into a K-padded matrix for the A[s] GEMM, builds B[c] both as a [C, H1] matrix (generic kernels) and
// as its four generating vectors wp[H1], wc[H1], phi_p[C], phi_c[C] (the 256x256 kernel rebuilds B[c]
// from them with two FMAs instead of fetching 4 bytes per element), and widens the output weights.
// ------------------------------------------------------------------------------------------------
struct PrepArgs {
    const void *W1; int32_t F, Fs, H1, ld;      // W1[H1, F]; packed copy w1s[H1, ld]
    void *w1s;
    const float *b1;
    const float *part; const float *cred; int32_t P, Q;
    ab_enc enc_part, enc_cred;
    float *b_term;                               // [P*Q, H1], or NULL: not wanted
    float *wp_f, *wc_f, *xp_f, *xc_f;            // [H1], [H1], [P*Q], [P*Q]
    const void *Wout; const float *b_out; int32_t H_last, n_out; float *w_out_f;   // w_out_f[H_last + 1]
};

template <typename T>
__device__ __forceinline__ float load_as_f32(const void *p, int64_t i)
{
    if constexpr (sizeof(T) == 2) return bf16_bits_to_f32(((const uint16_t *)p)[i]);
    else return ((const float *)p)[i];
}

template <typename T>
__device__ __forceinline__ void prep_layer1_item(const PrepArgs &a, int64_t gid)
{
    const int64_t n_pack = a.w1s ? (int64_t)a.H1 * a.ld : 0;
    const int64_t n_bt = a.b_term ? (int64_t)a.P * a.Q * a.H1 : 0;
    if (gid < n_pack) {
        const int h = (int)(gid / a.ld), k = (int)(gid - (int64_t)h * a.ld);
        if constexpr (sizeof(T) == 2) {
            uint16_t v = (k < a.Fs) ? ((const uint16_t *)a.W1)[(int64_t)h * a.F + k] : (uint16_t)0;
            ((uint16_t *)a.w1s)[gid] = v;
        } else {
            ((float *)a.w1s)[gid] = (k < a.Fs) ? ((const float *)a.W1)[(int64_t)h * a.F + k] : 0.f;
        }
    } else if (gid < n_pack + n_bt) {
        const int64_t e = gid - n_pack;
        const int c = (int)(e / a.H1), h = (int)(e - (int64_t)c * a.H1);
        const float xp = phi(a.part[c / a.Q], a.enc_part), xc = phi(a.cred[c % a.Q], a.enc_cred);
        const float wp = load_as_f32<T>(a.W1, (int64_t)h * a.F + a.Fs);
        const float wc = load_as_f32<T>(a.W1, (int64_t)h * a.F + a.Fs + 1);
        a.b_term[e] = wp * xp + wc * xc;
    } else if (gid < n_pack + n_bt + a.H_last) {
        const int h = (int)(gid - n_pack - n_bt);
        // the output layer folded to one unit: the mean over its n_out rows (a candidate's score is the mean
        // of the per-worker predictions); the folded bias follows the weights
        float acc = 0.f, bacc = 0.f;
        for (int w = 0; w < a.n_out; ++w) acc += load_as_f32<T>(a.Wout, (int64_t)w * a.H_last + h);
        a.w_out_f[h] = acc / (float)a.n_out;
        if (h == 0) {
            for (int w = 0; w < a.n_out; ++w) bacc += a.b_out[w];
            a.w_out_f[a.H_last] = bacc / (float)a.n_out;
        }
    } else if (gid < n_pack + n_bt + a.H_last + a.H1) {
        const int h = (int)(gid - n_pack - n_bt - a.H_last);
        a.wp_f[h] = load_as_f32<T>(a.W1, (int64_t)h * a.F + a.Fs);
        a.wc_f[h] = load_as_f32<T>(a.W1, (int64_t)h * a.F + a.Fs + 1);
    } else if (gid < n_pack + n_bt + a.H_last + a.H1 + (int64_t)a.P * a.Q) {
        const int c = (int)(gid - n_pack - n_bt - a.H_last - a.H1);
        a.xp_f[c] = phi(a.part[c / a.Q], a.enc_part);
        a.xc_f[c] = phi(a.cred[c % a.Q], a.enc_cred);
    }
}

// The fp32 preparation also lays out the hidden weights in their parts for gemm_split.hip, in the work-groups from parts.from on, the last.
struct NoParts {};
template <typename T> using PartsOf = std::conditional_t<sizeof(T) == 4, SplitWeightsArgs, NoParts>;
template <int NT> __device__ __forceinline__ bool parts_block(const SplitWeightsArgs &a)
{
    if (blockIdx.x < a.from) return false;
    split_weights_item(a, (int64_t)(blockIdx.x - a.from) * NT + threadIdx.x);
    return true;
}
template <int NT> __device__ __forceinline__ bool parts_block(const NoParts &) { return false; }
template <typename T> static PartsOf<T> parts_of(SplitWeightsArgs a, int64_t from)
{
    a.from = (uint32_t)from;
    if constexpr (sizeof(T) == 4) return a;
    else return NoParts{};
}

template <typename T>
__global__ __launch_bounds__(256) void prep_layer1_kernel(const PrepArgs a, const PartsOf<T> parts)
{
    if (parts_block<256>(parts)) return;
    prep_layer1_item<T>(a, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// What an encoder's launch takes along: the scalars' columns of the scenario rows and the layer-1 preparation, both independent of
// the encoder, in work-groups behind its own (they fill in where the encoder leaves CUs idle, or as it ends).  As two launches of
// their own / so, us a call, per-tensor encoder, 512-512 x 256 candidates: 200 scenarios 47.3 / 40.8, 512 75.1 / 71.0, 8192 898 / 887.
struct SideArgs { EncodeArgs e; QuadSplit g; PrepArgs p; unsigned enc_blocks, blocks; };
template <int NT>
__device__ __forceinline__ void side_block(const SideArgs &a, unsigned id)
{
    if (id < a.enc_blocks) encode_stats_quad_block<bf16_t, NT>(a.e, a.g, id);
    else prep_layer1_item<bf16_t>(a.p, (int64_t)(id - a.enc_blocks) * NT + threadIdx.x);
}

// Per-scenario candidate grids: the transformed pair (phi(S_p), phi(S_c)) of every (scenario, candidate) row
// of a chunk, row = s * P * Q + p * Q + q, from part[S, P] and cred[S, Q].
struct GridRowsArgs { const float *part, *cred; int32_t P, Q; ab_enc enc_part, enc_cred; float *xp_row, *xc_row; int64_t rows; };
__device__ __forceinline__ void grid_rows_item(const GridRowsArgs &a, int64_t row)
{
    if (row >= a.rows) return;
    const int Cn = a.P * a.Q;
    const int64_t s = row / Cn;
    const int c = (int)(row - s * Cn);
    a.xp_row[row] = phi(a.part[s * a.P + c / a.Q], a.enc_part);
    a.xc_row[row] = phi(a.cred[s * a.Q + c % a.Q], a.enc_cred);
}
__global__ __launch_bounds__(256) void grid_rows_kernel(const GridRowsArgs a) { grid_rows_item(a, (int64_t)blockIdx.x * 256 + threadIdx.x); }

// What opens a scoring pass of the flat model is independent of each other (the transform reads the statistics, the
// preparation the model and the grid, a per-scenario grid's rows the grid), so it shares one launch: the first
// `enc_blocks` work-groups do the feature transform (the long, memory-bound part starts at once), the short
// work-groups of the layer-1 preparation fill in behind them, then those of the grid rows (a launch of their own costs
// 4.6 us), where all scenarios are one chunk.
template <typename T>
__global__ __launch_bounds__(256) void encode_and_prep_kernel(const EncodeArgs a, const QuadSplit g, const PrepArgs p,
                                                              const GridRowsArgs r, unsigned enc_blocks, unsigned grid_from, const PartsOf<T> parts)
{
    if (blockIdx.x < enc_blocks) encode_stats_quad_block<T>(a, g, blockIdx.x);
    else if (blockIdx.x < grid_from) prep_layer1_item<T>(p, (int64_t)(blockIdx.x - enc_blocks) * 256 + threadIdx.x);
    else if (!parts_block<256>(parts)) grid_rows_item(r, (int64_t)(blockIdx.x - grid_from) * 256 + threadIdx.x);
}

// The same opening for few scenarios, with the scenario term's product in it: A[s] = W1_s phi(x_s) + b1 straight from the raw
// statistics and W1 as it lies, so neither the transformed rows nor a packed copy of W1 is written and read again, and a
// launch goes away.  A work-group makes 16 R scenarios x 16 R units on 16 x 16 instructions; its eight wavefronts share the
// summed index in steps of 64 bytes of a row of W1, each transforms just the values that its steps need (every column tile anew:
// cheap while there are few scenarios), the loads of two steps together and the next two under them.  Bound by latency: the
// arguments, one round trip for statistics and weights, the logarithms, the partial tiles.
// One scenario of 388 columns, 1024 units, bf16: 5.1 us where the two launches take 3.3 + 3.0 - 4.2 (the call 25.4 -> 23.1 us); on
// 32 x 32 tiles of 32 x 32 instructions 6.4, with half the work-groups and 32-byte pieces of W1's rows.
struct TermArgs { const float *b1; float *a_term; uint32_t magic_k; int32_t n_tiles, hw_log; };

template <typename T, int R>
__global__ __launch_bounds__(512) void scenario_term_kernel(const EncodeArgs a, const TermArgs q, const PrepArgs p, const GridRowsArgs r,
                                                            unsigned term_blocks, unsigned grid_from, const PartsOf<T> parts)
{
    constexpr int ES = sizeof(T), E = 16 / ES, KS = 4 * E, U = 2, EDGE = 16 * R;
    __shared__ __attribute__((aligned(16))) float part[8][R * R * 256];
    __shared__ f32x4 tab[AB_MAX_STATS + AB_MAX_SCALARS];     // statistics first, then the scalars
    if (blockIdx.x >= grid_from) {
        if (!parts_block<512>(parts)) grid_rows_item(r, (int64_t)(blockIdx.x - grid_from) * 512 + threadIdx.x);
        return;
    }
    if (blockIdx.x >= term_blocks) { prep_layer1_item<T>(p, (int64_t)(blockIdx.x - term_blocks) * 512 + threadIdx.x); return; }
    const int t = threadIdx.x, lane = t & 63, l15 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int tn = (int)(blockIdx.x % (unsigned)q.n_tiles);
    const int64_t m0 = (int64_t)(blockIdx.x / (unsigned)q.n_tiles) * EDGE;
    const int n0 = tn * EDGE, Fs = a.n_stat + a.n_scal;
    const float *dyn[R], *scal[R];
    const T *w_row[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t row = min(m0 + 16 * i + l15, a.S - 1);
        dyn[i] = a.dyn + row * a.n_stat;
        scal[i] = a.scal + row * a.n_scal;
        w_row[i] = (const T *)p.W1 + (int64_t)(n0 + 16 * i + l15) * p.F;
    }

    // A step: columns step * KS + g * E .. + E - 1 of this lane's scenarios and units.  The first `full` steps hold statistics only;
    // the few behind them (the last statistics, the scalars) go to one wavefront each and are taken value by value.
    auto pack = [](const float (&v)[E]) {
        if constexpr (ES == 2) return i32x4{(int)pack_bf16x2(v[0], v[1]), (int)pack_bf16x2(v[2], v[3]), (int)pack_bf16x2(v[4], v[5]), (int)pack_bf16x2(v[6], v[7])};
        else return __builtin_bit_cast(i32x4, f32x4{v[0], v[1], v[2], v[3]});
    };
    const int full = a.n_stat / KS, tail = full + 7 - wave, jt = tail * KS + g * E;
    const bool has_tail = tail * KS < Fs;
    // Rows of an odd number of bf16 columns: every other one begins in the middle of a word; the words around are taken and shifted.
    const bool odd = ES == 2 && (p.F & 1);
    float x[2][U][R][E];
    i32x4 w[2][U][R];
    int w5[2][U][R];
    auto request = [&](int set, int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(s0 + 8 * u, full - 1) * KS + g * E;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const unsigned char *word = (const unsigned char *)((uintptr_t)(w_row[i] + j) & ~(uintptr_t)3);
                w[set][u][i] = *(const i32x4_any *)word;
                if (odd) w5[set][u][i] = *(const int *)(word + 16);
#pragma unroll
                for (int h = 0; h < E / 4; ++h) {
                    const f32x4 v = *(const f32x4_any *)(dyn[i] + j + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[set][u][i][4 * h + e] = v[e];
                }
            }
        }
    };
    if (wave < full) request(0, wave);
    float xt[R][E], wt[R][E];
    if (has_tail) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int c = min(jt + e, Fs - 1);
                xt[i][e] = *(c < a.n_stat ? dyn[i] + c : scal[i] + (c - a.n_stat));
                wt[i][e] = load_as_f32<T>(w_row[i], c);
            }
    }
    if (t < AB_MAX_STATS + AB_MAX_SCALARS) {
        const ab_enc *e = t < AB_MAX_STATS ? &a.enc_stat[t] : &a.enc_scal[t - AB_MAX_STATS];
        tab[t] = f32x4{e->kind == AB_ENC_LOG ? 1.f : 0.f, e->shift, e->scale, 0.f};
    }
    __syncthreads();
    f32x4 acc[R][R];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const i32x4 (&fx)[R], const i32x4 (&fw)[R]) {                 // scenarios first: they end up in the registers
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if constexpr (ES == 2) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fx[i]), __builtin_bit_cast(bf16x8, fw[j]), acc[i][j], 0, 0, 0);
                } else {
                    const f32x4 u = __builtin_bit_cast(f32x4, fx[i]), v = __builtin_bit_cast(f32x4, fw[j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e], v[e], acc[i][j], 0, 0, 0);
                }
            }
    };
    auto run = [&](auto log_tag) {
        auto phi_of = [&](float v, const f32x4 &c) {
            float lg;
            if constexpr (decltype(log_tag)::value) lg = __builtin_amdgcn_logf(v) * 0.69314718056f;
            else lg = logf(v);
            return ((c.x != 0.f ? lg : v) - c.y) * c.z;
        };
        auto take = [&](int set, int s0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s0 + 8 * u >= full) break;
                const int j = (s0 + 8 * u) * KS + g * E;
                int k = q.magic_k ? j - (int)__umulhi((uint32_t)j, q.magic_k) * a.n_stats_per_layer : 0;     // j mod the statistics of a layer
                float v[R][E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const f32x4 c = tab[k];
#pragma unroll
                    for (int i = 0; i < R; ++i) v[i][e] = phi_of(x[set][u][i][e], c);
                    k = k + 1 == a.n_stats_per_layer ? 0 : k + 1;
                }
                i32x4 fx[R], fw[R];
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    fx[i] = pack(v[i]);
                    fw[i] = w[set][u][i];
                    if (odd && ((uintptr_t)w_row[i] & 2)) {
                        const uint32_t word[5] = {(uint32_t)fw[i].x, (uint32_t)fw[i].y, (uint32_t)fw[i].z, (uint32_t)fw[i].w, (uint32_t)w5[set][u][i]};
#pragma unroll
                        for (int h = 0; h < 4; ++h) fw[i][h] = (int)(word[h] >> 16 | word[h + 1] << 16);
                    }
                }
                mma(fx, fw);
            }
        };
        for (int s0 = wave; s0 < full; s0 += 16 * U) {
            if (s0 + 8 * U < full) request(1, s0 + 8 * U);
            take(0, s0);
            if (s0 + 16 * U < full) request(0, s0 + 16 * U);
            take(1, s0 + 8 * U);
        }
        if (has_tail) {
            i32x4 fx[R], fw[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float v[E], wv[E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = min(jt + e, Fs - 1);
                    const int k = c < a.n_stat ? (q.magic_k ? c - (int)__umulhi((uint32_t)c, q.magic_k) * a.n_stats_per_layer : 0)
                                               : AB_MAX_STATS + c - a.n_stat;
                    v[e] = jt + e < Fs ? phi_of(xt[i][e], tab[k]) : 0.f;
                    wv[e] = jt + e < Fs ? wt[i][e] : 0.f;
                }
                fx[i] = pack(v);
                fw[i] = pack(wv);
            }
            mma(fx, fw);
        }
    };
    if (ES == 2 && q.hw_log) run(std::true_type{});
    else                     run(std::false_type{});
    // the eight partial tiles
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave][(16 * i + 4 * g + e) * EDGE + 16 * j + l15] = acc[i][j][e];
    __syncthreads();
    for (int e = t; e < EDGE * EDGE; e += 512) {
        const int64_t row = m0 + e / EDGE;
        const int col = n0 + e % EDGE;
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) v += part[k][e];
        if (row < a.S) q.a_term[row * p.H1 + col] = v + q.b1[col];
    }
}

hipError_t launch_grid_rows(const ab_model_desc *d, const float *part, const float *cred, int P, int Q,
                            float *xp_row, float *xc_row, int64_t rows, hipStream_t st)
{
    if (rows == 0) return hipSuccess;
    GridRowsArgs a{part, cred, P, Q, d->enc_partition, d->enc_credit, xp_row, xc_row, rows};
    grid_rows_kernel<<<(unsigned)((rows + 255) / 256), 256, 0, st>>>(a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The predicted speed vector V of the chosen candidate (Table 1: V has one entry per worker; Eq. 1 returns V).
// Scoring ranks candidates by the mean of V through a folded output unit; for the one chosen candidate per
// scenario the hidden chain is run once more (one row per scenario) and the output layer applied unit by unit.
// ------------------------------------------------------------------------------------------------
// The chosen candidate's transformed pair (phi(S_p), phi(S_c)) per scenario; NaN where nothing was chosen.
__device__ __forceinline__ void chosen_pair(const ChosenArgs &a, int64_t s, int c)
{
    float xp = __builtin_nanf(""), xc = __builtin_nanf("");
    if (c >= 0 && c < a.P * a.Q) {
        const int p = c / a.Q, q = c - p * a.Q;
        xp = phi(a.part[(a.per_scenario ? s * a.P : 0) + p], a.enc_part);
        xc = phi(a.cred[(a.per_scenario ? s * a.Q : 0) + q], a.enc_cred);
    }
    a.xp_sel[s] = xp;
    a.xc_sel[s] = xc;
}
__global__ __launch_bounds__(256) void chosen_pair_kernel(const ChosenArgs a, const int32_t *best_idx, int64_t S)
{
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s < S) chosen_pair(a, s, best_idx[s]);
}

hipError_t launch_chosen_pair(const ChosenArgs &a, const int32_t *best_idx, int64_t S, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    chosen_pair_kernel<<<(unsigned)((S + 255) / 256), 256, 0, st>>>(a, best_idx, S);
    return hipGetLastError();
}

// V[s, o] = b[o] + sum_j W[o, j] * h[s, j]: a wavefront per scenario, lanes over j, up to AB_MAX_OUTPUTS sums.
// h is the last hidden activation in fp32 (h_last), or, for a scorer with one hidden layer, generated here as
// relu(a_term[s, j] + wp[j] * xp[s] + wc[j] * xc[s]).  A scenario without a choice (best_idx < 0) gets NaN.
struct OutputVArgs { const float *h_last; const float *a_term, *wp, *wc, *xp_sel, *xc_sel;
                     const void *W; const float *b; int32_t H, n_out; const int32_t *best_idx; float *V; int64_t S; };
template <typename T>
__global__ __launch_bounds__(256) void output_v_kernel(const OutputVArgs a)
{
    touch_arguments<sizeof(OutputVArgs)>();
    const int lane = threadIdx.x & 63;
    const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (s >= a.S) return;
    float acc[AB_MAX_OUTPUTS];
#pragma unroll
    for (int o = 0; o < AB_MAX_OUTPUTS; ++o) acc[o] = 0.f;
    const float xp = a.h_last ? 0.f : a.xp_sel[s], xc = a.h_last ? 0.f : a.xc_sel[s];
    // a lane takes eight adjacent units; everything it reads of eight outputs is requested before the first product
    // (one round trip per 512 units; V of 300 scenarios, 512 units, 8 outputs: 4.6 us a launch, 12.1 with a unit a lane and step)
    for (int j = lane * 8; j < a.H; j += 512) {
        float h[8];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            f32x4 v;
            if (a.h_last) v = *(const f32x4 *)(a.h_last + s * a.H + j + 4 * q);
            else {                                           // (the last hidden activation stays fp32 in the scoring pass too)
                const f32x4 at = *(const f32x4 *)(a.a_term + s * a.H + j + 4 * q);
                const f32x4 wp = *(const f32x4 *)(a.wp + j + 4 * q), wc = *(const f32x4 *)(a.wc + j + 4 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = relu_keep_nan(fmaf(wc[e], xc, fmaf(wp[e], xp, at[e])));
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) h[4 * q + e] = v[e];
        }
#pragma unroll
        for (int o0 = 0; o0 < AB_MAX_OUTPUTS; o0 += 8) {
            if (o0 >= a.n_out) break;
            i32x4 w[8][sizeof(T) / 2];
#pragma unroll
            for (int o = 0; o < 8; ++o)
#pragma unroll
                for (int q = 0; q < (int)sizeof(T) / 2; ++q)
                    w[o][q] = *(const i32x4 *)((const T *)a.W + (int64_t)min(o0 + o, a.n_out - 1) * a.H + j + 4 * q);
#pragma unroll
            for (int o = 0; o < 8; ++o)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float x;
                    if constexpr (sizeof(T) == 2) x = __uint_as_float(e & 1 ? (uint32_t)w[o][0][e >> 1] & 0xffff0000u : (uint32_t)w[o][0][e >> 1] << 16);
                    else x = __uint_as_float((uint32_t)w[o][e >> 2][e & 3]);
                    acc[o0 + o] = fmaf(x, h[e], acc[o0 + o]);
                }
        }
    }
    const bool none = a.best_idx[s] < 0;
#pragma unroll
    for (int o = 0; o < AB_MAX_OUTPUTS; ++o) {
        if (o < a.n_out) {
            const float v = wave_sum(acc[o]) + a.b[o];
            if (lane == 0) a.V[s * a.n_out + o] = none ? __builtin_nanf("") : v;
        }
    }
}

hipError_t launch_output_v(int dtype, const float *h_last, const float *a_term, const float *wp, const float *wc,
                           const float *xp_sel, const float *xc_sel, const void *W, const float *b, int H, int n_out,
                           const int32_t *best_idx, float *V, int64_t S, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    OutputVArgs a{h_last, a_term, wp, wc, xp_sel, xc_sel, W, b, H, n_out, best_idx, V, S};
    const unsigned blocks = (unsigned)((S + 3) / 4);
    if (dtype == AB_BF16) output_v_kernel<bf16_t><<<blocks, 256, 0, st>>>(a);
    else                  output_v_kernel<float><<<blocks, 256, 0, st>>>(a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Argmax helpers: (value, index) pairs, larger value wins, lower index wins ties, NaN never wins.
// "Nothing yet" is (-inf, INT_MAX).
// ------------------------------------------------------------------------------------------------
#define AB_NONE 0x7fffffff
__device__ __forceinline__ void amax_take(float &bv, int &bi, float v, int i)
{
    if (!(v != v) && (v > bv || (v == bv && i < bi))) { bv = v; bi = i; }
}
// Over the 64 lanes of a wavefront, result in every lane: the exchanges of wave_sum (no LDS round trips); a lane
// that an exchange does not reach takes "nothing yet", which changes nothing.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ void amax_dpp(float &bv, int &bi)
{
    const float ov = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp((int)0xff800000u, __builtin_bit_cast(int, bv),
                                                                           CTRL, ROW_MASK, 0xF, false));
    const int oi = __builtin_amdgcn_update_dpp(AB_NONE, bi, CTRL, ROW_MASK, 0xF, false);
    amax_take(bv, bi, ov, oi);
}
__device__ __forceinline__ void amax_wave(float &bv, int &bi)
{
    amax_dpp<0xB1>(bv, bi);
    amax_dpp<0x4E>(bv, bi);
    amax_dpp<0x141>(bv, bi);
    amax_dpp<0x140>(bv, bi);
    amax_dpp<0x142, 0xA>(bv, bi);    // row_bcast:15
    amax_dpp<0x143, 0xC>(bv, bi);    // row_bcast:31
    bv = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, bv), 63));
    bi = __builtin_amdgcn_readlane(bi, 63);
}

// One work-group per scenario.  score[c] = b_out + sum_t partial[(row0 + c)*nt + t]  (nt = 1 and
// b_out = 0 turn this into a plain argmax over stored scores with a row stride).
struct FinishArgs {
    const float *partial; int32_t nt; int64_t row_stride;   // elements between scenarios in `partial` (per nt)
    const float *b_out;                                      // one fp32 or NULL
    float *scores; int64_t score_stride;                     // NULL: do not store
    int32_t *best_idx; float *best_score;                    // may be NULL
    int32_t C;
    ChosenArgs chosen;                                       // xp_sel: also the chosen candidate's pair
};

// EIGHTS: nt is a multiple of eight, `partial` 16-byte aligned.  PAIR: the chosen candidate's pair as well (its arguments and
// registers cost a plain argmax of 36560 rows of 1476 columns 1.5 of 58.7 us).
template <bool EIGHTS, bool PAIR>
__global__ __launch_bounds__(256) void finish_select_kernel(const FinishArgs a)
{
    touch_arguments<sizeof(FinishArgs)>();
    const int64_t s = blockIdx.x;
    const float *p = a.partial + s * a.row_stride * a.nt;
    const float b = a.b_out ? a.b_out[0] : 0.f;
    float bv = -INFINITY;
    int bi = AB_NONE;
    for (int c0 = threadIdx.x; c0 < a.C; c0 += 1024) {      // four candidates per thread at a time, loads together
        float v[4];
        if constexpr (EIGHTS) {                              // eight per round trip
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = 0.f;
            for (int t = 0; t < a.nt; t += 8) {
                f32x4 x[4][2];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        x[u][h] = c0 + 256 * u < a.C ? *(const f32x4 *)(p + (int64_t)(c0 + 256 * u) * a.nt + t + 4 * h) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) v[u] += (x[u][h][0] + x[u][h][1]) + (x[u][h][2] + x[u][h][3]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + 256 * u;
                v[u] = c < a.C ? p[(int64_t)c * a.nt] : 0.f;
            }
            for (int t = 1; t < a.nt; ++t) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + 256 * u;
                    if (c < a.C) v[u] += p[(int64_t)c * a.nt + t];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + 256 * u;
            if (c < a.C) {
                const float x = v[u] + b;
                if (a.scores) a.scores[s * a.score_stride + c] = x;
                amax_take(bv, bi, x, c);
            }
        }
    }
    if (!a.best_idx) return;
    amax_wave(bv, bi);
    __shared__ float sv[4];
    __shared__ int si[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) amax_take(bv, bi, sv[w], si[w]);
        a.best_idx[s] = (bi == AB_NONE) ? -1 : bi;
        if (a.best_score) a.best_score[s] = (bi == AB_NONE) ? __uint_as_float(0x7fc00000u) : bv;
        if constexpr (PAIR) chosen_pair(a.chosen, s, (bi == AB_NONE) ? -1 : bi);
    }
}

// The same for short rows (C <= 1024): a wavefront per scenario, four scenarios per work-group, no LDS
// and no barrier.  NT fixes the number of partial sums per candidate (one 4*NT-byte load each).
template <int NT>
__global__ __launch_bounds__(256) void finish_select_wave_kernel(const FinishArgs a, int64_t S)
{
    touch_arguments<sizeof(FinishArgs)>();
    const int lane = threadIdx.x & 63;
    const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (s >= S) return;
    const float *p = a.partial + s * a.row_stride * NT;
    const float b = a.b_out ? a.b_out[0] : 0.f;
    float bv = -INFINITY;
    int bi = AB_NONE;
    {
        // four candidates of this lane at a time, their loads issued together
        typedef __attribute__((ext_vector_type(NT))) float vec_t;
        for (int c0 = lane; c0 < a.C; c0 += 256) {
            vec_t x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + 64 * u;
                if (c < a.C) {
                    if constexpr (NT == 1) x[u] = vec_t(__builtin_nontemporal_load(p + c));
                    else x[u] = __builtin_nontemporal_load((const vec_t *)(p + (int64_t)c * NT));
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + 64 * u;
                if (c < a.C) {
                    float v = x[u][0];
#pragma unroll
                    for (int t = 1; t < NT; ++t) v += x[u][t];
                    v += b;
                    if (a.scores) a.scores[s * a.score_stride + c] = v;
                    amax_take(bv, bi, v, c);
                }
            }
        }
    }
    if (!a.best_idx) return;
    amax_wave(bv, bi);
    if (lane == 0) {
        a.best_idx[s] = (bi == AB_NONE) ? -1 : bi;
        if (a.best_score) a.best_score[s] = (bi == AB_NONE) ? __uint_as_float(0x7fc00000u) : bv;
        if (a.chosen.xp_sel) chosen_pair(a.chosen, s, (bi == AB_NONE) ? -1 : bi);
    }
}

// Optimization Trigger (Section 3.3): argmax of a stored score row, relative gain over the configuration in
// use, and the two threshold tests; IEEE single precision throughout.
struct TriggerArgs {
    const float *scores; int64_t row_stride; int32_t C;
    const int32_t *cur_idx; const float *observed;
    float gain_threshold, error_threshold;
    int32_t *best_idx; float *gain; uint8_t *reconf; uint8_t *adapt;
};
// (bv, bi) = the row's best, vc = the score in use (NaN where the current index is outside the row)
__device__ __forceinline__ void trigger_write(const TriggerArgs &a, int64_t s, float bv, int bi, float vc, bool cur_ok, float obs)
{
    const bool has_best = bi != AB_NONE;
    a.best_idx[s] = has_best ? bi : -1;
    const float nan = __uint_as_float(0x7fc00000u);
    const float g = has_best && cur_ok ? (bv - vc) / fabsf(vc) : nan;
    if (a.gain) a.gain[s] = g;
    a.reconf[s] = (uint8_t)(g >= a.gain_threshold);
    if (a.adapt) {
        const float e = a.observed && cur_ok ? fabsf(vc - obs) / fabsf(obs) : nan;
        a.adapt[s] = (uint8_t)(e > a.error_threshold);
    }
}

// Decision on stored rows of at most 1024 columns: the plain argmax (FinishArgs) or the trigger (TriggerArgs).
// Bound by reading the rows once, so LANES lanes take a row and issue all of their loads before they look at the first
// value; the lanes of a row combine through DPP exchanges (no LDS, no barrier).  VEC: rows are 16-byte aligned and a multiple of
// four columns, a lane loads 16 bytes at a time; otherwise 4 bytes (adjacent lanes still read adjacent columns).  What the
// trigger reads besides the row (index in use, its score, the observed speed) is asked for in front of the row and hides behind it.
template <int LANES, int NLOAD, bool VEC, typename Args>
__global__ __launch_bounds__(256) void decide_rows_kernel(const Args a, int64_t S)
{
    constexpr bool TRIGGER = std::is_same<Args, TriggerArgs>::value;
    constexpr int ROWS = 256 / LANES;
    const int l = threadIdx.x & (LANES - 1);
    const int64_t s = (int64_t)blockIdx.x * ROWS + threadIdx.x / LANES;
    const bool live = s < S;
    const int64_t sr = live ? s : 0;
    const float *p;
    int ci = 0;
    float obs = 0.f;
    if constexpr (TRIGGER) {
        p = a.scores + sr * a.row_stride;
        ci = a.cur_idx[sr];
        if (a.observed) obs = a.observed[sr];
    } else {
        p = a.partial + sr * a.row_stride;
    }
    f32x4 x[NLOAD];
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        if constexpr (VEC) {
            const int c = (i * LANES + l) * 4;
            x[i] = (live && c < a.C) ? __builtin_nontemporal_load((const f32x4 *)(p + c))
                                     : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = (i * 4 + e) * LANES + l;
                x[i][e] = (live && c < a.C) ? __builtin_nontemporal_load(p + c) : -INFINITY;
            }
        }
    }
    bool cur_ok = false;
    float vc = __uint_as_float(0x7fc00000u);
    if constexpr (TRIGGER) {
        cur_ok = ci >= 0 && ci < a.C;
        if (cur_ok) vc = p[ci];
    }
    float bv = -INFINITY;
    int bi = AB_NONE;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = VEC ? (i * LANES + l) * 4 + e : (i * 4 + e) * LANES + l;
            if (c < a.C) amax_take(bv, bi, x[i][e], c);
        }
    }
    if constexpr (LANES == 64) {
        amax_wave(bv, bi);
    } else {
        amax_dpp<0xB1>(bv, bi);      // lanes ^ 1   (quad_perm 1,0,3,2)
        amax_dpp<0x4E>(bv, bi);      // lanes ^ 2   (quad_perm 2,3,0,1)
        amax_dpp<0x141>(bv, bi);     // the other quad of the half row (row_half_mirror)
        amax_dpp<0x140>(bv, bi);     // the other half of the row (row_mirror)
    }
    if (live && l == 0) {
        if constexpr (TRIGGER) {
            trigger_write(a, s, bv, bi, vc, cur_ok, obs);
        } else {
            a.best_idx[s] = (bi == AB_NONE) ? -1 : bi;
            if (a.best_score) a.best_score[s] = (bi == AB_NONE) ? __uint_as_float(0x7fc00000u) : bv;
        }
    }
}

// Lanes a row: sixteen (four rows a wavefront, fewer exchanges) where the rows fill the chip anyway, 64 (a quarter of the loads
// in a lane's chain) where a row is long or the rows are few.  Measured, 16 against 64 lanes, us a launch, aligned rows:
// 256 columns: 1 row 3.7 / 3.4, 4096 rows 4.2 / 4.2, 8192 rows 4.5 / 5.1, 65536 rows 13.0 / 23.0; 512 columns: 1 row 4.7 / 3.6,
// 8192 rows 6.2 / 5.8, 16384 rows 8.3 / 9.1, 65536 rows 22.2 / 29.6; 1024 columns: 1 row 7.6 / 3.8, 65536 rows 49.7 / 46.3.  4-byte loads, 65536
// rows: 257 columns 20.6 / 26.1, 512 columns 34.8 / 31.8.  (A work-group a row: 1024 columns 3.9 us at 1 row, 96.7 at 65536.)
int decide_lanes(int64_t S, int C, bool vec)
{
    if (C <= 128) return 16;
    if (C <= 256) return S > 4096 ? 16 : 64;
    return C <= (vec ? 512 : 320) && S > 8192 ? 16 : 64;
}

template <typename Args>
static void launch_decide_rows(const Args &a, const float *rows, int64_t row_stride, int64_t S, hipStream_t st)
{
    const bool vec = a.C % 4 == 0 && row_stride % 4 == 0 && ((uintptr_t)rows & 15) == 0;
    const int lanes = decide_lanes(S, a.C, vec);
    const unsigned blocks = (unsigned)((S + 256 / lanes - 1) / (256 / lanes));
    auto go = [&](auto l, auto n) {
        constexpr int L = decltype(l)::value, N = decltype(n)::value;
        if (vec) decide_rows_kernel<L, N, true, Args><<<blocks, 256, 0, st>>>(a, S);
        else     decide_rows_kernel<L, N, false, Args><<<blocks, 256, 0, st>>>(a, S);
    };
    constexpr std::integral_constant<int, 16> l16{};
    constexpr std::integral_constant<int, 64> l64{};
    if (lanes == 16) {
        if (a.C <= 64) go(l16, std::integral_constant<int, 1>{});
        else if (a.C <= 128) go(l16, std::integral_constant<int, 2>{});
        else if (a.C <= 256) go(l16, std::integral_constant<int, 4>{});
        else go(l16, std::integral_constant<int, 8>{});
    } else {
        if (a.C <= 256) go(l64, std::integral_constant<int, 1>{});
        else if (a.C <= 512) go(l64, std::integral_constant<int, 2>{});
        else if (a.C <= 768) go(l64, std::integral_constant<int, 3>{});
        else go(l64, std::integral_constant<int, 4>{});
    }
}

// ------------------------------------------------------------------------------------------------
// The whole pass in one launch for the size the paper runs it at (one job, tens of candidates, a small
// scorer; Section 3.3 "Meta network optimizer"): at that size the chain of launches of the batched path
// costs more than the arithmetic.  One work-group per scenario:
//   transformed features -> LDS; scenario term A[j] = W1[j, :Fs] x + b1[j] (a wavefront per output,
//   lanes over the inputs); then 64 candidates at a time, a candidate per lane and a sixteenth of a layer's
//   outputs per wavefront: h1 = relu(A + wp phi(S_p) + wc phi(S_c)), the further layers as dot products
//   whose weights are staged in LDS (wave-uniform broadcast reads) against the candidate's activations
//   (read once per layer into registers from LDS rows of stride H + 4 floats: no bank conflicts), the output unit, and
//   the running argmax.  With bf16 as compute type the values the batched path keeps in memory in bf16 (the
//   scenario's features, every hidden activation but the last layer's) are rounded to bf16 here too, so a
//   model scores the same whichever path a call takes.
// ------------------------------------------------------------------------------------------------
struct TinyArgs {
    const float *dyn, *scal, *part, *cred;
    int32_t part_stride, cred_stride;            // elements between two scenarios' grids (0: one shared grid)
    int32_t L, K, Ns, Q, C, F, Fs, D;
    int32_t H[AB_MAX_HIDDEN];
    const void *W[AB_MAX_HIDDEN + 1];
    const float *b[AB_MAX_HIDDEN + 1];
    ab_enc enc_stat[AB_MAX_STATS], enc_scalar[AB_MAX_SCALARS], enc_part, enc_cred;
    float *scores; int32_t *best_idx; float *best_score;
};

template <typename T>
__device__ __forceinline__ float as_stored(float v)        // what a value becomes when kept in the compute type
{
    if constexpr (sizeof(T) == 2) return bf16_bits_to_f32(pack_bf16x2(v, 0.f) & 0xffffu);
    else return v;
}

// One work-group = one scenario = one CU, so the kernel is a chain of short stages and its time is the sum of
// their latencies.  What does not depend on an earlier stage is done at the start (transformed grid values,
// hidden biases and the output unit -> LDS, each by a thread of its own instead of once per wavefront), and
// the hidden layers run on the matrix cores in fp32: 16 x 16 output blocks (outputs x candidates), one or two
// per wavefront, operands read from LDS as 16-byte pieces with one K order for both sides (piece q of a lane
// holds k = 16q + 4 (lane / 16) + e for the e-th instruction of the piece).
template <typename T>
__global__ __launch_bounds__(1024) void score_tiny_kernel(const TinyArgs a)
{
    constexpr int HM = 128, G = 64, STR = HM + 4, FS_MAX = 2048, NW = 16, CM = 256;   // sixteen wavefronts
    __shared__ float xs[FS_MAX];
    __shared__ float A1[HM], wp[HM], wc[HM];
    __shared__ __attribute__((aligned(16))) float b_s[AB_MAX_HIDDEN - 1][HM];   // biases of the hidden layers after the first
    __shared__ float wo_s[HM + 1];                                        // output unit: weights, then its bias
    __shared__ float xp_s[CM], xc_s[CM];                                  // transformed grid values per candidate
    __shared__ float red[NW][G];
    extern __shared__ __attribute__((aligned(16))) float tiny_dyn[];      // two activation buffers, one weight matrix
    float (*hb)[G * STR] = (float (*)[G * STR])tiny_dyn;
    float *w_lds = tiny_dyn + 2 * G * STR;                                // rows of hin + 4 floats
    const int64_t s = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int hl = a.H[a.D - 1];

    auto load_w4 = [&](const void *W, int e) {                 // four adjacent weights as fp32
        if constexpr (sizeof(T) == 2) {
            const uint2 r = *(const uint2 *)((const uint16_t *)W + e);
            return f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                         __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
        } else {
            return *(const f32x4 *)((const float *)W + e);
        }
    };
    auto park_w4 = [&](int hin, int e, f32x4 w) {              // ... to their place in the padded LDS rows
        const int j = hin == 64 ? e >> 6 : e >> 7;
        *(f32x4 *)(w_lds + j * (hin + 4) + (e & (hin - 1))) = w;
    };

    // transformed statistics and scalars of the scenario (threads from the front), everything else that only
    // depends on the arguments (threads from the back); the raw statistics are requested first, the second
    // layer's weights and this wavefront's first layer-1 rows right behind them
    const int n_stat = a.L * a.K;
    const int H1 = a.H[0];
    const bool first_x = t < a.Fs;
    float raw0 = 0.f;
    if (first_x) raw0 = t < n_stat ? a.dyn[s * n_stat + t] : a.scal[s * a.Ns + (t - n_stat)];
    const int n_w1 = a.D > 1 ? a.H[1] * H1 : 0;
    f32x4 w_pre[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (t * 4 + u * 4096 < n_w1) w_pre[u] = load_w4(a.W[1], t * 4 + u * 4096);
    float w0_pre[4] = {0.f, 0.f, 0.f, 0.f};
    if (wave * 4 < H1 && lane < a.Fs) {
#pragma unroll
        for (int u = 0; u < 4; ++u) w0_pre[u] = load_as_f32<T>(a.W[0], (int64_t)(wave * 4 + u) * a.F + lane);
    }
    if (first_x) xs[t] = as_stored<T>(phi(raw0, t < n_stat ? a.enc_stat[t % a.K] : a.enc_scalar[t - n_stat]));
    for (int i = t + 64 * NW; i < a.Fs; i += 64 * NW)
        xs[i] = as_stored<T>(i < n_stat ? phi(a.dyn[s * n_stat + i], a.enc_stat[i % a.K])
                                        : phi(a.scal[s * a.Ns + (i - n_stat)], a.enc_scalar[i - n_stat]));
    {
        const int r = 64 * NW - 1 - t;
        if (r < a.C) xp_s[r] = phi(a.part[(int64_t)blockIdx.x * a.part_stride + r / a.Q], a.enc_part);
        else if (r >= CM && r - CM < a.C) xc_s[r - CM] = phi(a.cred[(int64_t)blockIdx.x * a.cred_stride + (r - CM) % a.Q], a.enc_cred);
        else if (r >= 2 * CM && r - 2 * CM <= hl)
            wo_s[r - 2 * CM] = r - 2 * CM < hl ? load_as_f32<T>(a.W[a.D], r - 2 * CM) : a.b[a.D][0];
        for (int q = t; q < (a.D - 1) * HM; q += 64 * NW) {
            const int k = 1 + q / HM, jx = q % HM;
            if (jx < a.H[k]) b_s[k - 1][jx] = a.b[k][jx];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (t * 4 + u * 4096 < n_w1) park_w4(H1, t * 4 + u * 4096, w_pre[u]);
    __syncthreads();
    // scenario term of layer 1 and its two configuration columns
    for (int j0 = wave * 4; j0 < H1; j0 += 4 * NW) {           // four outputs at a time: four loads in flight
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        int i_from = lane;
        if (j0 == wave * 4 && lane < a.Fs) {                    // (the piece requested at the start)
            const float x = xs[lane];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = w0_pre[u] * x;
            i_from = lane + 64;
        }
        for (int i = i_from; i < a.Fs; i += 64) {
            const float x = xs[i];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = fmaf(load_as_f32<T>(a.W[0], (int64_t)(j0 + u) * a.F + i), x, acc[u]);
        }
        float mine = 0.f, mp = 0.f, mc = 0.f;                  // (requested before the sums are formed)
        if (lane < 4) {
            const int j = j0 + lane;
            mine = a.b[0][j];
            mp = load_as_f32<T>(a.W[0], (int64_t)j * a.F + a.Fs);
            mc = load_as_f32<T>(a.W[0], (int64_t)j * a.F + a.Fs + 1);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = wave_sum(acc[u]);
        if (lane < 4) {
            const int j = j0 + lane;
            const float av = lane == 0 ? acc[0] : lane == 1 ? acc[1] : lane == 2 ? acc[2] : acc[3];
            A1[j] = av + mine;
            wp[j] = mp;
            wc[j] = mc;
        }
    }
    __syncthreads();

    float bv = -INFINITY;
    int bi = AB_NONE;
    for (int c0 = 0; c0 < a.C; c0 += G) {
        const int c = c0 + lane;
        const int cc = c < a.C ? c : a.C - 1;
        const float xp = xp_s[cc], xc = xc_s[cc];
        {
            float *mine = &hb[0][lane * STR];
            const int hq = H1 / NW;
            for (int jj = 0; jj < hq; ++jj) {
                const int j = wave * hq + jj;
                const float h = relu_keep_nan(fmaf(wc[j], xc, fmaf(wp[j], xp, A1[j])));
                mine[j] = a.D > 1 ? as_stored<T>(h) : h;
            }
        }
        int cur = 0;
        for (int k = 1; k < a.D; ++k) {
            const int hin = a.H[k - 1], hout = a.H[k], ws = hin + 4;
            // the layer's weights -> LDS as fp32, once the layer before has read its own (the last layer of the
            // group before is behind the output unit's barriers); the second layer's are there from the start
            // and, being the only ones, stay for every group of candidates
            if (k > 1) __syncthreads();
            if (!(k == 1 && (c0 == 0 || a.D == 2))) {           // (the second layer's were parked at the start)
                for (int e = t * 4; e < hout * hin; e += 256 * NW) park_w4(hin, e, load_w4(a.W[k], e));
            }
            __syncthreads();                                    // weights and the layer's inputs are in place
            const bool keep = k == a.D - 1;                     // the last hidden layer is not kept in the compute type
            for (int blk = wave; blk < 4 * (hout >> 4); blk += NW) {
                const int cb = blk & 3, ob = blk >> 2;
                const int row = lane & 15, kq = (lane >> 4) * 4;
                const float *pw = w_lds + (16 * ob + row) * ws + kq;
                const float *ph = &hb[cur][(16 * cb + row) * STR + kq];
                f32x4 acc = *(const f32x4 *)&b_s[k - 1][16 * ob + kq];     // lane: outputs 16 ob + kq .. + 3 of candidate 16 cb + row
                for (int q = 0; q < hin; q += 16) {
                    const f32x4 wv = *(const f32x4 *)(pw + q), hv = *(const f32x4 *)(ph + q);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.x, hv.x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.y, hv.y, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.z, hv.z, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.w, hv.w, acc, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = relu_keep_nan(acc[e]);
                    acc[e] = keep ? v : as_stored<T>(v);
                }
                *(f32x4 *)&hb[cur ^ 1][(16 * cb + row) * STR + 16 * ob + kq] = acc;
            }
            cur ^= 1;
        }
        __syncthreads();
        {   // output unit: each wavefront its share of the dot product
            const int hq = hl / NW;
            const float *src = &hb[cur][lane * STR + wave * hq];
            const float *wo = wo_s + wave * hq;
            float acc = 0.f;
            for (int i = 0; i < hq; i += 4) {
                const f32x4 h = *(const f32x4 *)(src + i);
                acc = fmaf(wo[i + 3], h.w, fmaf(wo[i + 2], h.z, fmaf(wo[i + 1], h.y, fmaf(wo[i], h.x, acc))));
            }
            red[wave][lane] = acc;
        }
        __syncthreads();
        if (wave == 0 && c < a.C) {
            float v = wo_s[hl];
#pragma unroll
            for (int w = 0; w < NW; ++w) v += red[w][lane];
            if (a.scores) a.scores[s * a.C + c] = v;
            amax_take(bv, bi, v, c);
        }
        // (the next group's first writes go to hb[0]: its last readers, the first hidden layer's matrix
        // instructions or the output unit, are behind a barrier; red is rewritten two barriers later)
    }
    if (wave == 0 && a.best_idx) {
        amax_wave(bv, bi);
        if (lane == 0) {
            a.best_idx[s] = (bi == AB_NONE) ? -1 : bi;
            if (a.best_score) a.best_score[s] = (bi == AB_NONE) ? __uint_as_float(0x7fc00000u) : bv;
        }
    }
}

// The trigger on rows of more than 1024 columns: one work-group per scenario.
__global__ __launch_bounds__(256) void trigger_kernel(const TriggerArgs a)
{
    const int64_t s = blockIdx.x;
    const float *p = a.scores + s * a.row_stride;
    float bv = -INFINITY;
    int bi = AB_NONE;
    for (int c = threadIdx.x; c < a.C; c += 256) amax_take(bv, bi, p[c], c);
    amax_wave(bv, bi);
    __shared__ float sv[4];
    __shared__ int si[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) amax_take(bv, bi, sv[w], si[w]);
        const int ci = a.cur_idx[s];
        const bool cur_ok = ci >= 0 && ci < a.C;
        trigger_write(a, s, bv, bi, cur_ok ? p[ci] : __uint_as_float(0x7fc00000u), cur_ok, a.observed ? a.observed[s] : 0.f);
    }
}

// Scorer with a single hidden layer: score = w_out . relu(A[s] + B[c]) + b_out, one wavefront per
// (scenario, candidate) row, written into the same partial buffer layout (nt = 1, no bias yet).
struct ScoreD1Args {
    const float *a_term, *b_term, *w_out_f; float *partial; int64_t rows; int32_t C, H;
    const float *wp, *wc, *xp_row, *xc_row;      // xp_row != NULL: B = wp * xp_row[row] + wc * xc_row[row] instead of b_term[c]
};
__global__ __launch_bounds__(256) void score_single_hidden_kernel(const ScoreD1Args a)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.rows) return;
    const int lane = threadIdx.x & 63;
    const int64_t s = row / a.C;
    const int c = (int)(row - s * a.C);
    float acc = 0.f;
    if (a.xp_row) {
        const float xp = a.xp_row[row], xc = a.xc_row[row];
        for (int h = lane; h < a.H; h += 64)
            acc += relu_keep_nan(fmaf(a.wc[h], xc, fmaf(a.wp[h], xp, a.a_term[s * a.H + h]))) * a.w_out_f[h];
    } else {
        for (int h = lane; h < a.H; h += 64)
            acc += relu_keep_nan(a.a_term[s * a.H + h] + a.b_term[(int64_t)c * a.H + h]) * a.w_out_f[h];
    }
    acc = wave_sum(acc);
    if (lane == 0) a.partial[row] = acc;
}

// ------------------------------------------------------------------------------------------------
// Shared per-tensor encoder (Section 3.1 "Meta network architecture": the layer-wise statistics are
// embedded into a fixed-dimension feature space so that models with different layer counts can be
// handled).  A work-group takes scenarios blockIdx.x, blockIdx.x + grid, ... (two work-groups per CU):
//   e[l] = relu(W_b relu(W_a phi(stat[l]) + b_a) + b_b)   (K -> 128 -> 128), pooled[s] = mean_l e[l], written as the
//   first 128 columns of the scenario row.
// The four wavefronts work on their own 32-tensor blocks without meeting, each block's raw statistics fetched while the
// block before is computed; one reduction over the wavefronts at a scenario's end.  Both layers run on the matrix cores
// and the hidden row never leaves the registers: the first layer is taken transposed (32 x 32 x 2 in fp32: rows = units,
// columns = tensors, the bias as initial sums), so a lane ends with units 8 g + 4 half + 0..3 of its tensor, and the
// second product (bf16 operands, fp32 sums) simply numbers its summed index that way: K step q of lane half h is units
// 16 q + 4 h + 0..3 and 16 q + 8 + 4 h + 0..3, which is how W_b's chunks are laid out in LDS (bf16, 32 KB, once per
// work-group; 16-byte chunk c of row r at c ^ (r & 15)).  Bound by the matrix cores (1536 clocks a block: 512 + 1024); with
// the first layer on the vector ALUs (2700 clocks a block there) and its rows through LDS a batch of 8192 scenarios of
// 200 - 400 tensors took 235 us, now 145 - 160 us.
// ------------------------------------------------------------------------------------------------
struct TensorEncArgs {
    const float *dyn; int32_t L, K;
    const void *Wa; const float *ba;     // [128, K]
    const void *Wb; const float *bb;     // [128, 128]
    void *xs; int32_t ld;                // scenario rows; columns [0,128) written here
    const int32_t *layers_of;            // [S] or NULL: layers the scenario really has (clamped to [1, L])
    int64_t S;
    ab_enc enc_stat[AB_MAX_ENCODER_STATS];
};

template <int KS>                                          // KS: pairs of statistics (K <= 2 KS); weights and rows are bf16
__global__ __launch_bounds__(256, 2) void tensor_encoder_kernel(const TensorEncArgs a, const SideArgs side, const unsigned grid)
{
    if (blockIdx.x >= grid) {
        side_block<256>(side, blockIdx.x - grid);
        return;
    }
    constexpr int H = 128;
    __shared__ __attribute__((aligned(16))) unsigned char wb_s[H * 256];
    __shared__ float red[4][H];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, half = lane >> 5, l31 = lane & 31;
    auto layers = [&](int64_t sc) {                        // a scenario's own layer count
        int n = a.L;
        if (a.layers_of) { n = a.layers_of[sc]; n = n < 1 ? 1 : (n > a.L ? a.L : n); }
        return n;
    };

    for (int i = t; i < H * 16; i += 256) {                 // chunk c = 2 q + h of row n
        const int n = i >> 4, c = i & 15, u = (c >> 1) * 16 + (c & 1) * 4;
        const uint2 lo = *(const uint2 *)((const uint16_t *)a.Wb + n * H + u), hi = *(const uint2 *)((const uint16_t *)a.Wb + n * H + u + 8);
        *(i32x4 *)(wb_s + n * 256 + ((c ^ (n & 15)) << 4)) = i32x4{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
    }

    float bb[4], colsum[4] = {0.f, 0.f, 0.f, 0.f}, wa[4][KS];
    f32x16 ba[4];                                          // first layer's bias where its result has the units
#pragma unroll
    for (int jn = 0; jn < 4; ++jn) {
        bb[jn] = a.bb[jn * 32 + l31];
#pragma unroll
        for (int r = 0; r < 16; ++r) ba[jn][r] = a.ba[jn * 32 + (r >> 2) * 8 + half * 4 + (r & 3)];
#pragma unroll
        for (int k = 0; k < KS; ++k) wa[jn][k] = 2 * k + half < a.K ? load_as_f32<bf16_t>(a.Wa, (jn * 32 + l31) * a.K + 2 * k + half) : 0.f;
    }
    __syncthreads();

    // this lane's statistics of a block: 2 k + half of tensor l31
    ab_enc my_enc[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) my_enc[k] = a.enc_stat[2 * k + half];
    auto fetch_raw = [&](int64_t sc, int n_layers, int l0, float (&raw)[KS]) {
        const float *dyn = a.dyn + sc * (int64_t)a.L * a.K;
        const int l = l0 + l31;
#pragma unroll
        for (int k = 0; k < KS; ++k)
            raw[k] = (sc < a.S && l < n_layers && 2 * k + half < a.K) ? dyn[(int64_t)l * a.K + 2 * k + half] : 1.f;
    };

    int64_t sc = blockIdx.x;
    int Ls = sc < a.S ? layers(sc) : 0;
    int l0 = wave * 32;
    float raw[KS];
    fetch_raw(sc, Ls, l0, raw);
    for (; sc < a.S; ) {
      const bool has_block = l0 < Ls;                        // (its last block fetches the next scenario's first)
      for (; l0 < Ls; ) {
        // the block after this one (of this scenario, or the first of this wavefront in the next scenario)
        int64_t sc_n = sc;
        int Ls_n = Ls, l0_n = l0 + 128;
        if (l0_n >= Ls) { sc_n = sc + grid; Ls_n = sc_n < a.S ? layers(sc_n) : 0; l0_n = wave * 32; }
        float raw_n[KS], x[KS];
        fetch_raw(sc_n, Ls_n, l0_n, raw_n);
        // transformed statistics (zero past the end)
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const float lg = __builtin_amdgcn_logf(raw[k]) * 0.69314718056f;
            const float y = ((my_enc[k].kind == AB_ENC_LOG ? lg : raw[k]) - my_enc[k].shift) * my_enc[k].scale;
            x[k] = (l0 + l31 < Ls && 2 * k + half < a.K) ? y : 0.f;
        }
        f32x16 acc[4];
#pragma unroll
        for (int jn = 0; jn < 4; ++jn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[jn][r] = 0.f;
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {                     // 32 hidden units at a time
            asm volatile("" ::: "memory");                   // (W_b's fragments are read here and not kept in registers)
            f32x16 h = ba[jb];
#pragma unroll
            for (int k = 0; k < KS; ++k) h = __builtin_amdgcn_mfma_f32_32x32x2f32(wa[jb][k], x[k], h, 0, 0, 0);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int chunk = (jb * 2 + s) * 2 + half;
                i32x4 fa;
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    fa[p] = (int)pack_bf16x2(relu_keep_nan(h[s * 8 + 2 * p]), relu_keep_nan(h[s * 8 + 2 * p + 1]));
#pragma unroll
                for (int jn = 0; jn < 4; ++jn) {
                    const int n = jn * 32 + l31;
                    const i32x4 fb = *(const i32x4 *)(wb_s + n * 256 + ((chunk ^ (n & 15)) << 4));
                    // rows = tensors (first operand), columns = units (second operand)
                    acc[jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa),
                                                                      __builtin_bit_cast(bf16x8, fb), acc[jn], 0, 0, 0);
                }
            }
        }
        if (l0 + 32 <= Ls) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int jn = 0; jn < 4; ++jn) colsum[jn] += relu_keep_nan(acc[jn][r] + bb[jn]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int l = l0 + (r >> 2) * 8 + half * 4 + (r & 3);
                if (l < Ls) {
#pragma unroll
                    for (int jn = 0; jn < 4; ++jn) colsum[jn] += relu_keep_nan(acc[jn][r] + bb[jn]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < KS; ++k) raw[k] = raw_n[k];
        l0 += 128;
      }
      // the scenario is complete for this wavefront: combine the four wavefronts' column sums
#pragma unroll
      for (int jn = 0; jn < 4; ++jn) {
          const float v = colsum[jn] + __shfl_xor(colsum[jn], 32, 64);
          if (half == 0) red[wave][jn * 32 + l31] = v;
          colsum[jn] = 0.f;
      }
      __syncthreads();
      if (t < H) {
          const float pooled = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) / (float)Ls;
          ((uint16_t *)a.xs)[sc * a.ld + t] = (uint16_t)(pack_bf16x2(pooled, 0.f) & 0xffffu);
      }
      __syncthreads();                                       // `red` may be written again
      sc += grid;
      Ls = sc < a.S ? layers(sc) : 0;
      l0 = wave * 32;
      if (!has_block) fetch_raw(sc, Ls, l0, raw);
    }
}

// ------------------------------------------------------------------------------------------------
// host-side launch wrappers
// ------------------------------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

static void fill_encode_args(EncodeArgs &a, const ab_model_desc *d, const float *dyn, const float *scal,
                             void *xs, int64_t S, int ld, int col0, int with_stats)
{
    a.dyn = dyn; a.scal = scal; a.xs = xs; a.S = S; a.ld = ld; a.col0 = col0;
    a.n_stat = with_stats ? d->n_layers * d->n_stats : 0;
    a.n_stats_per_layer = d->n_stats; a.n_scal = d->n_scalars;
    for (int i = 0; i < AB_MAX_STATS; ++i) a.enc_stat[i] = d->enc_stat[i];
    for (int i = 0; i < AB_MAX_SCALARS; ++i) a.enc_scal[i] = d->enc_scalar[i];
}

// Whether the four-columns-per-thread form of the transform takes this layout; fills its index constants.
static bool quad_split(int dtype, const ab_model_desc *d, const EncodeArgs &a, QuadSplit &g)
{
    const int width = a.ld - a.col0;
    if (!(encode_quad_columns(a.n_stat, width) && a.col0 % 4 == 0 && width / 4 < 65536 && ((uintptr_t)a.dyn & 15) == 0 && ((uintptr_t)a.xs & 15) == 0 &&
          (a.ld * elem_size(dtype)) % 16 == 0))
        return false;
    // magic = floor(2^32 / n) + 1 turns index / n into a multiply-high, exact while index * n < 2^32
    auto magic = [](int n) { return n >= 2 ? (uint32_t)(0x100000000ull / (uint32_t)n) + 1u : 0u; };
    g.q4s = a.n_stat / 4; g.q4t = (width - a.n_stat) / 4;
    g.rpb = width / 4 >= 1792 ? 1 : 1792 / (width / 4);      // seven quads per thread (measured: 1000-2000 quads per
                                                             // work-group are alike, more are slower)
    g.magic_q4s = magic(g.q4s); g.magic_q4t = magic(g.q4t); g.magic_k = magic(d->n_stats);
    return true;
}

hipError_t launch_encode_stats(int dtype, const ab_model_desc *d, const float *dyn, const float *scal,
                               void *xs, int64_t S, int ld, int col0, int with_stats, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    EncodeArgs a;
    fill_encode_args(a, d, dyn, scal, xs, S, ld, col0, with_stats);
    const int width = ld - col0;
    QuadSplit g;
    if (quad_split(dtype, d, a, g)) {
        const unsigned blocks = (unsigned)((S + g.rpb - 1) / g.rpb);
        if (dtype == AB_BF16) encode_stats_quad_kernel<bf16_t><<<blocks, 256, 0, st>>>(a, g);
        else encode_stats_quad_kernel<float><<<blocks, 256, 0, st>>>(a, g);
        return hipGetLastError();
    }
    const int64_t n = S * (width / 2);
    if (dtype == AB_BF16) encode_stats_kernel<bf16_t><<<blocks_for(n), 256, 0, st>>>(a);
    else encode_stats_kernel<float><<<blocks_for(n), 256, 0, st>>>(a);
    return hipGetLastError();
}

static int64_t fill_prep_args(PrepArgs &a, const ab_model_desc *d, const void *W1, const float *b1, int F, int Fs,
                              int H1, int ld, void *w1s, const ab_grid *grid, float *b_term, float *cfg_vec,
                              const void *Wout, const float *b_out, int H_last, float *w_out_f);

hipError_t launch_prep_layer1(int dtype, const ab_model_desc *d, const void *W1, const float *b1, int F, int Fs,
                              int H1, int ld, void *w1s, const ab_grid *grid, float *b_term, float *cfg_vec,
                              const void *Wout, const float *b_out, int H_last, float *w_out_f, SplitWeightsArgs parts, hipStream_t st)
{
    PrepArgs a;
    const int64_t n = fill_prep_args(a, d, W1, b1, F, Fs, H1, ld, w1s, grid, b_term, cfg_vec, Wout, b_out, H_last, w_out_f);
    const int64_t own = (n + 255) / 256, blocks = own + (split_weights_items(parts) + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (dtype == AB_BF16) prep_layer1_kernel<bf16_t><<<(unsigned)blocks, 256, 0, st>>>(a, parts_of<bf16_t>(parts, own));
    else prep_layer1_kernel<float><<<(unsigned)blocks, 256, 0, st>>>(a, parts_of<float>(parts, own));
    return hipGetLastError();
}

// Transform of the flat model's statistics and layer-1 preparation in one launch.  *done = false (and nothing
// launched) when the layout needs the general form of the transform; the caller then makes the two launches.
hipError_t launch_encode_and_prep(int dtype, const ab_model_desc *d, const float *dyn, const float *scal, void *xs,
                                  int64_t S, int ld, const void *W1, const float *b1, int F, int Fs, int H1, void *w1s,
                                  const ab_grid *grid, float *b_term, float *cfg_vec, const void *Wout,
                                  const float *b_out, int H_last, float *w_out_f, float *xp_row, float *xc_row,
                                  SplitWeightsArgs parts, bool *done, hipStream_t st)
{
    *done = false;
    if (S == 0) return hipSuccess;
    EncodeArgs a;
    fill_encode_args(a, d, dyn, scal, xs, S, ld, 0, 1);
    QuadSplit g;
    if (!quad_split(dtype, d, a, g)) return hipSuccess;
    PrepArgs p;
    const int64_t n = fill_prep_args(p, d, W1, b1, F, Fs, H1, ld, w1s, grid, b_term, cfg_vec, Wout, b_out, H_last, w_out_f);
    const int64_t enc_blocks = (S + g.rpb - 1) / g.rpb, prep_blocks = (n + 255) / 256;
    const GridRowsArgs r{grid->partition_bytes, grid->credit_mult, grid->P, grid->Q, d->enc_partition, d->enc_credit, xp_row, xc_row,
                         xp_row ? S * grid->P * grid->Q : 0};
    const int64_t parts_from = enc_blocks + prep_blocks + (r.rows + 255) / 256, blocks = parts_from + (split_weights_items(parts) + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipSuccess;
    *done = true;
    auto launch = [&](auto kern, auto q) { kern<<<(unsigned)blocks, 256, 0, st>>>(a, g, p, r, (unsigned)enc_blocks, (unsigned)(enc_blocks + prep_blocks), q); };
    if (dtype == AB_BF16) launch(encode_and_prep_kernel<bf16_t>, parts_of<bf16_t>(parts, parts_from));
    else                  launch(encode_and_prep_kernel<float>, parts_of<float>(parts, parts_from));
    return hipGetLastError();
}

hipError_t launch_scenario_term(int dtype, const ab_model_desc *d, const float *dyn, const float *scal, int64_t S, const void *W1,
                                const float *b1, int F, int Fs, int H1, int Kp, float *a_term, const ab_grid *grid, float *b_term,
                                float *cfg_vec, const void *Wout, const float *b_out, int H_last, float *w_out_f, float *xp_row,
                                float *xc_row, SplitWeightsArgs parts, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    EncodeArgs a;
    fill_encode_args(a, d, dyn, scal, nullptr, S, Kp, 0, 1);
    QuadSplit g;
    PrepArgs p;
    const int64_t n = fill_prep_args(p, d, W1, b1, F, Fs, H1, Kp, nullptr, grid, b_term, cfg_vec, Wout, b_out, H_last, w_out_f);
    const int edge = S <= 16 || dtype == AB_BF16 ? 16 : 32;
    const TermArgs q{b1, a_term, d->n_stats >= 2 ? (uint32_t)(0x100000000ull / (uint32_t)d->n_stats) + 1u : 0u, H1 / edge,
                     quad_split(dtype, d, a, g)};            // (the transform's two forms take the logarithm differently in bf16)
    const GridRowsArgs r{grid->partition_bytes, grid->credit_mult, grid->P, grid->Q, d->enc_partition, d->enc_credit, xp_row, xc_row,
                         xp_row ? S * grid->P * grid->Q : 0};
    const int64_t term_blocks = (S + edge - 1) / edge * q.n_tiles, grid_from = term_blocks + (n + 511) / 512, parts_from = grid_from + (r.rows + 511) / 512,
                  blocks = parts_from + (split_weights_items(parts) + 511) / 512;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    auto launch = [&](auto kern, auto w) { kern<<<(unsigned)blocks, 512, 0, st>>>(a, q, p, r, (unsigned)term_blocks, (unsigned)grid_from, w); };
    if (dtype == AB_BF16) launch(scenario_term_kernel<bf16_t, 1>, parts_of<bf16_t>(parts, parts_from));
    else if (edge == 16)  launch(scenario_term_kernel<float, 1>, parts_of<float>(parts, parts_from));
    else                  launch(scenario_term_kernel<float, 2>, parts_of<float>(parts, parts_from));
    return hipGetLastError();
}

static int64_t fill_prep_args(PrepArgs &a, const ab_model_desc *d, const void *W1, const float *b1, int F, int Fs,
                              int H1, int ld, void *w1s, const ab_grid *grid, float *b_term, float *cfg_vec,
                              const void *Wout, const float *b_out, int H_last, float *w_out_f)
{
    a.W1 = W1; a.F = F; a.Fs = Fs; a.H1 = H1; a.ld = ld; a.w1s = w1s; a.b1 = b1;
    a.part = grid->partition_bytes; a.cred = grid->credit_mult; a.P = grid->P; a.Q = grid->Q;
    a.enc_part = d->enc_partition; a.enc_cred = d->enc_credit; a.b_term = b_term;
    const int Cn = grid->P * grid->Q;
    a.wp_f = cfg_vec; a.wc_f = cfg_vec + H1; a.xp_f = cfg_vec + 2 * H1; a.xc_f = cfg_vec + 2 * H1 + Cn;
    a.Wout = Wout; a.b_out = b_out; a.H_last = H_last; a.n_out = d->n_outputs > 1 ? d->n_outputs : 1; a.w_out_f = w_out_f;
    return (w1s ? (int64_t)H1 * ld : 0) + (b_term ? (int64_t)Cn * H1 : 0) + H_last + H1 + Cn;
}

hipError_t launch_finish_select(const float *partial, int nt, int64_t row_stride, const float *b_out,
                                float *scores, int64_t score_stride, int32_t *best_idx, float *best_score,
                                int64_t S, int C, const ChosenArgs *chosen, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    FinishArgs a;
    if (chosen) a.chosen = *chosen;
    else memset(&a.chosen, 0, sizeof(a.chosen));
    a.partial = partial; a.nt = nt; a.row_stride = row_stride; a.b_out = b_out; a.scores = scores;
    a.score_stride = score_stride; a.best_idx = best_idx; a.best_score = best_score; a.C = C;
    const unsigned wave_blocks = (unsigned)((S + 3) / 4);
    if (C <= 1024 && nt == 1 && !b_out && !scores && best_idx && !chosen) {
        launch_decide_rows(a, partial, row_stride, S, st);
    } else if (C <= 1024 && nt == 1)
        finish_select_wave_kernel<1><<<wave_blocks, 256, 0, st>>>(a, S);
    else if (C <= 1024 && nt == 2 && ((uintptr_t)partial & 7) == 0)
        finish_select_wave_kernel<2><<<wave_blocks, 256, 0, st>>>(a, S);
    else if (C <= 1024 && nt == 4 && ((uintptr_t)partial & 15) == 0)
        finish_select_wave_kernel<4><<<wave_blocks, 256, 0, st>>>(a, S);
    else {
        const bool eights = nt % 8 == 0 && ((uintptr_t)partial & 15) == 0;
        if (chosen) eights ? finish_select_kernel<true, true><<<(unsigned)S, 256, 0, st>>>(a) : finish_select_kernel<false, true><<<(unsigned)S, 256, 0, st>>>(a);
        else        eights ? finish_select_kernel<true, false><<<(unsigned)S, 256, 0, st>>>(a) : finish_select_kernel<false, false><<<(unsigned)S, 256, 0, st>>>(a);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// A scorer without hidden layers (Section 3.1 leaves the depth open; with none the network is the linear map
// V = W x + b): a candidate's score is  mean_o W[o, :Fs] . x_s + mean_o b[o]  +  wp phi(S_p) + wc phi(S_c),
// wp / wc the means of W's two configuration columns.  One work-group per scenario: its wavefronts share the
// dot product over the transformed statistics (values kept as the compute type keeps them), then every thread
// takes candidates.  With v_out the per-output dot products of the chosen candidate are written as well.
// ------------------------------------------------------------------------------------------------
struct LinearArgs {
    const float *dyn, *scal, *part, *cred; int32_t part_stride, cred_stride;
    int32_t n_stat, K, Ns, Q, C, F, n_out;
    const void *W; const float *b;
    ab_enc enc_stat[AB_MAX_STATS], enc_scalar[AB_MAX_SCALARS], enc_part, enc_cred;
    float *scores; int32_t *best_idx; float *best_score; float *v_best;
};

template <typename T>
__global__ __launch_bounds__(256) void score_linear_kernel(const LinearArgs a)
{
    __shared__ float red[4][AB_MAX_OUTPUTS + 2];
    __shared__ float sv[4];
    __shared__ int si[4];
    const int64_t s = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int Fs = a.n_stat + a.Ns;
    // per output: the dot product over the statistics block and the scalars
    float acc[AB_MAX_OUTPUTS];
#pragma unroll
    for (int o = 0; o < AB_MAX_OUTPUTS; ++o) acc[o] = 0.f;
    for (int j = t; j < Fs; j += 256) {
        float x = j < a.n_stat ? phi(a.dyn[s * a.n_stat + j], a.enc_stat[j % a.K])
                               : phi(a.scal[s * a.Ns + (j - a.n_stat)], a.enc_scalar[j - a.n_stat]);
        x = as_stored<T>(x);
#pragma unroll
        for (int o = 0; o < AB_MAX_OUTPUTS; ++o)
            if (o < a.n_out) acc[o] = fmaf(load_as_f32<T>(a.W, (int64_t)o * a.F + j), x, acc[o]);
    }
#pragma unroll
    for (int o = 0; o < AB_MAX_OUTPUTS; ++o) {
        if (o < a.n_out) {
            const float v = wave_sum(acc[o]);
            if (lane == 0) red[wave][o] = v;
        }
    }
    __syncthreads();
    float a0 = 0.f, wp = 0.f, wc = 0.f;                    // folded over the outputs: mean of the rows, mean of the biases
    for (int o = 0; o < a.n_out; ++o) {
        a0 += ((red[0][o] + red[1][o]) + (red[2][o] + red[3][o])) + a.b[o];
        wp += load_as_f32<T>(a.W, (int64_t)o * a.F + Fs);
        wc += load_as_f32<T>(a.W, (int64_t)o * a.F + Fs + 1);
    }
    const float inv = 1.f / (float)a.n_out;
    a0 *= inv; wp *= inv; wc *= inv;
    const float *part = a.part + s * a.part_stride, *cred = a.cred + s * a.cred_stride;
    float bv = -INFINITY;
    int bi = AB_NONE;
    for (int c = t; c < a.C; c += 256) {
        const float xp = phi(part[c / a.Q], a.enc_part), xc = phi(cred[c % a.Q], a.enc_cred);
        const float v = fmaf(wc, xc, fmaf(wp, xp, a0));
        if (a.scores) a.scores[s * a.C + c] = v;
        amax_take(bv, bi, v, c);
    }
    if (!a.best_idx) return;
    amax_wave(bv, bi);
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    for (int w = 0; w < 4; ++w) if (w != wave) amax_take(bv, bi, sv[w], si[w]);     // every thread ends with the block's choice
    if (t == 0) {
        a.best_idx[s] = (bi == AB_NONE) ? -1 : bi;
        if (a.best_score) a.best_score[s] = (bi == AB_NONE) ? __uint_as_float(0x7fc00000u) : bv;
    }
    if (a.v_best && t < a.n_out) {
        float v = __uint_as_float(0x7fc00000u);
        if (bi != AB_NONE) {
            const float xp = phi(part[bi / a.Q], a.enc_part), xc = phi(cred[bi % a.Q], a.enc_cred);
            const float d = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) + a.b[t];
            v = fmaf(load_as_f32<T>(a.W, (int64_t)t * a.F + Fs + 1), xc, fmaf(load_as_f32<T>(a.W, (int64_t)t * a.F + Fs), xp, d));
        }
        a.v_best[s * a.n_out + t] = v;
    }
}

hipError_t launch_score_linear(int dtype, const ab_model_desc *d, const ab_params *prm, const float *dyn,
                               const float *scal, const ab_grid *grid, int64_t S, float *scores, int32_t *best_idx,
                               float *best_score, float *v_best, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    if (S > 0x7fffffffLL) return hipErrorInvalidValue;
    LinearArgs a = {};
    a.dyn = dyn; a.scal = scal; a.part = grid->partition_bytes; a.cred = grid->credit_mult;
    a.part_stride = grid->per_scenario ? grid->P : 0; a.cred_stride = grid->per_scenario ? grid->Q : 0;
    a.n_stat = d->n_layers * d->n_stats; a.K = d->n_stats; a.Ns = d->n_scalars; a.Q = grid->Q; a.C = grid->P * grid->Q;
    a.F = a.n_stat + a.Ns + 2; a.n_out = d->n_outputs > 1 ? d->n_outputs : 1;
    a.W = prm->W[0]; a.b = prm->b[0];
    for (int i = 0; i < AB_MAX_STATS; ++i) a.enc_stat[i] = d->enc_stat[i];
    for (int i = 0; i < AB_MAX_SCALARS; ++i) a.enc_scalar[i] = d->enc_scalar[i];
    a.enc_part = d->enc_partition; a.enc_cred = d->enc_credit;
    a.scores = scores; a.best_idx = best_idx; a.best_score = best_score; a.v_best = v_best;
    if (dtype == AB_BF16) score_linear_kernel<bf16_t><<<(unsigned)S, 256, 0, st>>>(a);
    else                  score_linear_kernel<float><<<(unsigned)S, 256, 0, st>>>(a);
    return hipGetLastError();
}

bool score_tiny_supported(const ab_model_desc *d, int64_t S, int32_t C)
{
    if (d->tensor_encoder || d->n_hidden < 1 || d->n_outputs > 1) return false;
    for (int k = 0; k < d->n_hidden; ++k) if (d->hidden[k] > 128) return false;     // (multiples of 64 already)
    const int64_t Fs = (int64_t)d->n_layers * d->n_stats + d->n_scalars;
    return Fs <= 2048 && C <= 256 && S >= 1 && S * C <= 16384;
}

hipError_t launch_score_tiny(int dtype, const ab_model_desc *d, const ab_params *prm, const float *dyn,
                             const float *scal, const float *part, const float *cred, int32_t P, int32_t Q,
                             int per_scenario, int64_t S, float *scores, int32_t *best_idx, float *best_score,
                             hipStream_t st)
{
    TinyArgs a = {};
    a.dyn = dyn; a.scal = scal; a.part = part; a.cred = cred;
    a.part_stride = per_scenario ? P : 0; a.cred_stride = per_scenario ? Q : 0;
    a.L = d->n_layers; a.K = d->n_stats; a.Ns = d->n_scalars; a.Q = Q; a.C = P * Q;
    a.Fs = d->n_layers * d->n_stats + d->n_scalars; a.F = a.Fs + 2; a.D = d->n_hidden;
    for (int k = 0; k < d->n_hidden; ++k) a.H[k] = d->hidden[k];
    for (int k = 0; k <= d->n_hidden; ++k) { a.W[k] = prm->W[k]; a.b[k] = prm->b[k]; }
    for (int i = 0; i < AB_MAX_STATS; ++i) a.enc_stat[i] = d->enc_stat[i];
    for (int i = 0; i < AB_MAX_SCALARS; ++i) a.enc_scalar[i] = d->enc_scalar[i];
    a.enc_part = d->enc_partition; a.enc_cred = d->enc_credit;
    a.scores = scores; a.best_idx = best_idx; a.best_score = best_score;
    constexpr int smem = (2 * 64 * 132 + 128 * 132) * 4;       // activation buffers + one weight matrix as fp32, padded rows
    hipError_t e;
    if (dtype == AB_BF16) {
        static DeviceOnce once;
        e = ensure_dynamic_lds((const void *)score_tiny_kernel<bf16_t>, smem, once);
        if (e != hipSuccess) return e;
        score_tiny_kernel<bf16_t><<<(unsigned)S, 1024, smem, st>>>(a);
    } else {
        static DeviceOnce once;
        e = ensure_dynamic_lds((const void *)score_tiny_kernel<float>, smem, once);
        if (e != hipSuccess) return e;
        score_tiny_kernel<float><<<(unsigned)S, 1024, smem, st>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_trigger(const float *scores, int64_t S, int C, int64_t row_stride, const int32_t *cur_idx,
                          const float *observed, float gain_threshold, float error_threshold, int32_t *best_idx,
                          float *gain, uint8_t *reconf, uint8_t *adapt, hipStream_t st)
{
    if (S == 0) return hipSuccess;
    TriggerArgs a{scores, row_stride, C, cur_idx, observed, gain_threshold, error_threshold, best_idx, gain, reconf, adapt};
    if (C <= 1024) launch_decide_rows(a, scores, row_stride, S, st);
    else trigger_kernel<<<(unsigned)S, 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_score_single_hidden(const float *a_term, const float *b_term, const float *w_out_f,
                                      float *partial, int64_t rows, int C, int H, const float *wp, const float *wc,
                                      const float *xp_row, const float *xc_row, hipStream_t st)
{
    if (rows == 0) return hipSuccess;
    ScoreD1Args a{a_term, b_term, w_out_f, partial, rows, C, H, wp, wc, xp_row, xc_row};
    score_single_hidden_kernel<<<(unsigned)((rows + 3) / 4), 256, 0, st>>>(a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Temporal encoder (Section 3.1 "Meta network architecture": the layer-wise statistics are embedded into
// a fixed width and a two-layer LSTM extracts the sequential features): e_t = W_e phi(stat[t]) + b_e
// (K -> 32), two stacked LSTM layers of 64 units over t = 0..L-1 with zero initial state, gate blocks in
// the order input, forget, candidate, output; the second layer's last hidden state becomes the first 64
// columns of the scenario row.
// One work-group of eight wavefronts per 2 G scenarios, the whole sequence in one launch; four wavefronts run
// the first layer, four the second one step behind:
//   - a wavefront owns 16 units of its layer and keeps their rows of [W_ih | W_hh] (bf16) in registers as first operands of
//     16 x 16 blocks, permuted so that the four gates of a unit land in one lane: row 4 u + g of block b is gate g of
//     unit 16 w + 4 u + b;  the bias is the addend of the first matrix instruction;
//   - the scenarios are two groups, half a step apart: while the gates of one group's step go through the vector ALUs,
//     the products of the other group's are on the matrix cores, then they change places (a step in one piece has all
//     wavefronts at the matrix cores first and at the vector ALUs afterwards);
//   - the recurrent operands live in LDS as rows [e | h1 | h2] (bf16), read in one half step and written in the next, a barrier
//     between: in iteration t layer 1 makes h1_t from (e_t, h1_{t-1}) and layer 2 makes h2_{t-1} from (h1_{t-1}, h2_{t-2});
//   - cell states stay in fp32 registers; sigmoid and tanh through exp2 and reciprocal;
//   - the statistics come in chunks of 16 steps, one chunk ahead; their loads are in flight over fourteen steps (a barrier
//     waits for LDS traffic only) and are transformed then.
// Columns of a block are scenarios; with G < 16 they repeat the group, and column c takes its cells from blocks
// (c / G) G / 4 ... alone: G / 4 cells a lane and group.
// ------------------------------------------------------------------------------------------------
struct LstmEncArgs {
    const float *dyn; int32_t L, K; int64_t S;
    const void *We; const float *be;      // [32, K]
    const void *W1; const float *b1;      // [256, 32 + 64]
    const void *W2; const float *b2;      // [256, 64 + 64]
    void *xs; int32_t ld;                 // scenario rows; columns [0, 64) written here
    const int32_t *layers_of;             // [S] or NULL: layers the scenario really has (clamped to [1, L])
    ab_enc enc_stat[AB_MAX_ENCODER_STATS];
};

__device__ __forceinline__ float fast_sigmoid(float x)
{
    return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896f * x));
}
__device__ __forceinline__ float fast_tanh(float x)
{
    return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(2.88539008177793f * x));
}

template <int G, int NG, int KQ>                           // NG groups of G scenarios, K <= 4 KQ
struct LstmLds {
    static constexpr int STRIDE = 336, TC = 16;    // bytes per row: (32 + 64 + 64) bf16 + 16 (bank spread); steps of a chunk
    alignas(16) unsigned char act[2 * G * STRIDE];   // rows of the two groups (of one group: by the step's parity)
    alignas(16) float stat[2][NG * G][TC][4 * KQ];   // (zero beyond K)
};
template <int G, int NG, int KQ, int ROLE>                 // ROLE 0: the first LSTM layer's wavefronts, 1: the second's
__device__ __forceinline__ void lstm_layer(const LstmEncArgs &a, LstmLds<G, NG, KQ> &lds)
{
    constexpr int E = 32, H = 64, TC = 16, R = NG * G, NC = G / 4, KM = 4 * KQ;
    constexpr int STRIDE = LstmLds<G, NG, KQ>::STRIDE, COL_H1 = E, COL_H2 = E + H;
    auto &act = lds.act;
    auto &stat = lds.stat;

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wu = wave & 3;                       // which 16 units
    const int col = lane & 15, u = lane >> 4, scen = col % G, b0 = col / G * NC;
    const int64_t s0 = (int64_t)blockIdx.x * R;
    const int L = a.L, K = a.K;

    // ---- statistics chunks: R rows x TC steps x K values; TPS threads to a row's step, KP values each
    constexpr int TPS = 32 / R, KP = KM > TPS ? KM / TPS : 1;
    const int prow = t / (TPS * TC), pstep = t / TPS % TC, k0 = t % TPS * KP;
    float pre[KP];
    ab_enc enc[KP];
#pragma unroll
    for (int i = 0; i < KP; ++i) enc[i] = a.enc_stat[k0 + i];
    const float *src = a.dyn + min(s0 + prow, a.S - 1) * (int64_t)L * K;
    float *mine = &stat[0][prow][pstep][k0];
    auto fetch_chunk = [&](int n) {
        const float *q = src + (int64_t)min(n * TC + pstep, L - 1) * K;
#pragma unroll
        for (int i = 0; i < KP; ++i) pre[i] = q[min(k0 + i, K - 1)];
        asm volatile("");                                // (keeps the compiler from merging this with put_chunk's stores: pre stays in registers)
    };
    auto put_chunk = [&](int buf) {
#pragma unroll
        for (int i = 0; i < KP; ++i)
            if (k0 < KM) {
                const float l = logf(pre[i]), v = ((enc[i].kind == AB_ENC_LOG ? l : pre[i]) - enc[i].shift) * enc[i].scale;      // phi, branch-free
                mine[buf * (R * TC * KM) + i] = k0 + i < K ? v : 0.f;
            }
    };
    // ---- embedding of a group's rows by the second layer's wavefronts: thread -> row, EO outputs (with G = 4 twice over)
    constexpr int EO = G == 16 ? 2 : 1;
    const int te = t & 255, erow = te / (E / EO) % G, ej = te % (E / EO) * EO;
    f32x4 we[EO][KQ];
    float be[EO];
#pragma unroll
    for (int i = 0; i < EO; ++i) {
        be[i] = a.be[ej + i];
#pragma unroll
        for (int k = 0; k < KM; ++k) we[i][k / 4][k % 4] = k < K ? bf16_bits_to_f32(((const uint16_t *)a.We)[(ej + i) * K + k]) : 0.f;
    }
    auto embed_step = [&](int step, int grp, int rows) { // e_step of a group -> columns [0, 32) of rows `rows` G ..
        const float *sp = &stat[(step / TC) & 1][grp * G + erow][step % TC][0];
        float e[EO];
#pragma unroll
        for (int i = 0; i < EO; ++i) e[i] = be[i];
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const f32x4 x = *(const f32x4 *)(sp + 4 * q);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < EO; ++i) e[i] = fmaf(we[i][q][k], x[k], e[i]);
        }
        const uint32_t pk = pack_bf16x2(e[0], e[EO - 1]);
        unsigned char *dst = act + (rows * G + erow) * STRIDE + ej * 2;
        if constexpr (EO == 2) *(uint32_t *)dst = pk;
        else                   *(uint16_t *)dst = (uint16_t)(pk & 0xffffu);
    };
    auto meet = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- start: zero state, first chunk, e_0
    for (int i = t; i < 2 * G * STRIDE / 4; i += 512) ((uint32_t *)act)[i] = 0u;
    fetch_chunk(0);
    put_chunk(0);
    __syncthreads();
    if (ROLE) {
        embed_step(0, 0, 0);
        if constexpr (NG == 2) embed_step(0, 1, 1);
    }
    meet();

    constexpr int NK = ROLE ? 4 : 3;
    constexpr int COL = ROLE ? COL_H1 : 0, OUT = ROLE ? COL_H2 : COL_H1, KIN = ROLE ? 2 * H : E + H;
    // this wavefront's weights: lane -> row (col) of a block and eight k values (u)
    bf16x8 wf[4][NK];
    f32x4 bias[4];
    const uint16_t *W = (const uint16_t *)(ROLE ? a.W2 : a.W1);
    const float *bsrc = ROLE ? a.b2 : a.b1;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int wrow = (col & 3) * H + 16 * wu + 4 * (col >> 2) + b;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) wf[b][ks] = __builtin_bit_cast(bf16x8, *(const i32x4 *)(W + (size_t)wrow * KIN + ks * 32 + 8 * u));
#pragma unroll
        for (int g = 0; g < 4; ++g) bias[b][g] = bsrc[g * H + 16 * wu + 4 * u + b];
    }
    // the scenario of a lane may have fewer layers than the block runs for: its result is the second layer's hidden state
    // after its own last layer; what the recurrence does to that row afterwards is unused
    int my_len[NG];
#pragma unroll
    for (int x = 0; x < NG; ++x) my_len[x] = L;
    if (ROLE && a.layers_of) {
#pragma unroll
        for (int x = 0; x < NG; ++x) {
            const int n = a.layers_of[min(s0 + x * G + scen, a.S - 1)];
            my_len[x] = n < 1 ? 1 : (n > L ? L : n);
        }
    }
    float c[NG][NC], hv[NC], hlast[NG][NC];
#pragma unroll
    for (int x = 0; x < NG; ++x)
#pragma unroll
        for (int i = 0; i < NC; ++i) c[x][i] = hlast[x][i] = 0.f;
    f32x4 z[NG][4];
    const unsigned char *frag = act + scen * STRIDE + 16 * u + COL * 2;
    unsigned char *h_wr = act + scen * STRIDE + (16 * wu + 4 * u + b0 + OUT) * 2;

    auto products = [&](int x, int rows) {
        bf16x8 xf[NK];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) xf[ks] = __builtin_bit_cast(bf16x8, *(const i32x4 *)(frag + rows * G * STRIDE + ks * 64));
#pragma unroll
        for (int ks = 0; ks < NK; ++ks)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                z[x][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[b][ks], xf[ks], ks == 0 ? bias[b] : z[x][b], 0, 0, 0);
    };
    auto cells = [&](int x) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            f32x4 y = z[x][i];
            if constexpr (G == 8) {
#pragma unroll
                for (int g = 0; g < 4; ++g) y[g] = b0 ? z[x][2 + i][g] : z[x][i][g];
            }
            if constexpr (G == 4) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float lo = b0 & 1 ? z[x][1][g] : z[x][0][g], hi = b0 & 1 ? z[x][3][g] : z[x][2][g];
                    y[g] = b0 & 2 ? hi : lo;
                }
            }
            const float ig = fast_sigmoid(y[0]), fg = fast_sigmoid(y[1]), gg = fast_tanh(y[2]), og = fast_sigmoid(y[3]);
            c[x][i] = fmaf(fg, c[x][i], ig * gg);
            hv[i] = og * fast_tanh(c[x][i]);
        }
    };
    auto put = [&](int rows) {
        unsigned char *dst = h_wr + rows * G * STRIDE;
        if constexpr (NC == 4)      *(uint2 *)dst = uint2{pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3])};
        else if constexpr (NC == 2) *(uint32_t *)dst = pack_bf16x2(hv[0], hv[1]);
        else                        *(uint16_t *)dst = (uint16_t)(pack_bf16x2(hv[0], 0.f) & 0xffffu);
    };
    // Half a step: the gates of group X's step tau, the products of the other group's next ones.  (One group: all of a step.)
    // Past its last step a layer makes rows that nobody reads.
    auto half_step = [&](auto x_tag, int tau) {
        constexpr int X = decltype(x_tag)::value;
        const int from = NG == 2 ? X ^ 1 : tau & 1, to = NG == 2 ? X : from ^ 1;
        if constexpr (ROLE) embed_step(min(tau + 1, L - 1), X, to);
        products(NG == 2 ? X ^ 1 : 0, from);
        cells(X);
        put(to);
        if constexpr (ROLE) {
#pragma unroll
            for (int i = 0; i < NC; ++i) hlast[X][i] = tau == my_len[X] ? hv[i] : hlast[X][i];
        }
        if constexpr (NG == 2) {                     // one matrix instruction, then some of the gates' work
            __builtin_amdgcn_sched_group_barrier(0x100, NK + (ROLE ? KQ : 0), 0);
            __builtin_amdgcn_sched_group_barrier(0x002, G, 0);
#pragma unroll
            for (int i = 0; i < 4 * NK; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
            }
        }
        meet();
    };
    auto chunks = [&](int tau) {
        const int tc = tau % TC, n = tau / TC;
        if (tc == 0 && (n + 1) * TC < L) fetch_chunk(n + 1);
        if (tc == TC - 2 && (n + 1) * TC < L) put_chunk((n + 1) & 1);
    };
    int tau = 0;
    if constexpr (NG == 2) {
        products(0, 0);
        meet();
    }
    if constexpr (ROLE) {                            // (the second layer has no step yet)
        chunks(0);
        embed_step(min(1, L - 1), 0, NG == 2 ? 0 : 1);
        if constexpr (NG == 2) {
            products(1, 1);
            meet();
            embed_step(min(1, L - 1), 1, 1);
            products(0, 0);
        }
        meet();
        tau = 1;
    }
    for (; tau <= L; ++tau) {
        chunks(tau);
        half_step(std::integral_constant<int, 0>{}, tau);
        if constexpr (NG == 2) half_step(std::integral_constant<int, 1>{}, tau);
    }
    // ---- second layer's hidden state after the scenario's last layer
    if constexpr (ROLE) {
#pragma unroll
        for (int x = 0; x < NG; ++x) {
            if (s0 + x * G + scen >= a.S) continue;
            uint16_t *dst = (uint16_t *)a.xs + (s0 + x * G + scen) * (int64_t)a.ld + 16 * wu + 4 * u + b0;
            if constexpr (NC == 4)      *(uint2 *)dst = uint2{pack_bf16x2(hlast[x][0], hlast[x][1]), pack_bf16x2(hlast[x][2], hlast[x][3])};
            else if constexpr (NC == 2) *(uint32_t *)dst = pack_bf16x2(hlast[x][0], hlast[x][1]);
            else                        *dst = (uint16_t)(pack_bf16x2(hlast[x][0], 0.f) & 0xffffu);
        }
    }
}

template <int G, int NG, int KQ>
__global__ __launch_bounds__(512) void lstm_encoder_kernel(const LstmEncArgs a, const SideArgs side, const unsigned grid)
{
    if (blockIdx.x >= grid) {
        side_block<512>(side, blockIdx.x - grid);
        return;
    }
    __shared__ LstmLds<G, NG, KQ> lds;
    // Of the two wavefronts of a SIMD the one of the second layer has more to do per step (four k steps against three,
    // and the next step's embedding) and, being the younger one, would be served last: it gets the higher priority.
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 8)) {
        __builtin_amdgcn_s_setprio(2);
        lstm_layer<G, NG, KQ, 1>(a, lds);
    } else lstm_layer<G, NG, KQ, 0>(a, lds);
}

// As few scenarios a work-group as fill the CUs once: a call runs its steps one after another, and a step takes 0.50, 0.58, 0.81
// and 1.49 us with 4, 8, 16 and 32 of them.  A call of 200 steps, us, with 4 / 8 / 16 / 32 a work-group: 16 scenarios 125 / 140 / 186 /
// 325, 1024 153 / 167 / 213 / 353, 2048 287 / 196 / 242 / 380, 4096 557 / 374 / 298 / 436.  Beyond 16 a CU: 32.
template <int KQ>
static hipError_t launch_lstm(const LstmEncArgs &a, const SideArgs &side, hipStream_t st)
{
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    const int r = a.S <= 4 * (int64_t)cus ? 4 : a.S <= 8 * (int64_t)cus ? 8 : a.S <= 16 * (int64_t)cus ? 16 : 32;
    const int64_t grid = (a.S + r - 1) / r;
    if (grid + side.blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    auto launch = [&](auto kern) { kern<<<(unsigned)grid + side.blocks, 512, 0, st>>>(a, side, (unsigned)grid); };
    if (r == 4)       launch(lstm_encoder_kernel<4, 1, KQ>);
    else if (r == 8)  launch(lstm_encoder_kernel<8, 1, KQ>);
    else if (r == 16) launch(lstm_encoder_kernel<16, 1, KQ>);
    else              launch(lstm_encoder_kernel<16, 2, KQ>);
    return hipGetLastError();
}

// The work beside an encoder, for work-groups of `threads`; none, and o.done false, where the scalars' layout needs the general
// transform or the candidate table is large (its blocks run slower beside an encoder's, of which few fit a CU).
static SideArgs encoder_side(const ab_model_desc *d, const float *dyn, void *xs, int ld, int64_t S, const EncoderSide &o, int threads, bool *done)
{
    SideArgs a;
    memset(&a, 0, sizeof(a));
    fill_encode_args(a.e, d, dyn, o.scal, xs, S, ld, d->enc_hidden[1], 0);
    *done = quad_split(AB_BF16, d, a.e, a.g) && !(o.b_term && (int64_t)o.grid->P * o.grid->Q * o.H1 > 1 << 19);
    if (!*done) return a;
    const int64_t n = fill_prep_args(a.p, d, o.W1, o.b1, o.F, o.Fs, o.H1, ld, o.w1s, o.grid, o.b_term, o.cfg_vec, o.Wout, o.b_out, o.H_last, o.w_out_f);
    const int64_t enc_blocks = (S + a.g.rpb - 1) / a.g.rpb, blocks = enc_blocks + (n + threads - 1) / threads;
    if (blocks > 0x3fffffffLL) { *done = false; return a; }
    a.enc_blocks = (unsigned)enc_blocks;
    a.blocks = (unsigned)blocks;
    return a;
}

hipError_t launch_lstm_encoder(const ab_model_desc *d, const float *dyn, const void *We, const float *be,
                               const void *W1, const float *b1, const void *W2, const float *b2, void *xs,
                               int ld, int64_t S, const int32_t *layers_of, const EncoderSide &o, bool *side_done, hipStream_t st)
{
    *side_done = false;
    if (S == 0) return hipSuccess;
    LstmEncArgs a;
    a.layers_of = layers_of;
    a.dyn = dyn; a.L = d->n_layers; a.K = d->n_stats; a.S = S;
    a.We = We; a.be = be; a.W1 = W1; a.b1 = b1; a.W2 = W2; a.b2 = b2; a.xs = xs; a.ld = ld;
    for (int i = 0; i < AB_MAX_ENCODER_STATS; ++i) a.enc_stat[i] = d->enc_stat[i];
    const SideArgs side = encoder_side(d, dyn, xs, ld, S, o, 512, side_done);
    return a.K <= 4 ? launch_lstm<1>(a, side, st) : launch_lstm<2>(a, side, st);
}

hipError_t launch_tensor_encoder(const ab_model_desc *d, const float *dyn, const void *Wa, const float *ba,
                                 const void *Wb, const float *bb, void *xs, int ld,
                                 int64_t S, const int32_t *layers_of, const EncoderSide &o, bool *side_done, hipStream_t st)
{
    *side_done = false;
    if (S == 0) return hipSuccess;
    TensorEncArgs a;
    a.layers_of = layers_of;
    a.dyn = dyn; a.L = d->n_layers; a.K = d->n_stats; a.Wa = Wa; a.ba = ba; a.Wb = Wb; a.bb = bb;
    a.xs = xs; a.ld = ld; a.S = S;
    for (int i = 0; i < AB_MAX_ENCODER_STATS; ++i) a.enc_stat[i] = d->enc_stat[i];
    int cus = 0;
    hipError_t e;
    if ((e = compute_units(&cus)) != hipSuccess) return e;
    const unsigned grid = (unsigned)(S < 2 * (int64_t)cus ? S : 2 * (int64_t)cus);      // two work-groups a CU (their registers)
    const SideArgs side = encoder_side(d, dyn, xs, ld, S, o, 256, side_done);
    if (a.K <= 4) tensor_encoder_kernel<2><<<grid + side.blocks, 256, 0, st>>>(a, side, grid);
    else          tensor_encoder_kernel<4><<<grid + side.blocks, 256, 0, st>>>(a, side, grid);
    return hipGetLastError();
}

}  // namespace ab
