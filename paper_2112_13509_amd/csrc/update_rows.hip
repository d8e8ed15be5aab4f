// The online update in row-block form: forward pass, output unit, loss terms and the delta chain of a block of 16 or 32
// batch rows in one work-group, then all weight gradients in one launch, with the Adam step in it (update_step_kernel) or in a
// launch of update.hip behind it (update.hip decides when).
//
// Why this form: a chain of GEMM launches pays about 5 us a launch before its first product (dispatch, arguments, first
// misses: what a launch reads was written by other XCDs and comes from the Infinity Cache) and the chain has one launch
// per layer and direction.  Everything up to the deltas is local to a batch row, so a work-group can take a block of
// rows through all layers; what it pays for that is streaming every weight matrix (twice, where a delta is needed) from
// its XCD's L2 by itself.  16 KB transfers into LDS reach 48 - 53 bytes a clock and CU, i.e. 4.5 us for a 512 x 512 bf16 matrix,
// whether one CU or all 256 stream (the row-major fragments loaded straight into registers take 13 us, their 16 rows at a
// power-of-two pitch fall on few L2 channels).
// Where the time goes, by clock stamps in the middle work-group, us: 4096 rows of 390-512-512-512-1 in bf16, 36.5 (39.3 with
// launch and drain): prologue 3.3, the five products 26.4 (4.8 - 5.6 each), the barriers behind them 4.5 (about 0.9 each: the
// wavefronts end apart), output unit 0.9, its delta 1.0.  1000 rows, last layer and output unit trainable, 24.2: prologue 3.6,
// three products 14.2, barriers 2.9, output unit 1.0, its delta 2.0.  200 rows of 54-64-64-1 in fp32, 12.7: prologue 2.5, three
// products 2.4 - 3.1 each (eight wavefronts share one slice: a few units each, their latency and the exchange in LDS).
// So the stream bounds the large networks to about two thirds; the rest is the chain around it.
#include "update_rows.hpp"
#include "stream_util.hpp"

namespace ab {

// ---------------------------------------------------------------------------------------------
// Rows kernel.  Eight wavefronts; a layer's outputs are cut into slices of 64 columns, a slice a wavefront (wider layers
// take several passes; for narrower ones the wavefronts of a slice split the inputs and their sums meet in LDS).
// A wavefront streams its own weights through a private ring of four 2 KB units (no barrier inside a layer, two
// transfers a unit, six may stay in flight when a unit is consumed); the stream runs on across layers.  Products on
// 16 x 16 blocks, weights first operand: a lane ends with batch row (lane & 15) and four adjacent columns.
//   forward unit: 16 rows of W (outputs) x 128 bytes of inputs; chunk c of row r sits at c ^ (r & 7).
//   backward unit (W used transposed): 16 (fp32: 8) rows of W = inputs of the product, 64 columns = its outputs.  bf16
//     fragments come through the transposing LDS read, whose sixteen lanes take 4 rows x 32 bytes: chunk c of row r sits
//     at c ^ 2 (r & 3), so the four rows fall into different bank groups; fp32 fragments are 4-byte reads, 64-byte
//     group q of row r sits at q ^ ((r >> 2) & 3).
// Activations and deltas of the block live in LDS (two buffers by layer parity, chunk c of row r at c ^ (r & 7)); a
// layer's result goes to memory as well, for the gradient launch, straight from the registers: those stores stand in the queue
// behind the units on their way, so a layer's first waits also wait for some of them (never for less than their units).  The block's input
// rows, biases, output weights and targets come by DMA too: ahead of the first weights, all of them in flight at once.  ReLU masks are kept as one
// bit per result in the lane that will need it again.
// ---------------------------------------------------------------------------------------------
static constexpr int NU = 4, UNIT = 2048;

template <typename T>
__device__ __forceinline__ f32x4 mma16(const i32x4 &w, const i32x4 &x, f32x4 acc)
{
    if constexpr (sizeof(T) == 2) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
    } else {
        const f32x4 a = __builtin_bit_cast(f32x4, w), b = __builtin_bit_cast(f32x4, x);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
        return acc;
    }
}

// Four bf16 down a column: sixteen lanes read 4 rows x 16 columns (8 bytes each), lane i ends with column i.  Written out,
// because the compiler drains all global->LDS transfers in front of the builtin; the reads of a block and their wait are one
// statement, so that no register of theirs can be touched while a read is on its way.
// v[i] = the four rows at p[i], w[i] = those OFF bytes on.
template <int OFF>
__device__ __forceinline__ void lds_read_tr_4x2(uint2 (&v)[4], uint2 (&w)[4], const unsigned char *const (&p)[4])
{
    auto at = [](const unsigned char *q) { return (uint32_t)(uintptr_t)(lds_void *)q; };
    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %4, %8 offset:%12\n\t"
                 "ds_read_b64_tr_b16 %1, %9\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
                 "ds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %6, %10 offset:%12\n\t"
                 "ds_read_b64_tr_b16 %3, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(at(p[0])), "v"(at(p[1])), "v"(at(p[2])), "v"(at(p[3])), "i"(OFF) : "memory");
}
// v[i][...] = the four rows at p[i], those 4, 16 and 20 rows of ROWB bytes on.
template <int ROWB>
__device__ __forceinline__ void lds_read_tr_4x4(uint2 (&v)[4][4], const unsigned char *const (&p)[4])
{
    auto at = [](const unsigned char *q) { return (uint32_t)(uintptr_t)(lds_void *)q; };
    asm volatile("ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:%20\n\t"
                 "ds_read_b64_tr_b16 %2, %16 offset:%21\n\tds_read_b64_tr_b16 %3, %16 offset:%22\n\t"
                 "ds_read_b64_tr_b16 %4, %17\n\tds_read_b64_tr_b16 %5, %17 offset:%20\n\t"
                 "ds_read_b64_tr_b16 %6, %17 offset:%21\n\tds_read_b64_tr_b16 %7, %17 offset:%22\n\t"
                 "ds_read_b64_tr_b16 %8, %18\n\tds_read_b64_tr_b16 %9, %18 offset:%20\n\t"
                 "ds_read_b64_tr_b16 %10, %18 offset:%21\n\tds_read_b64_tr_b16 %11, %18 offset:%22\n\t"
                 "ds_read_b64_tr_b16 %12, %19\n\tds_read_b64_tr_b16 %13, %19 offset:%20\n\t"
                 "ds_read_b64_tr_b16 %14, %19 offset:%21\n\tds_read_b64_tr_b16 %15, %19 offset:%22\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0][0]), "=&v"(v[0][1]), "=&v"(v[0][2]), "=&v"(v[0][3]), "=&v"(v[1][0]), "=&v"(v[1][1]),
                   "=&v"(v[1][2]), "=&v"(v[1][3]), "=&v"(v[2][0]), "=&v"(v[2][1]), "=&v"(v[2][2]), "=&v"(v[2][3]),
                   "=&v"(v[3][0]), "=&v"(v[3][1]), "=&v"(v[3][2]), "=&v"(v[3][3])
                 : "v"(at(p[0])), "v"(at(p[1])), "v"(at(p[2])), "v"(at(p[3])), "i"(4 * ROWB), "i"(16 * ROWB), "i"(20 * ROWB)
                 : "memory");
}
__device__ __forceinline__ i32x4 join(const uint2 &lo, const uint2 &hi) { return i32x4{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y}; }

template <int R16> using RowsArgsOf = std::conditional_t<R16 == 1, RowsArgs, Rows32Args>;

template <typename T, int R16, bool FOLD>
__global__ __launch_bounds__(512) void update_rows_kernel(const RowsArgsOf<R16> a)
{
    constexpr int R = 16 * R16, ES = sizeof(T);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * R;
    // touch_arguments, written out: through the function the compiler orders this opening otherwise (the figures are at Rows32Args)
    {
        typedef __attribute__((address_space(4))) const uint32_t karg;
        karg *ka = (karg *)__builtin_amdgcn_kernarg_segment_ptr();
        uint32_t sink = 0;
#pragma unroll
        for (int i = 0; i < (int)sizeof(a); i += 64) sink ^= ka[i / 4];
        asm volatile("" ::"s"(sink));
    }
    const int D = a.D, k0 = a.k0, n_out = a.n_out;
    unsigned char *ring = smem + wave * (NU * UNIT);
    auto buf = [&](int k) { return smem + (k & 1 ? a.o_odd : a.o_even); };         // holds h_k, then delta_k (x: k = -1)
    // byte `o` of row `row` of an activation buffer `width` wide
    auto at = [](int width, int row, int o) { return row * width * ES + (o ^ ((row & 7) << 4)); };

    // ---- the stream of weight blocks (four units): job, pass, block
    struct { const unsigned char *base; uint32_t step, blk_step, off0, off1, flip; int job, pass, left; bool done; } cur;
    auto range = [&](const RowsJob &j, int pass, int &slice, int &b0, int &b1) {     // this wavefront's part of a pass
        if (j.ks_shift == 0) {
            slice = pass * 8 + wave;
            b0 = 0;
            b1 = slice < j.n_slices ? j.n_blk : 0;
        } else {
            const int ks = (wave * j.recip) >> 5;
            slice = wave - ks * j.n_slices;
            b0 = (j.n_blk * ks) >> j.ks_shift;
            b1 = (j.n_blk * (ks + 1)) >> j.ks_shift;
            if (ks >> j.ks_shift) b0 = b1 = 0;
        }
    };
    auto open = [&](int job, int pass) {                    // first unit of (job, pass), or of the next one with work
        for (; job < a.n_jobs; ++job, pass = 0) {
            const RowsJob j = a.job[job];
            for (; pass < j.passes; ++pass) {
                int slice, b0, b1;
                range(j, pass, slice, b0, b1);
                if (b0 >= b1) continue;
                cur.job = job; cur.pass = pass; cur.left = b1 - b0; cur.flip = 0;
                cur.step = 16 * j.ld;
                cur.blk_step = j.back ? 4 * cur.step : 128;
                cur.base = j.W + (j.back ? (int64_t)b0 * cur.blk_step + slice * (64 * ES) : (int64_t)slice * 64 * j.ld + b0 * 128);
                const uint32_t row = lane >> 3, ch = (lane & 7) ^ (j.back ? (row & 3) << 1 : row);
                cur.off0 = row * j.ld + ch * 16;
                cur.off1 = cur.off0 + 8 * j.ld;
                if (ES == 4 && j.back) {
                    cur.step = 8 * j.ld; cur.blk_step = 4 * cur.step; cur.flip = 128;
                    cur.base = j.W + (int64_t)b0 * cur.blk_step + slice * 256;
                    cur.off0 = (lane >> 4) * j.ld + (lane & 15) * 16;
                    cur.off1 = ((lane >> 4) + 4) * j.ld + ((lane & 15) ^ 4) * 16;
                }
                return;
            }
        }
        cur.done = true;                                    // (the last block is fetched again into slots nobody reads)
    };
    auto issue = [&](int u) {
        const unsigned char *src = cur.base + u * cur.step;
        unsigned char *dst = ring + u * UNIT;
        const uint32_t xr = u & 1 ? cur.flip : 0;
        dma16<false>(src + (cur.off0 ^ xr), dst);
        dma16<false>(src + (cur.off1 ^ xr), dst + 1024);
    };
    auto next = [&]() {
        if (cur.done) return;
        if (--cur.left > 0) cur.base += cur.blk_step;
        else open(cur.job, cur.pass + 1);
    };
    cur.done = false;
    cur.base = a.job[0].W;
    cur.step = cur.off0 = cur.off1 = cur.flip = 0;
    open(0, 0);

    // ---- the block's input rows and the tables, then the first weights
    {
        const int cpr = a.l[0].in * ES / 16;                // 16-byte chunks a row, a multiple of 8
        const unsigned char *x = (const unsigned char *)a.x + row0 * (int64_t)(cpr * 16);
        for (int p = wave; p < R * cpr / 64; p += 8) {
            const int c = p * 64 + lane, row = c / cpr, ch = (c - row * cpr) ^ (row & 7);
            dma16<false>(x + (row * cpr + ch) * 16, buf(-1) + p * 1024);
        }
        int turn = 0;                                       // pieces of 64 words, dealt out over the wavefronts
        auto table = [&](const void *src, int words, int o) {        // (the last piece repeats its last word)
            for (int p = 0; p < words; p += 64, ++turn)
                if ((turn & 7) == wave) {
                    const int i = p + lane < words ? p + lane : words - 1;
                    dma4((const uint32_t *)src + i, smem + o + p * 4);
                }
        };
        int o = a.o_bias;
        for (int k = 0; k < D; o += a.l[k].out * 4, ++k) table(a.l[k].b, a.l[k].out, o);
        table(a.w_out, n_out * a.l[D - 1].out * ES / 4, a.o_wout);
        table(a.b_out, n_out, a.o_bout);
        const int64_t rows = a.B - row0 < R ? a.B - row0 : R;
        if (rows > 0) table(a.target + row0 * n_out, (int)rows * n_out, a.o_tgt);
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) issue(u);
    next();
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    __builtin_amdgcn_s_barrier();

    f32x4 acc[R16][4];
    auto clear = [&]() {
#pragma unroll
        for (int rr = 0; rr < R16; ++rr)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) acc[rr][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // FOLD: shares of the inputs that a wavefront takes one after the other (32-row blocks, where the LDS does not hold the sums of
    // more wavefronts): each share's sums begin at zero, as they do in a wavefront of its own.  (In all kernels of 32 rows: 0.6 % of a step.)
    f32x4 whole[R16][4];
    int cut = 0, share = 0, fold = 0;
    auto first_cut = [&](const RowsJob &j, int job) {
        if constexpr (FOLD) {
            fold = a.folds >> (2 * job) & 3;
            if (!fold) { cut = -1; return; }
            share = ((wave * j.recip) >> 5) << fold;
            cut = (j.n_blk * (share + 1)) >> (j.ks_shift + fold);
#pragma unroll
            for (int q = 0; q < R16 * 4; ++q) whole[q >> 2][q & 3] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto end_of_block = [&](const RowsJob &j, int b, int b1) {
        if constexpr (!FOLD) return;
        if (b + 1 != cut) return;
#pragma unroll
        for (int q = 0; q < R16 * 4; ++q) whole[q >> 2][q & 3] += acc[q >> 2][q & 3];
        if (b + 1 == b1) {
#pragma unroll
            for (int q = 0; q < R16 * 4; ++q) acc[q >> 2][q & 3] = whole[q >> 2][q & 3];
            return;
        }
        clear();
        cut = (j.n_blk * (++share + 1)) >> (j.ks_shift + fold);        // (every share has a block)
    };
    // sums of the wavefronts that split a slice's inputs; true in the wavefront that goes on with the slice
    auto combine = [&](const RowsJob &j) {
        if (j.ks_shift == 0) return true;
        const int ks = (wave * j.recip) >> 5, n = j.n_slices, slice = wave - ks * n;
        unsigned char *part = smem + a.o_scratch + slice * (R16 * 4096) + lane * 16;
        if (ks > 0 && !(ks >> j.ks_shift)) {
#pragma unroll
            for (int q = 0; q < R16 * 4; ++q)
                lds_write16(part + (ks - 1) * n * (R16 * 4096) + q * 1024, __builtin_bit_cast(i32x4, acc[q >> 2][q & 3]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if (ks > 0) return false;
        for (int q2 = 0; q2 < (1 << j.ks_shift) - 1; ++q2)
#pragma unroll
            for (int q = 0; q < R16 * 4; ++q)
                acc[q >> 2][q & 3] += *(const f32x4 *)(part + q2 * n * (R16 * 4096) + q * 1024);
        return true;
    };
    // a layer's result (64-column slice in acc), rounded to the compute type -> its buffer and its place in memory
    auto put = [&](unsigned char *dst, void *out, int width, int slice) {
#pragma unroll
        for (int rr = 0; rr < R16; ++rr)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int row = 16 * rr + r, o = (slice * 64 + nb * 16 + g * 4) * ES;
                unsigned char *p = dst + at(width, row, o), *q = (unsigned char *)out + (row0 + row) * (int64_t)(width * ES) + o;
                const f32x4 v = acc[rr][nb];
                if constexpr (ES == 2) {
                    const uint2 b = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                    lds_write8(p, b);
                    *(uint2 *)q = b;
                } else {
                    lds_write16(p, __builtin_bit_cast(i32x4, v));
                    *(f32x4 *)q = v;
                }
            }
    };
    auto meet = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };

    // ---- forward
    int o_bias = a.o_bias, o_mask = a.o_mask;
    for (int k = 0; k < D; ++k) {
        const int in = a.l[k].in, out = a.l[k].out;
        const RowsJob j = a.job[k];
        const unsigned char *src = buf(k - 1);
        for (int pass = 0; pass < j.passes; ++pass) {
            int slice, b0, b1;
            range(j, pass, slice, b0, b1);
            clear();
            first_cut(j, k);
            for (int b = b0; b < b1; ++b) {
                i32x4 x[R16][2];
#pragma unroll
                for (int rr = 0; rr < R16; ++rr)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) x[rr][ks] = *(const i32x4 *)(src + at(in, 16 * rr + r, b * 128 + ks * 64 + g * 16));
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
                    const unsigned char *u = ring + nb * UNIT + r * 128;
                    const i32x4 w0 = *(const i32x4 *)(u + ((g ^ (r & 7)) << 4)), w1 = *(const i32x4 *)(u + (((4 + g) ^ (r & 7)) << 4));
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    issue(nb);
#pragma unroll
                    for (int rr = 0; rr < R16; ++rr) {
                        acc[rr][nb] = mma16<T>(w0, x[rr][0], acc[rr][nb]);
                        acc[rr][nb] = mma16<T>(w1, x[rr][1], acc[rr][nb]);
                    }
                }
                next();
                end_of_block(j, b, b1);
            }
            const bool mine = combine(j) && slice < j.n_slices;
            if (mine) {
                uint32_t bits = 0;
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    const f32x4 bv = *(const f32x4 *)(smem + o_bias + (slice * 64 + nb * 16 + g * 4) * 4);
#pragma unroll
                    for (int rr = 0; rr < R16; ++rr) {
                        const bool live = row0 + 16 * rr + r < a.B;         // (rows of the padding stay zero)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = live ? relu_keep_nan(acc[rr][nb][e] + bv[e]) : 0.f;
                            bits |= v > 0.f ? 1u << (rr * 16 + nb * 4 + e) : 0u;
                            acc[rr][nb][e] = v;
                        }
                    }
                }
                put(buf(k), a.l[k].h, out, slice);
                lds_write4(smem + o_mask + (pass * 512 + t) * 4, __uint_as_float(bits));
            }
        }
        meet();
        o_bias += out * 4;
        o_mask += j.passes * 2048;
    }

    // ---- output unit: sixteen output rows (the last one again past n_out), the inputs split over the wavefronts
    const int H = a.l[D - 1].out;
    auto sums = [&]() { if constexpr (R16 == 1) return smem + a.o_scratch; else return smem + a.o_sums; };
    {
#pragma unroll
        for (int rr = 0; rr < R16; ++rr) acc[rr][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        const unsigned char *wsrc = smem + a.o_wout + (r < n_out ? r : n_out - 1) * H * ES + g * 16;
        for (int b = wave; b < H * ES / 64; b += 8) {
            const i32x4 w = *(const i32x4 *)(wsrc + b * 64);
#pragma unroll
            for (int rr = 0; rr < R16; ++rr) acc[rr][0] = mma16<T>(w, *(const i32x4 *)(buf(D - 1) + at(H, 16 * rr + r, b * 64 + g * 16)), acc[rr][0]);
        }
#pragma unroll
        for (int rr = 0; rr < R16; ++rr)
            lds_write16(sums() + ((wave * R16 + rr) * 64 + lane) * 16, __builtin_bit_cast(i32x4, acc[rr][0]));
        meet();
    }
    float *dout_s = (float *)(smem + a.o_dout);             // [R][16]
    if (t < R * 16) {
        const int row = t >> 4, w = t & 15;
        float yh = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            yh += ((const float *)sums())[((q * R16 + (row >> 4)) * 64 + (row & 15) + 16 * (w >> 2)) * 4 + (w & 3)];
        const bool live = row0 + row < a.B && w < n_out;
        float e = 0.f;
        if (live) e = (yh + ((const float *)(smem + a.o_bout))[w]) - ((const float *)(smem + a.o_tgt))[row * n_out + w];
        float sq = e * e;
        sq += dpp_move<0xB1>(sq);
        sq += dpp_move<0x4E>(sq);
        sq += dpp_move<0x141>(sq);
        sq += dpp_move<0x140>(sq);
        const float nrm = sqrtf(sq);
        const float f = a.loss_kind == AB_LOSS_L2NORM ? (nrm > 0.f ? 1.f / (nrm * (float)a.B) : 0.f) : 2.f / (float)a.B;
        e *= f;
        lds_write4(dout_s + t, e);
        if (w < n_out) a.dout[(row0 + row) * n_out + w] = e;
        if (w == 0) a.lossrow[row0 + row] = a.loss_kind == AB_LOSS_L2NORM ? nrm : sq;
    }
    meet();

    // ---- deltas
    // mask and put a slice of delta_k
    auto finish = [&](int k, int pass, int slice) {
        const uint32_t bits = *(const uint32_t *)(smem + o_mask + (pass * 512 + t) * 4);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int rr = 0; rr < R16; ++rr)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[rr][nb][e] = (bits >> (rr * 16 + nb * 4 + e)) & 1u ? acc[rr][nb][e] : 0.f;
        put(buf(k), a.l[k].d, a.l[k].out, slice);
    };
    if (k0 < D) {                                           // delta_{D-1} = (dout W_out) * [h > 0], slices as in the forward layer
        const RowsJob j = a.job[D - 1];
        o_mask -= j.passes * 2048;
        for (int pass = 0; pass < j.passes; ++pass) {
            const int slice = pass * 8 + wave;              // (of the wavefronts that shared a slice the first kept the mask)
            if (slice >= j.n_slices) break;
            clear();
            for (int w = 0; w < n_out; ++w) {
                float e[R16];
#pragma unroll
                for (int rr = 0; rr < R16; ++rr) e[rr] = dout_s[(16 * rr + r) * 16 + w];
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    const unsigned char *p = smem + a.o_wout + (w * H + slice * 64 + nb * 16 + g * 4) * ES;
                    f32x4 wv;
                    if constexpr (ES == 2) {
                        const uint2 b = *(const uint2 *)p;
                        wv = f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u),
                                   __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
                    } else wv = *(const f32x4 *)p;
#pragma unroll
                    for (int rr = 0; rr < R16; ++rr)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[rr][nb][q] = fmaf(e[rr], wv[q], acc[rr][nb][q]);
                }
            }
            finish(D - 1, pass, slice);
        }
        meet();
    }
    for (int k = D - 1; k > k0; --k) {                      // delta_{k-1} = (delta_k W_k) * [h_{k-1} > 0]
        const int in = a.l[k].out;
        const RowsJob j = a.job[2 * D - 1 - k];
        o_mask -= j.passes * 2048;
        const unsigned char *src = buf(k);
        for (int pass = 0; pass < j.passes; ++pass) {
            int slice, b0, b1;
            range(j, pass, slice, b0, b1);
            clear();
            first_cut(j, 2 * D - 1 - k);
            for (int b = b0; b < b1; ++b) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    i32x4 x[R16], w[4];
#pragma unroll
                    for (int rr = 0; rr < R16; ++rr) x[rr] = *(const i32x4 *)(src + at(in, 16 * rr + r, b * 128 + h * 64 + g * 16));
                    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
                    const unsigned char *u = ring + h * 2 * UNIT;
                    if constexpr (ES == 2) {
                        // lane i of a group of sixteen asks for row 8 g + (i >> 2) (then + 4), columns 4 (i & 3) .. + 3 of the block
                        const int row = 8 * g + (r >> 2);
                        uint2 lo[4], hi[4];
                        const unsigned char *p[4];
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb)
                            p[nb] = u + row * 128 + (((nb * 2 + ((r & 3) >> 1)) ^ ((r >> 2) << 1)) << 4) + (r & 1) * 8;
                        lds_read_tr_4x2<512>(lo, hi, p);
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb) w[nb] = join(lo[nb], hi[nb]);
                    } else {
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                w[nb][e] = *(const int *)(u + (4 * g + e) * 256 + (((nb * 4 + (r >> 2)) ^ (4 * g)) << 4) + (r & 3) * 4);
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    issue(2 * h);
                    issue(2 * h + 1);
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                        for (int rr = 0; rr < R16; ++rr) acc[rr][nb] = mma16<T>(w[nb], x[rr], acc[rr][nb]);
                }
                next();
                end_of_block(j, b, b1);
            }
            const bool mine = combine(j) && slice < j.n_slices;
            if (mine) finish(k - 1, pass, slice);
        }
        meet();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // no transfer may still target LDS when the group ends
}

// The jobs and the LDS of a rows launch, of blocks of 32 rows where `wide` says what they have beyond `a`; false where it does not fit.
// At most 1 << most_shift wavefronts share a slice (16 rows: eight, as many as there are).
static bool rows_layout(RowsArgs &a, int es, Rows32Args *wide, int most_shift, int *bytes)
{
    const int r16 = wide ? 2 : 1;
    auto fill = [&](RowsJob &j, int k, bool back) {
        const int n = (back ? a.l[k].in : a.l[k].out) / 64;
        j.W = (const unsigned char *)a.l[k].W; j.ld = (uint32_t)(a.l[k].in * es);
        j.n_blk = (uint16_t)((back ? a.l[k].out : a.l[k].in) * es / 128);
        j.n_slices = (uint16_t)n; j.back = back;
        // The wavefronts that a narrow layer's slices leave over share the slices' inputs, but none without a block of them: its
        // zeros would be written and added too.  Eight / as many as there are blocks, us a step: 54-64-64-1 fp32 200 rows 23.9 / 20.9,
        // 54-64-64-1 bf16 500 rows 24.1 / 22.0, 126-256-128-64-1 fp32 500 rows 35.0 / 33.3; two blocks each at least: 22.7, 22.0, 34.6
        j.ks_shift = n >= 5 ? 0 : n >= 3 ? 1 : n == 2 ? 2 : 3;
        while (j.ks_shift && (1 << j.ks_shift) > j.n_blk) --j.ks_shift;
        const int fold = j.ks_shift > most_shift ? j.ks_shift - most_shift : 0;
        if (wide) wide->folds |= (uint32_t)fold << 2 * (int)(&j - a.job);
        j.ks_shift -= fold;
        j.passes = (uint16_t)((n + 7) / 8);
        j.recip = (uint16_t)((31 + n) / n);
    };
    int even = 0, odd = a.l[0].in * es, bias = 0, masks = 0, part = 0;
    if (wide) wide->folds = 0;
    a.n_jobs = 0;
    for (int k = 0; k < a.D; ++k) {
        int &side = k & 1 ? odd : even;
        if (a.l[k].out * es > side) side = a.l[k].out * es;
        bias += a.l[k].out * 4;
        RowsJob &j = a.job[a.n_jobs++];
        fill(j, k, false);
        masks += j.passes * 2048;
    }
    for (int k = a.D - 1; k > a.k0; --k) fill(a.job[a.n_jobs++], k, true);
    for (int i = 0; i < a.n_jobs; ++i) {                    // sums that meet in LDS: a product's wavefronts beyond the first of a slice
        const int n = a.job[i].n_slices * ((1 << a.job[i].ks_shift) - 1);
        if (n > part) part = n;
    }
    int o = 8 * NU * UNIT;
    auto take = [&](int n) { const int at = o; o += (n + 255) / 256 * 256; return at; };      // (tables arrive in pieces of 256 bytes)
    a.o_even = take(16 * r16 * even);
    a.o_odd = take(16 * r16 * odd);
    a.o_bias = take(bias);
    a.o_wout = take(a.n_out * a.l[a.D - 1].out * es);
    a.o_bout = take(a.n_out * 4);
    a.o_tgt = take(16 * r16 * a.n_out * 4);
    a.o_mask = take(masks);
    a.o_dout = take(16 * r16 * 64);
    // the output unit's partial sums: in 32-row blocks where the last layer's inputs were, done with by then
    const bool free = wide && 16 * r16 * (a.D & 1 ? odd : even) >= r16 * 8192;
    a.o_scratch = take(r16 * (part * 4096 > 8192 || free ? part * 4096 : 8192));
    if (wide) wide->o_sums = !free ? a.o_scratch : a.D & 1 ? a.o_odd : a.o_even;
    *bytes = o;
    return o <= 160 * 1024;
}

template <typename T, int R16, bool FOLD>
static hipError_t launch_rows_one(const RowsArgsOf<R16> &a, int bytes, hipStream_t st)
{
    auto kern = update_rows_kernel<T, R16, FOLD>;
    static DeviceOnce once;
    hipError_t e = ensure_dynamic_lds((const void *)kern, 160 * 1024, once);
    if (e != hipSuccess) return e;
    const int64_t blocks = (a.B + 63) / 64 * (4 / R16);     // the padded batch: the gradient launch reads whole slabs of it
    kern<<<(unsigned)blocks, 512, bytes, st>>>(a);
    return hipGetLastError();
}

// Widths up to 1024, all weights together within an XCD's 4 MB L2 (beyond it the stream comes from the Infinity Cache at
// a fifth of the rate), activations and tables in LDS.
bool update_rows_supported(const RowsArgs &shape, int dtype)
{
    if (shape.D < 1) return false;
    const int es = dtype == AB_BF16 ? 2 : 4;
    int64_t weights = 0;
    for (int k = 0; k < shape.D; ++k) {
        if (shape.l[k].in > 1024 || shape.l[k].out > 1024) return false;
        weights += (int64_t)shape.l[k].in * shape.l[k].out * es;
    }
    RowsArgs a = shape;
    int bytes;
    return weights <= (int64_t)7 << 19 && rows_layout(a, es, nullptr, 3, &bytes);
}

// How many shares (1 << n) a wavefront takes at most one after the other in blocks of 32 rows; -1: such blocks do not fit the LDS, or
// only with one wavefront on a slice that four share in blocks of 16 (in those / so, fp32, us a step: 256-128-64 and 194 columns, 6000
// rows 80.6 / 82.1; 128-256 and 362, 4200 rows 67.5 / 72.9; two on a slice that eight share, 64-64 and 394 with eight outputs 57.3 / 54.0).
// The layout is left in `a`.
static int rows32_fold(Rows32Args &a, int es, int *bytes)
{
    for (int most = 3; most >= 0; --most) {
        const bool fits = rows_layout(a, es, &a, most, bytes);
        int fold = 0;
        for (int i = 0; i < a.n_jobs; ++i) {
            const int f = a.folds >> (2 * i) & 3;
            if (f > 1 && a.job[i].ks_shift == 0) return -1;
            if (f > fold) fold = f;
        }
        if (fits) return fold;
    }
    return -1;
}
int update_rows32_fold(const RowsArgs &shape, int dtype)
{
    Rows32Args a{shape};
    int bytes;
    return rows32_fold(a, dtype == AB_BF16 ? 2 : 4, &bytes);
}

// A work-group streams all weights whether it has 16 or 32 rows: 32 once there are more blocks of 16 than CUs, with fewer
// wavefronts on a slice where the LDS does not hold the sums of more.  Blocks of 16 / of 32 so, us a step: bf16, 512-512-512 with eight
// outputs, 4200 rows 93.5 / 71.7, 8192 110 / 89; 512-512 5500 74.4 / 59.4; fp32, 194 columns, 6000 rows: 64-64 50.7 / 44.4, 128-128 56.8 / 51.2,
// 256-256 81.3 / 76.9 (no slice is shared); 256-128-64, 62 columns 76.8 / 69.7.
template <typename T>
static hipError_t launch_rows(RowsArgs &a, int cus, hipStream_t st)
{
    int bytes = 0;
    Rows32Args w{a};
    const int fold = (a.B + 15) / 16 > cus ? rows32_fold(w, sizeof(T), &bytes) : -1;
    // (the kernel of 16 rows is named first, which is where the code object has it then: behind the others' 100 KB a step of 1000 or
    // 4096 rows took 0.1 us more)
    if (fold < 0) return rows_layout(a, sizeof(T), nullptr, 3, &bytes) ? launch_rows_one<T, 1, false>(a, bytes, st) : hipErrorInvalidValue;
    return fold ? launch_rows_one<T, 2, true>(w, bytes, st) : launch_rows_one<T, 2, false>(w, bytes, st);
}

hipError_t launch_update_rows(int dtype, RowsArgs a, hipStream_t st)
{
    int cus = 0;
    hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    return dtype == AB_BF16 ? launch_rows<bf16_t>(a, cus, st) : launch_rows<float>(a, cus, st);
}

// ---------------------------------------------------------------------------------------------
// Gradients launch: dW_k = delta_k^T h_{k-1} for every trainable hidden layer on W x W tiles (W = 128, for small networks
// 64), split over the batch, straight from the row-major deltas and activations (the batch, the summed index, is the slow
// one of both operands: fragments come through the transposing LDS read, fp32 ones as 4-byte reads); the bias gradients
// as column sums in the work-groups of a layer's first column tile; the output unit's weight gradient on the vector ALUs
// (64 columns and a share of the rows per work-group), its bias gradient and the loss: these come first, they are the
// longer chains.
// Bound by what a CU takes in (L2, then LDS): a 128 x 128 tile with 64 x 64 outputs a wavefront reads half the L2 bytes and
// half the LDS bytes of 64 x 64 with 32 x 32.  A slab is 8 KB of batch rows of either operand, by DMA into a ring of ST
// stages, one barrier a slab.  The batch split is the work-group number modulo the splits: with eight (four, ...) of them a
// share of the batch is read by one XCD (two, ...) only.
// ---------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void output_gradient(const GradsArgs &a, unsigned id, unsigned char *smem)
{
    constexpr int ES = sizeof(T), E = 16 / ES, CH = 64 / E, RG = 256 / CH;      // columns a thread, chunks a row, rows at a time
    constexpr int CHUNK = 8 * RG;                            // rows whose dout sits in LDS
    float *dout_s = (float *)smem, *red = (float *)(smem + CHUNK * AB_MAX_OUTPUTS * 4), *red2 = red + RG * 64;
    const int t = threadIdx.x, ch = t % CH, rg = t / CH;
    const int split = (int)(id % (unsigned)a.out_splits), c0 = (int)(id / (unsigned)a.out_splits) * 64;
    const int64_t per = (a.Bp / 64 + a.out_splits - 1) / a.out_splits * 64, b0 = split * per, b1 = min((int64_t)a.Bp, b0 + per);
    constexpr int OW = 8;                                    // outputs at a time (more would crowd the registers)
    for (int w0 = 0; w0 < a.n_out; w0 += OW) {
        float acc[OW][E];
#pragma unroll
        for (int w = 0; w < OW; ++w)
#pragma unroll
            for (int e = 0; e < E; ++e) acc[w][e] = 0.f;
        for (int64_t b = b0; b < b1; b += CHUNK) {               // (rows of the padding are zeros)
            const int rows = (int)min((int64_t)CHUNK, b1 - b);
            i32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = rg + RG * i < rows ? rg + RG * i : 0;
                v[i] = *(const i32x4 *)((const unsigned char *)a.h_last + ((b + row) * a.H_last + c0 + ch * E) * ES);
            }
            __syncthreads();
            for (int i = t; i < CHUNK * a.n_out; i += 256) dout_s[i] = i < rows * a.n_out ? a.dout[b * a.n_out + i] : 0.f;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float hv[E];
                if constexpr (ES == 2) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        hv[2 * q] = __uint_as_float((uint32_t)v[i][q] << 16);
                        hv[2 * q + 1] = __uint_as_float((uint32_t)v[i][q] & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) hv[q] = __uint_as_float((uint32_t)v[i][q]);
                }
#pragma unroll
                for (int w = 0; w < OW; ++w)
                    if (w0 + w < a.n_out) {
                        const float dv = dout_s[(rg + RG * i) * a.n_out + w0 + w];
#pragma unroll
                        for (int e = 0; e < E; ++e) acc[w][e] = fmaf(dv, hv[e], acc[w][e]);
                    }
            }
        }
#pragma unroll
        for (int w = 0; w < OW; ++w) {
            if (w0 + w < a.n_out) {
#pragma unroll
                for (int e = 0; e < E; ++e) red[rg * 64 + ch * E + e] = acc[w][e];
                __syncthreads();
                float s = 0.f;
#pragma unroll
                for (int q = 0; q < RG / 4; ++q) s += red[((t >> 6) * (RG / 4) + q) * 64 + (t & 63)];
                red2[t] = s;
                __syncthreads();
                if (t < 64) a.gw_out[((int64_t)split * a.n_out + w0 + w) * a.H_last + c0 + t] = (red2[t] + red2[64 + t]) + (red2[128 + t] + red2[192 + t]);
            }
        }
    }
}

template <typename T, int W>
__global__ __launch_bounds__(256, W == 128 ? 2 : 3) void update_grads_kernel(const GradsArgs a)
{
    touch_arguments<sizeof(GradsArgs)>();
    constexpr int ES = sizeof(T), ROWB = W * ES, BK = 8192 / ROWB, ST = W == 128 ? 4 : 3, STAGE = 16384, MB = W / 64;
    __shared__ __attribute__((aligned(16))) unsigned char smem[ST * STAGE];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    unsigned id = blockIdx.x;
    if (id < a.n_out_blocks) {
        output_gradient<T>(a, id, smem);
        return;
    }
    id -= a.n_out_blocks;
    if (id < (unsigned)a.n_out + 1) {                        // output bias gradients and the loss
        const int w = (int)id;
        float v = 0.f;
        if (w < a.n_out) {
#pragma unroll 8
            for (int64_t b = t; b < a.B; b += 256) v += a.dout[b * a.n_out + w];
        } else {
#pragma unroll 8
            for (int64_t b = t; b < a.B; b += 256) v += a.lossrow[b];
        }
        v = wave_sum(v);
        float *red = (float *)smem;
        if (lane == 0) red[wave] = v;
        __syncthreads();
        if (t == 0) {
            const float s = (red[0] + red[1]) + (red[2] + red[3]);
            if (w < a.n_out) a.gb_out[w] = s;
            else if (a.loss_out) a.loss_out[0] = s / (float)a.B;
        }
        return;
    }
    id -= (unsigned)a.n_out + 1;

    // ---- a W x W tile of one layer's weight gradient, one share of the batch
    const int split = (int)(id % (unsigned)a.splits);
    int tile = (int)(id / (unsigned)a.splits), k = 0;
    while (k + 1 < a.n && tile >= a.l[k + 1].start) ++k;
    tile -= a.l[k].start;
    const int H = a.l[k].H, in_w = a.l[k].in_w, tiles_n = (in_w + W - 1) / W, tm = tile / tiles_n, tn = tile - tm * tiles_n;
    const int slabs = (int)(a.Bp / BK), s0 = (int)((int64_t)slabs * split / a.splits), s1 = (int)((int64_t)slabs * (split + 1) / a.splits);

    // DMA: wavefront w brings 1 KB pieces 2 w, 2 w + 1 of both operands.  bf16: chunk c of row r sits at c ^ 2 (r & 3); fp32:
    // odd rows have their 128-byte halves exchanged.  Columns past the matrix (a width that is an odd multiple of 64) read
    // the tile's first columns and are not stored.
    auto chunk = [](int row, int c) { return ES == 2 ? c ^ ((row & 3) << 1) : c ^ ((row & 1) << 3); };
    const unsigned char *pa = (const unsigned char *)a.l[k].d + tm * ROWB, *pb = (const unsigned char *)a.l[k].h_in + tn * ROWB;
    const int ch_a = (H - tm * W) * ES / 16, ch_b = (in_w - tn * W) * ES / 16;
    uint32_t off_a[2], off_b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave * 2 + i) * (1024 / ROWB) + lane / (ROWB / 16), c = chunk(row, lane & (ROWB / 16 - 1));
        off_a[i] = (uint32_t)(row * H * ES + (c < ch_a ? c : 0) * 16);
        off_b[i] = (uint32_t)(row * in_w * ES + (c < ch_b ? c : 0) * 16);
    }
    auto fetch = [&](int slab, int stage) {
        if (slab > s1 - 1) slab = s1 - 1;                    // (past the end: the last one again, nobody reads it)
        const int64_t b = (int64_t)slab * BK;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dma16<false>(pa + b * H * ES + off_a[i], smem + stage * STAGE + (wave * 2 + i) * 1024);
            dma16<false>(pb + b * in_w * ES + off_b[i], smem + stage * STAGE + 8192 + (wave * 2 + i) * 1024);
        }
    };
    f32x16 acc[MB][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
    constexpr int BE = 16 / ES, BCH = W / BE;                // bias sums: columns a thread, chunks a row
    float bsum[BE];
#pragma unroll
    for (int e = 0; e < BE; ++e) bsum[e] = 0.f;
    const int wm = wave >> 1, wn = wave & 1, l31 = lane & 31, half = lane >> 5;
    int o_a[MB], o_b[MB];                                    // this lane's place in a slab (first K step), per block of 32 columns
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (ES == 2) {
            const int q = lane & 15, sub = (lane >> 4) & 1, row = 8 * half + (q >> 2), in = sub * 2 + ((q & 3) >> 1);
            o_a[i] = row * ROWB + (chunk(row, (wm * (W / 2) + i * 32) / 8 + in) << 4) + (q & 1) * 8;
            o_b[i] = row * ROWB + (chunk(row, (wn * (W / 2) + i * 32) / 8 + in) << 4) + (q & 1) * 8;
        } else {
            o_a[i] = half * ROWB + (chunk(half, (wm * (W / 2) + i * 32 + l31) / 4) << 4) + (l31 & 3) * 4;
            o_b[i] = half * ROWB + (chunk(half, (wn * (W / 2) + i * 32 + l31) / 4) << 4) + (l31 & 3) * 4;
        }
    }
    if (s0 < s1) {
#pragma unroll
        for (int i = 0; i < ST - 1; ++i) fetch(s0 + i, i);
        for (int s = s0, stage = 0; s < s1; ++s) {
            if constexpr (ST == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else                   asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();                    // slab s is there for everybody, slab s - 1 is done with
            fetch(s + ST - 1, stage == 0 ? ST - 1 : stage - 1);
            const unsigned char *sa = smem + stage * STAGE, *sb = sa + 8192;
            if constexpr (ES == 2) {
                // sixteen reads a slab: K steps 2 q and 2 q + 1 of a block of 32 columns are the four of one address
                constexpr int KQ = BK / 32;
                static_assert(KQ * MB == 2, "four addresses a slab");
                uint2 f[4][4];
                const unsigned char *p[4];
#pragma unroll
                for (int q = 0; q < KQ; ++q)
#pragma unroll
                    for (int i = 0; i < MB; ++i) {
                        p[q * MB + i] = sa + o_a[i] + q * 32 * ROWB;
                        p[2 + q * MB + i] = sb + o_b[i] + q * 32 * ROWB;
                    }
                lds_read_tr_4x4<ROWB>(f, p);
#pragma unroll
                for (int ks = 0; ks < 2 * KQ; ++ks)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < MB; ++j) {
                            const uint2 *fa = f[(ks >> 1) * MB + i] + 2 * (ks & 1), *fb = f[2 + (ks >> 1) * MB + j] + 2 * (ks & 1);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, join(fa[0], fa[1])),
                                                                                __builtin_bit_cast(bf16x8, join(fb[0], fb[1])), acc[i][j], 0, 0, 0);
                        }
            } else {
#pragma unroll
                for (int ks = 0; ks < BK / 2; ++ks) {
                    float fa[MB], fb[MB];
#pragma unroll
                    for (int i = 0; i < MB; ++i) {
                        fa[i] = *(const float *)(sa + o_a[i] + ks * 2 * ROWB);
                        fb[i] = *(const float *)(sb + o_b[i] + ks * 2 * ROWB);
                    }
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < MB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
                }
            }
            if (tn == 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int row = t / BCH + i * (BK / 2);
                    const i32x4 v = *(const i32x4 *)(sa + row * ROWB + (chunk(row, t % BCH) << 4));
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if constexpr (ES == 2) {
                            bsum[2 * q] += __uint_as_float((uint32_t)v[q] << 16);
                            bsum[2 * q + 1] += __uint_as_float((uint32_t)v[q] & 0xffff0000u);
                        } else bsum[q] += __uint_as_float((uint32_t)v[q]);
                    }
                }
            }
            stage = stage == ST - 1 ? 0 : stage + 1;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    float *gw = a.l[k].gw + (int64_t)split * H * in_w;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int col = tn * W + wn * (W / 2) + j * 32 + l31;
        if (MB > 1 && col >= in_w) continue;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int row0 = tm * W + wm * (W / 2) + i * 32;
            if (MB > 1 && row0 >= H) continue;
#pragma unroll
            for (int q = 0; q < 16; ++q) gw[(int64_t)(row0 + 8 * (q >> 2) + 4 * half + (q & 3)) * in_w + col] = acc[i][j][q];
        }
    }
    if (tn == 0) {
        __syncthreads();
        float *red = (float *)smem;                          // [row group][W columns]
#pragma unroll
        for (int e = 0; e < BE; ++e) red[(t / BCH) * W + (t % BCH) * BE + e] = bsum[e];
        __syncthreads();
        if (t < W && tm * W + t < H) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 256 / BCH; ++q) s += red[q * W + t];
            a.l[k].gb[(int64_t)split * H + tm * W + t] = s;
        }
    }
}

hipError_t launch_update_grads(int dtype, int tile, const GradsArgs &a, hipStream_t st)
{
    const unsigned blocks = a.n_out_blocks + (unsigned)a.n_out + 1 + a.n_tile_blocks;
    if (dtype == AB_BF16) {
        if (tile == 128) update_grads_kernel<bf16_t, 128><<<blocks, 256, 0, st>>>(a);
        else             update_grads_kernel<bf16_t, 64><<<blocks, 256, 0, st>>>(a);
    } else {
        if (tile == 128) update_grads_kernel<float, 128><<<blocks, 256, 0, st>>>(a);
        else             update_grads_kernel<float, 64><<<blocks, 256, 0, st>>>(a);
    }
    return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------
// Gradients and Adam in one launch: a work-group of eight wavefronts owns a tile of one weight matrix (128 bytes of the
// compute type wide and as many rows: 64 x 64 in bf16, 32 x 32 in fp32) over the whole batch, and takes the Adam step for it.
// The wavefronts share the batch, a share each: private rings of two 8 KB slabs (32 batch rows of both operands) by DMA, no
// barrier before the partial tiles meet in LDS, in share order.  Against the split launch above it saves the partial sums'
// way through memory (eight copies of every gradient written and read again) and a launch.
// By kernel time, 390-512-512-512-1 in bf16: 64 rows 9.2 us (the rest of a large batch's time: old values in, partial tiles
// together, Adam, out), 1000 rows 12.2, 4096 22.2, i.e. 3.2 us a thousand rows: 35 bytes a clock and CU, each of them into
// LDS and out again (gradients and Adam as two launches: 4096 rows 17.6 + 9.5).  The output unit's work-groups: one output 4.2
// us for 64 rows, 11.7 for 4096; eight 6.0 and 14.3.
// ---------------------------------------------------------------------------------------------
struct AdamRates { float lr, beta1, beta2, eps, c1, c2; };
template <typename T>
__device__ __forceinline__ void adam_store(const AdamTensor &t, const AdamRates &r, int64_t e, float g, float m, float v, float w)
{
    m = r.beta1 * m + (1.f - r.beta1) * g;
    v = r.beta2 * v + (1.f - r.beta2) * g * g;
    w = w - r.lr * (m / r.c1) / (sqrtf(v / r.c2) + r.eps);
    t.m[e] = m;
    t.v[e] = v;
    t.w[e] = w;
    if (t.wc) {
        if constexpr (sizeof(T) == 2) ((uint16_t *)t.wc)[e] = (uint16_t)(pack_bf16x2(w, 0.f) & 0xffffu);
        else ((float *)t.wc)[e] = w;
    }
}

// The output unit's weights: sixteen columns of all its rows, on the vector ALUs (its deltas are fp32).  A wavefront takes an
// eighth of the batch, a lane every RG-th row of it and 16 bytes of columns; the deltas come by DMA (as per-lane loads they kept
// the address units busy: 4096 rows, eight outputs 28 us), the next piece of both under the sums.  OW: outputs at a time.
template <typename T, int OW>
__device__ __forceinline__ void output_step(const StepArgs &a, const AdamRates &rt, unsigned id, unsigned char *smem)
{
    constexpr int ES = sizeof(T), E = 16 / ES, CH = 16 / E, RG = 64 / CH, U = OW == 1 ? 8 : 4, ROWS = RG * U;
    constexpr int STAGE = OW == 1 ? 1024 : ROWS * AB_MAX_OUTPUTS * 4;     // staged deltas, whole requests of 1 KB
    static_assert(STAGE >= ROWS * OW * 4 && STAGE % 1024 == 0, "a piece's deltas fit");
    const int t = threadIdx.x, lane = t & 63, ch = lane % CH, rg = lane / CH, c0 = (int)id * 16;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), n_out = OW == 1 ? 1 : a.n_out;
    unsigned char *stage = smem + wave * (2 * STAGE);
    float *red = (float *)(smem + 8 * (2 * STAGE));          // [512]
    const int64_t r0 = a.Bp / 8 * wave, r1 = r0 + a.Bp / 8;              // (rows of the padding are zeros on both sides)
    const unsigned char *src = (const unsigned char *)a.h_last + (c0 + ch * E) * ES;
    const int64_t pitch = (int64_t)a.H_last * ES, last = a.Bp * n_out * 4 - 16;
    for (int w0 = 0; w0 < n_out; w0 += OW) {
        // the old values of what this thread will step (outputs w0 + t / 16, column t & 15), under the sums
        const int mw = w0 + (t >> 4);
        const bool mine = t < OW * 16 && mw < n_out;
        const int64_t e = mine ? (int64_t)mw * a.H_last + c0 + (t & 15) : 0;
        const float m0 = a.Wo.m[e], v0 = a.Wo.v[e], x0 = a.Wo.w[e];
        float acc[OW][E];
#pragma unroll
        for (int w = 0; w < OW; ++w)
#pragma unroll
            for (int q = 0; q < E; ++q) acc[w][q] = 0.f;
        i32x4 h[U];
        auto load = [&](int set, int64_t b) {                // (past the batch: its last row, whose sums are not taken)
            unsigned char *to = stage + set * STAGE;
            for (int o = 0; o < ROWS * n_out * 4; o += 1024)
                dma16<false>((const unsigned char *)a.dout + min(b * n_out * 4 + o + lane * 16, last), to + o);
#pragma unroll
            for (int i = 0; i < U; ++i) h[i] = *(const i32x4 *)(src + min(b + rg + RG * i, a.Bp - 1) * pitch);
        };
        load(0, r0);
        int set = 0;
        for (int64_t b = r0; b < r1; b += ROWS, set ^= 1) {
            i32x4 g[U];
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");      // this piece is there, the one before it read: its room is refilled
#pragma unroll
            for (int i = 0; i < U; ++i) g[i] = b + rg + RG * i < r1 ? h[i] : i32x4{0, 0, 0, 0};      // (other shares' rows: an infinity times zero is NaN)
            if (b + ROWS < r1) load(set ^ 1, b + ROWS);
            const float *dl = (const float *)(stage + set * STAGE);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                float hv[E];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (ES == 2) {
                        hv[2 * q] = __uint_as_float((uint32_t)g[i][q] << 16);
                        hv[2 * q + 1] = __uint_as_float((uint32_t)g[i][q] & 0xffff0000u);
                    } else hv[q] = __uint_as_float((uint32_t)g[i][q]);
                }
                const bool in = b + rg + RG * i < r1;
#pragma unroll
                for (int w = 0; w < OW; ++w) {
                    const float d = dl[(rg + RG * i) * n_out + min(w0 + w, n_out - 1)], dv = in ? d : 0.f;
#pragma unroll
                    for (int q = 0; q < E; ++q) acc[w][q] = fmaf(dv, hv[q], acc[w][q]);
                }
            }
        }
        // the lanes' sums meet in LDS (each wavefront's where its deltas were: rows of OW x 16, 16-byte chunk c of row r at
        // c ^ r), are added in PARTS runs of rows, then over the runs
        constexpr int NC = OW * 4, PARTS = 512 / (OW * 16);
        auto at = [](int r, int c) { return r * (NC * 16) + ((c ^ (r & (NC - 1))) << 4); };
        static_assert(RG * NC * 16 <= 2 * STAGE, "a wavefront's sums fit its deltas' room");
#pragma unroll
        for (int w = 0; w < OW; ++w)
#pragma unroll
            for (int q = 0; q < E / 4; ++q)
                *(f32x4 *)(stage + at(rg, w * 4 + ch * (E / 4) + q)) = f32x4{acc[w][4 * q], acc[w][4 * q + 1], acc[w][4 * q + 2], acc[w][4 * q + 3]};
        __syncthreads();
        {
            const int v = t % (OW * 16), p = t / (OW * 16);
            float s[4] = {0.f, 0.f, 0.f, 0.f};               // (four chains: less rounding than one)
#pragma unroll
            for (int i = 0; i < 8 * RG / PARTS; ++i) {
                const int r = p * (8 * RG / PARTS) + i;
                s[i & 3] += *(const float *)(smem + (r / RG) * (2 * STAGE) + at(r % RG, v >> 2) + (v & 3) * 4);
            }
            red[t] = (s[0] + s[1]) + (s[2] + s[3]);
        }
        __syncthreads();
        if (mine) {
            float g[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < PARTS; ++q) g[q & 3] += red[q * OW * 16 + t];
            adam_store<T>(a.Wo, rt, e, (g[0] + g[1]) + (g[2] + g[3]), m0, v0, x0);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(512) void update_step_kernel(const StepArgs a)
{
    constexpr int ES = sizeof(T), W = 128 / ES, MB = W / 32, BK = 32, SLAB = 8192, RING = 2 * SLAB;
    constexpr int EPT = W * W / 512;                        // elements of the tile a thread steps
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, l31 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    touch_arguments<sizeof(StepArgs)>();
    const AdamRates rt{a.lr, a.beta1, a.beta2, a.eps, a.scal[0], a.scal[1]};
    unsigned id = blockIdx.x;
    if (id < a.n_out_blocks) {
        if (a.n_out == 1) output_step<T, 1>(a, rt, id, smem);
        else              output_step<T, 8>(a, rt, id, smem);
        return;
    }
    id -= a.n_out_blocks;
    if (id < (unsigned)a.n_out + 1) {                        // the output unit's biases and the loss
        const int w = (int)id;
        float v = 0.f;
        if (w < a.n_out) {
#pragma unroll 8
            for (int64_t b = t; b < a.B; b += 512) v += a.dout[b * a.n_out + w];
        } else {
#pragma unroll 8
            for (int64_t b = t; b < a.B; b += 512) v += a.lossrow[b];
        }
        v = wave_sum(v);
        float *red = (float *)smem;
        if (lane == 0) red[wave] = v;
        __syncthreads();
        if (t == 0) {
            const float s = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
            if (w < a.n_out) adam_store<T>(a.bo, rt, w, s, a.bo.m[w], a.bo.v[w], a.bo.w[w]);
            else if (a.loss_out) a.loss_out[0] = s / (float)a.B;
        }
        return;
    }
    id -= (unsigned)a.n_out + 1;

    // ---- tiles: each XCD takes a run of neighbours (they share panels of deltas and inputs in its L2)
    const int per = (a.n_tiles + 7) / 8, local = (int)(id >> 3);
    int tile = (int)(id & 7) * per + local, k = 0;
    if (tile >= a.n_tiles) return;
    while (k + 1 < a.n && tile >= a.l[k + 1].start) ++k;
    tile -= a.l[k].start;
    const int H = a.l[k].H, in_w = a.l[k].in_w, cols = a.l[k].cols, tiles_n = in_w / W, tm = tile / tiles_n, tn = tile - tm * tiles_n;
    const int slabs = (int)(a.Bp / BK), s0 = slabs * wave / 8, s1 = slabs * (wave + 1) / 8;

    // the old values of this thread's elements (rows i * 512 / W + t / W, column t % W), under the products
    const AdamTensor tw = a.l[k].W;
    const int col = tn * W + t % W, e0 = (tm * W + t / W) * cols + col;
    float om[EPT], ov[EPT], ow[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = col < cols ? e0 + i * (512 / W) * cols : 0;
        om[i] = tw.m[e]; ov[i] = tw.v[e]; ow[i] = tw.w[e];
    }

    // DMA: four requests of eight rows an operand; bf16: chunk c of row r sits at c ^ 2 (r & 3) (the transposing reads take four
    // rows x 32 bytes at a time), fp32: rows as they are
    auto chunk = [](int row, int c) { return ES == 2 ? c ^ ((row & 3) << 1) : c; };
    unsigned char *ring = smem + wave * RING;
    const unsigned char *pa = (const unsigned char *)a.l[k].d + tm * 128, *pb = (const unsigned char *)a.l[k].h_in + tn * 128;
    const uint32_t lda = H * ES, ldb = in_w * ES, c16 = chunk(lane >> 3, lane & 7) * 16;      // (8 i rows on: the same chunk)
    const uint32_t off_a = (lane >> 3) * lda + c16, off_b = (lane >> 3) * ldb + c16;
    auto fetch = [&](int slab, int slot) {
        if (slab > s1 - 1) slab = s1 - 1;                    // (past the end: the last one again, nobody reads it)
        const unsigned char *qa = pa + (int64_t)slab * BK * lda, *qb = pb + (int64_t)slab * BK * ldb;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dma16<false>(qa + off_a + i * 8 * lda, ring + slot * SLAB + i * 1024);
            dma16<false>(qb + off_b + i * 8 * ldb, ring + slot * SLAB + 4096 + i * 1024);
        }
    };
    f32x16 acc[MB][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
    f32x16 bacc[MB];                                         // bias sums of layer's first column tiles: every column the same
    float bsum = 0.f;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q) bacc[i][q] = 0.f;
    int o_f[MB];                                             // this lane's place in an operand's slab, per block of 32 columns
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (ES == 2) {
            const int q = lane & 15, sub = (lane >> 4) & 1, row = 8 * half + (q >> 2), in = sub * 2 + ((q & 3) >> 1);
            o_f[i] = row * 128 + (chunk(row, i * 4 + in) << 4) + (q & 1) * 8;
        } else o_f[i] = half * 128 + l31 * 4;
    }
    if (s0 < s1) {
        fetch(s0, 0);
        fetch(s0 + 1, 1);
        for (int s = s0, slot = 0; s < s1; ++s, slot ^= 1) {
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            const unsigned char *sa = ring + slot * SLAB, *sb = sa + 4096;
            if constexpr (ES == 2) {
                uint2 f[4][4];
                const unsigned char *p[4] = {sa + o_f[0], sa + o_f[MB - 1], sb + o_f[0], sb + o_f[MB - 1]};
                lds_read_tr_4x4<128>(f, p);
                fetch(s + 2, slot);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < MB; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, join(f[i][2 * ks], f[i][2 * ks + 1])),
                                                                                __builtin_bit_cast(bf16x8, join(f[2 + j][2 * ks], f[2 + j][2 * ks + 1])),
                                                                                acc[i][j], 0, 0, 0);
                if (tn == 0) {                               // bias sums: the same product with ones
                    const bf16x8 ones = __builtin_bit_cast(bf16x8, i32x4{0x3f803f80, 0x3f803f80, 0x3f803f80, 0x3f803f80});
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int i = 0; i < MB; ++i)
                            bacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, join(f[i][2 * ks], f[i][2 * ks + 1])), ones, bacc[i], 0, 0, 0);
                }
            } else {
                float fa[BK / 2], fb[BK / 2];
#pragma unroll
                for (int ks = 0; ks < BK / 2; ++ks) {
                    fa[ks] = *(const float *)(sa + o_f[0] + ks * 256);
                    fb[ks] = *(const float *)(sb + o_f[0] + ks * 256);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                fetch(s + 2, slot);
#pragma unroll
                for (int ks = 0; ks < BK / 2; ++ks) {
                    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[ks], fb[ks], acc[0][0], 0, 0, 0);
                    if (tn == 0) bsum += fa[ks];             // (this lane's column, the rows of its half)
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // nothing is on its way into the ring
    // partial tiles, a wavefront's in its own ring: column c of row r at c, in bf16 tiles c ^ 32 in rows with bit 2 set (the two
    // halves of a wavefront write rows four apart)
    auto at = [&](int q, int r, int c) { return (float *)(smem + q * RING) + r * W + (W == 64 ? c ^ ((r & 4) << 3) : c); };
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) *at(wave, i * 32 + 8 * (q >> 2) + 4 * half + (q & 3), j * 32 + l31) = acc[i][j][q];
    float *bred = (float *)(smem + 8 * RING);                // [wavefront][half (fp32)][W]
    if (tn == 0) {
        if constexpr (ES == 2) {
            if (l31 == 0) {
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int q = 0; q < 16; ++q) bred[wave * W + i * 32 + 8 * (q >> 2) + 4 * half + (q & 3)] = bacc[i][q];
            }
        } else bred[(wave * 2 + half) * W + l31] = bsum;
    }
    __syncthreads();
    if (col < cols) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            float g = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) g += *at(q, i * (512 / W) + t / W, t % W);
            adam_store<T>(tw, rt, e0 + i * (512 / W) * cols, g, om[i], ov[i], ow[i]);
        }
    }
    if (tn == 0 && t < W) {
        const AdamTensor &tb = a.l[k].b;
        const int e = tm * W + t;
        float g = 0.f;
#pragma unroll
        for (int q = 0; q < (ES == 2 ? 8 : 16); ++q) g += bred[q * W + t];
        adam_store<T>(tb, rt, e, g, tb.m[e], tb.v[e], tb.w[e]);
    }
}

hipError_t launch_update_step(int dtype, const StepArgs &a, hipStream_t st)
{
    constexpr int smem = 8 * 16384 + 4096;                   // rings, bias sums (or the output unit's)
    auto kb = update_step_kernel<bf16_t>;
    auto kf = update_step_kernel<float>;
    static DeviceOnce once_b, once_f;
    const hipError_t e = dtype == AB_BF16 ? ensure_dynamic_lds((const void *)kb, smem, once_b) : ensure_dynamic_lds((const void *)kf, smem, once_f);
    if (e != hipSuccess) return e;
    const unsigned blocks = a.n_out_blocks + (unsigned)a.n_out + 1 + (unsigned)(a.n_tiles + 7) / 8 * 8;
    if (dtype == AB_BF16) kb<<<blocks, 512, smem, st>>>(a);
    else                  kf<<<blocks, 512, smem, st>>>(a);
    return hipGetLastError();
}

}  // namespace ab
