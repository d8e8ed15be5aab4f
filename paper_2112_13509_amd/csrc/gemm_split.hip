// fp32 products on the bf16 matrix cores: both operands in three bf16 parts, six partial products, two accumulators.  The
// parts and partial products are those of Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype
// for higher-precision computations" (ARITH 2019); the second accumulator, the shape and the repair below are this file's.
//
// An fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significant bits, each part the round-to-nearest of
// what the parts before leave), and a product of two bf16 values is exact in fp32.  Of the nine partial products the
// six that matter are taken: a0 w0 into one accumulator, a0 w1, a1 w0, a0 w2, a1 w1, a2 w0 into a second one that is
// added at the end; the other three lie below 2^-24 of a term.  The second accumulator is what keeps the error down:
// the large one is rounded once per sixteen summed indices, where the fp32 instruction rounds it at every index.
// Relative error against fp64 (2-norm, ReLU'd normal activations, 256 columns): K = 64 / 256 / 1024 4.1e-8 / 7.1e-8 /
// 1.4e-7, the fp32 instruction 1.06e-7 / 2.1e-7 / 4.1e-7; with one accumulator for all six 1.3e-7 / 2.5e-7 / 4.7e-7.
//
// What bounds it: the matrix pipe at a power-limited clock, and beside it the vector work of splitting.  Six bf16 instructions of 32
// cycles do the work of eight fp32 ones of 64 cycles.  4.2 M rows x 256 x 256 with generated operand and fused output unit, in four
// launches: 1.15 ms a launch on the fp32 instruction (76 % of its peak); the whole call 2.60 ms with the weights split in each
// work-group, 2.42 with weights that lie split (PARTS), 2.38 so on tiles of 256 columns; six bf16 products of that size 2.23 at the
// rate of the large bf16 kernels.
//
// Shape: a work-group of 256 threads (2 x 2 wavefronts) owns 128 rows and walks its column tiles of BN columns, K in
// slabs of 16.  A wavefront's 64 x BN/2 outputs take 128 accumulator registers with both sets, so two wavefronts fit a
// SIMD: two work-groups share a CU, and one's LDS latencies, barriers and epilogues run under the other's matrix work.
//
// Split weights (PARTS, where the pass has room for them: split_parts.hpp, made once a pass by its first launch) come by DMA, a slab
// ahead, in the order in which LDS holds them.  All of a wavefront's requests are waited for at the end of the slab that makes
// them, which is where the next slab wants them; waiting for the DMA alone would leave the compiler to wait for the activations in
// the next slab, which it does for everything in flight.  2 x 4 wavefronts on 256 columns split each activation once where 2 x 2 on two
// tiles of 128 do it twice; on 64 x 256 (1 x 4, two work-groups a CU) the weights' traffic into LDS doubles: 2.53 ms.
// The vector work of a slab (operand generation, splitting) is spread over its matrix instructions, five between two (1.30 M cycles
// a launch; in one piece a fifth more); with PARTS, where the activations alone are split, three, in the larger work-group two.  LDS: two stages; a stage holds, per operand, part and half of the
// slab's sixteen k, 16 bytes per row one row after the other: a thread writes the eight k it has split and a fragment
// is one 16-byte read, both over consecutive addresses (no bank conflicts, no swizzle).  Slab j + 1's raw values are in
// registers while slab j is multiplied; where the work-group splits its weights, slab j + 2's are on their way across the barrier
// (requested only half a slab ahead: 5 % slower).
// A third stage, with the next slab's first fragments read in front of the barrier, was 5 % slower again.
//
// Infinities: inf splits into (inf, NaN, NaN), so a row that holds one has a NaN in the second accumulator where fp32 arithmetic
// may give an infinity.  The first one, a0 w0, has by itself what fp32 arithmetic gives for a row with an infinity or a NaN in it
// (a part a0 or w0 is infinite, NaN or zero where the value is), so a wavefront that finds a NaN or an infinity among its sums
// looks through those rows, which ends with the first chunk as a rule, and takes the first accumulator.  Where a row holds
// neither (its columns do, or a value or a product close to fp32's largest, which its parts round beyond), the tile is
// computed again with the fp32 instruction, operands straight from memory.  So is a tile with rows of tiny sums: the third part
// of a value below 2^-109 has bits below bf16's smallest (activations of 1e-36: error 2e-5 without this).  1024 scenarios x 4096 candidates, 256-256, every
// scenario with a NaN or an infinity: 2.53 -> 2.30 ms a call (7.15 with all such tiles computed again, one scenario in 64 like that 2.62).
#include "stream_util.hpp"
#include "split_parts.hpp"
#include <type_traits>

namespace ab {

template <int AMODE, int EPI, int WM, int WN, int JN, bool PARTS>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_split_kernel(const GemmArgs g)
{
    touch_arguments<sizeof(GemmArgs)>();
    constexpr int NW = WM * WN, NT = 64 * NW, BM = 64 * WM, BN = 32 * JN * WN, BK = 16;
    constexpr int AE = BM * BK / NT;                       // activations a thread splits per slab (8 or 4)
    constexpr int WE = PARTS ? 4 : BN * BK / NT;           // weights a thread splits per slab (8 or 4), unless they lie split
    constexpr int W_REQ = 6 * BN / 64, W_MINE = (W_REQ + NW - 1) / NW;     // a slab's KB of split weights, a wavefront's
    constexpr int A_PLANE = BM * 16, W_PLANE = BN * 16;    // one part, one half of the slab's k
    constexpr int W_BASE = 6 * A_PLANE, STAGE = 6 * (A_PLANE + W_PLANE);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // column groups of one row panel stay on one XCD (they share the activations)
    const int64_t local = blockIdx.x >> 3;
    const int tn = (int)(local % g.n_tiles);
    const int64_t tm = (local / g.n_tiles) * 8 + (blockIdx.x & 7);
    if (tm >= g.m_tiles) return;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wave_m = wave / WN, wave_n = wave % WN, half = lane >> 5, l31 = lane & 31;
    const int64_t m0 = tm * BM;
    const int KT = g.K / BK, n_first = tn * g.n_loop * BN;

    // ---- this thread's share of a slab: AE k of one activation row, WE k of one weight row
    const int a_row = t & (BM - 1), a_part = wave * 64 / BM;                   // which AE of the sixteen k
    const int w_row = t & (BN - 1), w_part = wave * 64 / BN;                   // which WE of the sixteen k
    const int64_t gr = min(m0 + a_row, g.M - 1);
    const float *a_src;
    float xp = 0.f, xc = 0.f;
    if constexpr (AMODE == AMODE_LOAD) {
        a_src = (const float *)g.A + gr * g.lda + a_part * AE;
    } else {
        const int64_t s = gr / g.C, x = g.x_per_row ? gr : gr - s * g.C;
        a_src = g.a_term + s * g.ldt + a_part * AE;
        xp = g.xp[x];
        xc = g.xc[x];
    }
    const float *w_src = (const float *)g.B + (int64_t)(n_first + w_row) * g.ldb + w_part * WE;
    f32x4 ra[2][AE / 4], rw[2][WE / 4];                    // two sets: requested a slab ahead (rw, w_src: not with PARTS)
    typedef float vec_u __attribute__((ext_vector_type(AE), aligned(4)));
    typedef __attribute__((address_space(4))) vec_u const_vec;
    vec_u rp[2], rc[2];                                    // wp, wc of the slab: the same for the whole wavefront
    const unsigned char *w_img = nullptr;                  // PARTS: the slab that is requested next,
    if constexpr (PARTS) w_img = (const unsigned char *)g.B_parts + (int64_t)(n_first / BN) * KT * (6 * W_PLANE) + lane * 16;
    int w_left = g.n_loop * KT;                            // slabs from there on
    auto request_parts = [&](unsigned char *stage) {
#pragma unroll
        for (int i = 0; i < W_MINE; ++i) {
            const int r = W_REQ % NW == 0 || i < W_REQ / NW ? i * NW + wave : i * NW + wave % (W_REQ % NW);   // (a remainder: some twice)
            dma16<false>(w_img + r * 1024, stage + W_BASE + r * 1024);
        }
        if (--w_left > 0) w_img += 6 * W_PLANE;            // (behind the last slab: that one again, not used)
    };
    int ld_k = 0, ld_n = 0;                                // the slab that is requested next: its k, its column tile
    auto request = [&](int set) {
#pragma unroll
        for (int i = 0; i < AE / 4; ++i) ra[set][i] = *(const f32x4 *)(a_src + ld_k + 4 * i);
#pragma unroll
        for (int i = 0; i < (PARTS ? 0 : WE / 4); ++i) rw[set][i] = *(const f32x4 *)(w_src + ld_k + 4 * i);
    };
    auto request_vectors = [&](int set) {                  // ... and wp, wc by scalar loads; then on to the slab after it
        if constexpr (AMODE != AMODE_LOAD) {
            rp[set] = *(const const_vec *)(uintptr_t)(g.wp + ld_k + a_part * AE);
            rc[set] = *(const const_vec *)(uintptr_t)(g.wc + ld_k + a_part * AE);
        }
        ld_k += BK;
        if (ld_k == g.K) {                                 // (behind the last column tile: that one again, not used)
            ld_k = 0;
            if (!PARTS && ++ld_n < g.n_loop) w_src += (int64_t)BN * g.ldb;
        }
    };
    uint32_t pa[4][3], pw[4][3];                           // the split pairs of this thread's shares
    auto split_half = [&](int set, int h) {
#pragma unroll
        for (int e = AE / 4 * h; e < AE / 4 * (h + 1); ++e) {
            float v[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                v[i] = ra[set][e >> 1][2 * (e & 1) + i];
                if constexpr (AMODE != AMODE_LOAD)
                    v[i] = relu_keep_nan(fmaf(rc[set][2 * e + i], xc, fmaf(rp[set][2 * e + i], xp, v[i])));
            }
            split3(v[0], v[1], pa[e]);
            if (!PARTS && e < WE / 2) split3(rw[set][e >> 1][2 * (e & 1)], rw[set][e >> 1][2 * (e & 1) + 1], pw[e]);
        }
    };
    auto write_parts = [&](unsigned char *stage) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if constexpr (PARTS && AE == 8)
                lds_write16(stage + (i * 2 + a_part) * A_PLANE + a_row * 16, i32x4{(int)pa[0][i], (int)pa[1][i], (int)pa[2][i], (int)pa[3][i]});
            else if constexpr (PARTS)
                lds_write8(stage + (i * 2 + (a_part >> 1)) * A_PLANE + a_row * 16 + (a_part & 1) * 8, uint2{pa[0][i], pa[1][i]});
            else
                *(i32x4 *)(stage + (i * 2 + a_part) * A_PLANE + a_row * 16) = i32x4{(int)pa[0][i], (int)pa[1][i], (int)pa[2][i], (int)pa[3][i]};
            if constexpr (PARTS) continue;
            if constexpr (WE == 8)
                *(i32x4 *)(stage + W_BASE + (i * 2 + w_part) * W_PLANE + w_row * 16) = i32x4{(int)pw[0][i], (int)pw[1][i], (int)pw[2][i], (int)pw[3][i]};
            else
                *(uint2 *)(stage + W_BASE + (i * 2 + (w_part >> 1)) * W_PLANE + w_row * 16 + (w_part & 1) * 8) = uint2{pw[0][i], pw[1][i]};
        }
    };

    const int a_rd = half * A_PLANE + (wave_m * 64 + l31) * 16;
    const int w_rd = W_BASE + half * W_PLANE + (wave_n * (32 * JN) + l31) * 16;
    f32x16 big[JN][2], small[JN][2];
    float row_sum[2] = {0.f, 0.f};                         // EPI_SCORE: over this wavefront's columns of all column tiles

    // What leaves a column tile, from `small`: bias, ReLU, and the stored values or the output unit's dot product.
    auto emit = [&](int nw) {
        float sum[2] = {0.f, 0.f};
        int in_panel = wave_m * 64 + l31;
        if constexpr (EPI == EPI_STORE) asm volatile("" : "+v"(in_panel));     // (the rows' addresses are not worth registers in the slab loop)
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int col = nw + j * 32 + rg * 8 + half * 4;
                const f32x4 bv = *(const f32x4_any *)(g.bias + col);     // (biases may lie on any 4 bytes)
                f32x4 wv = {0.f, 0.f, 0.f, 0.f};
                if constexpr (EPI == EPI_SCORE) wv = *(const f32x4 *)(g.w_out + col);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = relu_keep_nan(small[j][i][rg * 4 + e] + bv[e]);
                        if constexpr (EPI == EPI_SCORE) sum[i] = fmaf(v[e], wv[e], sum[i]);
                    }
                    if constexpr (EPI == EPI_STORE) {
                        const int64_t row = m0 + in_panel + i * 32;
                        if (row < g.M) *(f32x4 *)((float *)g.out + row * g.ldo + col) = v;
                    }
                }
            }
        row_sum[0] += sum[0];
        row_sum[1] += sum[1];
    };
    // Sums that are not finite, or tiny, once more (bad: in which of this lane's two rows): the first accumulator where the row's operand holds a NaN
    // or an infinity, or all of the tile anew.
    auto repair = [&](int nw, const bool (&bad)[2]) {
        int ln = lane, C = g.C;
        asm volatile("" : "+v"(ln), "+s"(C));              // (nor is anything of this)
        const float *pa[2];
        float px[2] = {0.f, 0.f}, pc[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t r = min(m0 + wave_m * 64 + i * 32 + (ln & 31), g.M - 1);
            if constexpr (AMODE == AMODE_LOAD) {
                pa[i] = (const float *)g.A + r * g.lda;
            } else {
                const uint32_t s = (uint32_t)r / (uint32_t)C;      // (rows of a chunk: 31 bits)
                const int64_t x = g.x_per_row ? r : r - (int64_t)s * C;
                pa[i] = g.a_term + s * g.ldt;
                px[i] = g.xp[x];
                pc[i] = g.xc[x];
            }
        }
        auto operand = [&](int i, int k) {
            if constexpr (AMODE == AMODE_LOAD) return *(const i32x4 *)(pa[i] + k);
            else return gen_chunk_v<float>(pa[i] + k, g.wp + k, g.wc + k, px[i], pc[i]);
        };
        bool open[2] = {bad[0], bad[1]};                   // rows whose operand has shown neither so far
#pragma unroll 1
        for (int k = (ln >> 5) * 4; k < g.K && __any(open[0] || open[1]); k += 8)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4 v = __builtin_bit_cast(f32x4, operand(i, k));
                bool found = false;
#pragma unroll
                for (int e = 0; e < 4; ++e) found |= !(fabsf(v[e]) < INFINITY);
                const uint64_t m = __ballot(found);        // (lanes 32 apart share a row)
                if ((m | m >> 32 | m << 32) >> ln & 1) open[i] = false;
            }
        if (!__any(open[0] || open[1])) {
#pragma unroll
            for (int j = 0; j < JN; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) small[j][i][r] = bad[i] ? big[j][i][r] : small[j][i][r];
            return;
        }
        const float *pw = (const float *)g.B + (int64_t)(nw + (ln & 31)) * g.ldb;
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) small[j][i][r] = 0.f;
#pragma unroll 1
        for (int k = (ln >> 5) * 4; k < g.K; k += 8) {
            i32x4 fa[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[i] = operand(i, k);
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const i32x4 fw = *(const i32x4 *)(pw + (int64_t)(j * 32) * g.ldb + k);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma_chunk<float>(fw, fa[i], small[j][i]);
            }
        }
    };
    auto epilogue = [&](int n0) {
        const int nw = n0 + wave_n * (32 * JN);
        float worst[2] = {0.f, 0.f};
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    small[j][i][r] += big[j][i][r];
                    small[j][i][r + 1] += big[j][i][r + 1];
                    worst[i] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(worst[i], fabsf(small[j][i][r])), fabsf(small[j][i][r + 1]));
                }
        // (a row's sums all below 2^-80, but not zero: its parts may be below what bf16 holds)
        auto doubtful = [](float v) { return !(v < INFINITY) || (v < 0x1p-80f && v > 0.f); };
        const bool bad[2] = {doubtful(worst[0]), doubtful(worst[1])};
        if (__any(bad[0] || bad[1])) repair(nw, bad);
        emit(nw);
    };

    if constexpr (PARTS) request_parts(smem);
    request(0);
    request_vectors(0);
    request(1);
    request_vectors(1);
    split_half(0, 0);
    split_half(0, 1);
    write_parts(smem);
    if constexpr (PARTS) {
        AB_FENCE();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x70);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        AB_FENCE();
    } else __syncthreads();
    auto slab = [&](auto first_tag, int par) {             // slab j, par = j & 1; a column tile's first one starts the sums
        constexpr bool FIRST = decltype(first_tag)::value;
        const unsigned char *stage = smem + par * STAGE;
        unsigned char *next = smem + (par ^ 1) * STAGE;
        bf16x8 fa[3][2], fw[3][JN];
        auto mma = [&](auto zero_tag, int p, int w, f32x16 (&acc)[JN][2]) {
            f32x16 zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
            for (int jn = 0; jn < JN; ++jn)
#pragma unroll
                for (int im = 0; im < 2; ++im)
                    acc[jn][im] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[w][jn], fa[p][im],
                                                                          decltype(zero_tag)::value ? zero : acc[jn][im], 0, 0, 0);
        };
        const std::integral_constant<bool, FIRST> first{};
        const std::false_type on{};
        AB_FENCE();
        if constexpr (PARTS) request_parts(next);          // slab j + 1
        AB_FENCE();
        request(par);                                      // slab j + 2
        AB_FENCE();
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[p][i] = *(const bf16x8 *)(stage + a_rd + p * 2 * A_PLANE + i * 512);
#pragma unroll
            for (int i = 0; i < JN; ++i) fw[p][i] = *(const bf16x8 *)(stage + w_rd + p * 2 * W_PLANE + i * 512);
        }
        // the vector work goes into the shadows of the matrix instructions
        constexpr int VPM = PARTS ? (AE == 8 ? 3 : 2) : 5;
        auto interleave = [&]() {
#pragma unroll
            for (int i = 0; i < 6 * JN; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        };
        split_half(par ^ 1, 0);                            // slab j + 1 (behind the last: a stage that nobody reads)
        mma(first, 0, 0, big);
        mma(first, 0, 1, small);
        mma(on, 1, 0, small);
        __builtin_amdgcn_sched_group_barrier(0x100, 6 + 3 * JN, 0);
        interleave();
        AB_FENCE();
        request_vectors(par);
        split_half(par ^ 1, 1);
        write_parts(next);
        mma(on, 0, 2, small);
        mma(on, 1, 1, small);
        mma(on, 2, 0, small);
        interleave();
        AB_FENCE();
        if constexpr (AMODE != AMODE_LOAD) asm volatile("" ::"s"(rp[par]), "s"(rc[par]));
        if constexpr (PARTS) {                             // everything: slab j + 1's weights, and slab j + 2's activations with them
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0x70);
            asm volatile("" ::: "memory");
        } else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        AB_FENCE();
    };
    for (int n = 0; n < g.n_loop; ++n) {
        slab(std::true_type{}, 0);
        slab(std::false_type{}, 1);
        for (int kt = 2; kt < KT; kt += 2) { slab(std::false_type{}, 0); slab(std::false_type{}, 1); }   // (K is a multiple of 32)
        epilogue(n_first + n * BN);
    }

    if constexpr (EPI == EPI_SCORE) {
        float *red = (float *)smem;                        // (the last slab ended with a barrier, its successor's stage is this one)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float v = row_sum[i] + __shfl_xor(row_sum[i], 32, 64);
            if (half == 0) red[wave_n * BM + wave_m * 64 + i * 32 + l31] = v;
        }
        __syncthreads();
        if (t < BM && m0 + t < g.M) {
            float sum = red[t];
#pragma unroll
            for (int w = 1; w < WN; ++w) sum += red[w * BM + t];
            g.partial[(m0 + t) * g.n_tiles + tn] = sum;
        }
    }
}

template <int AMODE, int EPI, int WM, int WN, int JN, bool PARTS>
static hipError_t launch_one(const GemmArgs &g, hipStream_t st)
{
    constexpr int smem = 2 * 6 * (64 * WM + 32 * JN * WN) * 16;
    const int64_t blocks = (g.m_tiles + 7) / 8 * 8 * g.n_tiles;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    auto kern = gemm_split_kernel<AMODE, EPI, WM, WN, JN, PARTS>;
    static DeviceOnce once;
    if (smem > 64 * 1024) { const hipError_t e = ensure_dynamic_lds((const void *)kern, smem, once); if (e != hipSuccess) return e; }
    kern<<<(unsigned)blocks, 64 * WM * WN, smem, st>>>(g);
    return hipGetLastError();
}

template <int WM, int WN, int JN, bool PARTS>
static hipError_t launch_shape(int amode, int epi, GemmArgs &g, int n_groups, hipStream_t st)
{
    constexpr int bn = 32 * JN * WN;
    if (g.N % bn != 0 || g.N / bn % n_groups != 0) return hipErrorInvalidValue;
    g.m_tiles = (g.M + 64 * WM - 1) / (64 * WM);
    g.n_tiles = n_groups;
    g.n_loop = g.N / bn / n_groups;
    if constexpr (WM * WN == 4) {
        if (epi == EPI_STORE)
            return amode == AMODE_LOAD ? launch_one<AMODE_LOAD, EPI_STORE, WM, WN, JN, PARTS>(g, st) : launch_one<AMODE_GENV, EPI_STORE, WM, WN, JN, PARTS>(g, st);
    } else if (epi == EPI_STORE) return hipErrorInvalidValue;
    return amode == AMODE_LOAD ? launch_one<AMODE_LOAD, EPI_SCORE, WM, WN, JN, PARTS>(g, st) : launch_one<AMODE_GENV, EPI_SCORE, WM, WN, JN, PARTS>(g, st);
}

hipError_t launch_gemm_split(int amode, int epi, GemmArgs g, int n_groups, int tile, hipStream_t st)
{
    if (g.M <= 0) return hipSuccess;
    if (g.N % 64 != 0 || g.K <= 0 || g.K % 32 != 0 || !g.bias) return hipErrorInvalidValue;
    if (!g.B_parts)
        return g.N % 128 == 0 ? launch_shape<2, 2, 2, false>(amode, epi, g, n_groups, st) : launch_shape<2, 2, 1, false>(amode, epi, g, n_groups, st);
    return tile == 256 ? launch_shape<2, 4, 2, true>(amode, epi, g, n_groups, st)
         : tile == 128 ? launch_shape<2, 2, 2, true>(amode, epi, g, n_groups, st) : launch_shape<2, 2, 1, true>(amode, epi, g, n_groups, st);
}

}  // namespace ab
