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
// What bounds it: the matrix pipe at a power-limited clock.  Six bf16 instructions of 32 cycles do the work of eight fp32
// ones of 64 cycles.  4.2 M rows x 256 x 256 with generated operand and fused output unit, in four launches: 1.15 ms a
// launch on the fp32 instruction (76 % of its peak), 0.63 - 0.66 ms here (0.70 under the profiler); matrix pipe busy 61 % of the
// cycles, clock 1.95 GHz.
//
// Shape: a work-group of 256 threads (2 x 2 wavefronts) owns 128 rows and walks its column tiles of BN columns, K in
// slabs of 16.  A wavefront's 64 x BN/2 outputs take 128 accumulator registers with both sets, so two wavefronts fit a
// SIMD: two work-groups share a CU, and one's LDS latencies, barriers and epilogues run under the other's matrix work.
// The vector work of a slab (operand generation, splitting) is spread over its matrix instructions, five between two
// (1.30 M cycles a launch; in one piece a fifth more).  LDS: two stages; a stage holds, per operand, part and half of the
// slab's sixteen k, 16 bytes per row one row after the other: a thread writes the eight k it has split and a fragment
// is one 16-byte read, both over consecutive addresses (no bank conflicts, no swizzle).  Slab j + 1's raw values are in
// registers while slab j is multiplied, and slab j + 2's are on their way (requested only half a slab ahead: 5 % slower).
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
#include <type_traits>

namespace ab {

// The three parts of two fp32 values, packed: p[i] = part i of a (low half) and b.
__device__ __forceinline__ void split3(float a, float b, uint32_t (&p)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = pack_bf16x2(a, b);                          // round to nearest even
        asm("" : "+v"(p[i]));                              // (one conversion of the pair: not once more for each half)
        if (i < 2) {
            a -= __uint_as_float(p[i] << 16);              // exact; what is left after two parts fits bf16
            b -= __uint_as_float(p[i] & 0xffff0000u);
        }
    }
}

template <int AMODE, int EPI, int BN>
__global__ __launch_bounds__(256, 2) void gemm_split_kernel(const GemmArgs g)
{
    touch_arguments<sizeof(GemmArgs)>();
    constexpr int BM = 128, BK = 16, JN = BN / 64;
    constexpr int WE = BN / 16;                            // weights a thread splits per slab (8 or 4)
    constexpr int A_PLANE = BM * 16, W_PLANE = BN * 16;    // one part, one half of the slab's k
    constexpr int W_BASE = 6 * A_PLANE, STAGE = 6 * (A_PLANE + W_PLANE);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // column groups of one row panel stay on one XCD (they share the activations)
    const int64_t local = blockIdx.x >> 3;
    const int tn = (int)(local % g.n_tiles);
    const int64_t tm = (local / g.n_tiles) * 8 + (blockIdx.x & 7);
    if (tm >= g.m_tiles) return;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1, half = lane >> 5, l31 = lane & 31;
    const int64_t m0 = tm * BM;
    const int KT = g.K / BK, n_first = tn * g.n_loop * BN;

    // ---- this thread's share of a slab: eight k of one activation row, WE k of one weight row
    const int a_row = t & (BM - 1), a_kh = wave >> 1;
    const int w_row = t & (BN - 1), w_part = BN == 128 ? wave >> 1 : wave;     // which WE of the sixteen k
    const int64_t gr = min(m0 + a_row, g.M - 1);
    const float *a_src;
    float xp = 0.f, xc = 0.f;
    if constexpr (AMODE == AMODE_LOAD) {
        a_src = (const float *)g.A + gr * g.lda + a_kh * 8;
    } else {
        const int64_t s = gr / g.C, x = g.x_per_row ? gr : gr - s * g.C;
        a_src = g.a_term + s * g.ldt + a_kh * 8;
        xp = g.xp[x];
        xc = g.xc[x];
    }
    const float *w_src = (const float *)g.B + (int64_t)(n_first + w_row) * g.ldb + w_part * WE;
    f32x4 ra[2][2], rw[2][WE / 4];                         // two sets: requested a slab ahead
    f32x8_unaligned rp[2], rc[2];                          // wp, wc of the slab: the same for the whole wavefront
    int ld_k = 0, ld_n = 0;                                // the slab that is requested next: its k, its column tile
    auto request = [&](int set) {
        ra[set][0] = *(const f32x4 *)(a_src + ld_k);
        ra[set][1] = *(const f32x4 *)(a_src + ld_k + 4);
#pragma unroll
        for (int i = 0; i < WE / 4; ++i) rw[set][i] = *(const f32x4 *)(w_src + ld_k + 4 * i);
    };
    auto request_vectors = [&](int set) {                  // ... and wp, wc by scalar loads; then on to the slab after it
        if constexpr (AMODE != AMODE_LOAD) {
            rp[set] = *(const const_f32x8 *)(uintptr_t)(g.wp + ld_k + a_kh * 8);
            rc[set] = *(const const_f32x8 *)(uintptr_t)(g.wc + ld_k + a_kh * 8);
        }
        ld_k += BK;
        if (ld_k == g.K) {                                 // (behind the last column tile: that one again, not used)
            ld_k = 0;
            if (++ld_n < g.n_loop) w_src += (int64_t)BN * g.ldb;
        }
    };
    uint32_t pa[4][3], pw[4][3];                           // the split pairs of this thread's shares
    auto split_half = [&](int set, int h) {
#pragma unroll
        for (int e = 2 * h; e < 2 * h + 2; ++e) {
            float v[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                v[i] = ra[set][e >> 1][2 * (e & 1) + i];
                if constexpr (AMODE != AMODE_LOAD)
                    v[i] = relu_keep_nan(fmaf(rc[set][2 * e + i], xc, fmaf(rp[set][2 * e + i], xp, v[i])));
            }
            split3(v[0], v[1], pa[e]);
            if (e < WE / 2) split3(rw[set][e >> 1][2 * (e & 1)], rw[set][e >> 1][2 * (e & 1) + 1], pw[e]);
        }
    };
    auto write_parts = [&](unsigned char *stage) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            *(i32x4 *)(stage + (i * 2 + a_kh) * A_PLANE + a_row * 16) = i32x4{(int)pa[0][i], (int)pa[1][i], (int)pa[2][i], (int)pa[3][i]};
            if constexpr (WE == 8)
                *(i32x4 *)(stage + W_BASE + (i * 2 + w_part) * W_PLANE + w_row * 16) = i32x4{(int)pw[0][i], (int)pw[1][i], (int)pw[2][i], (int)pw[3][i]};
            else
                *(uint2 *)(stage + W_BASE + (i * 2 + (w_part >> 1)) * W_PLANE + w_row * 16 + (w_part & 1) * 8) = uint2{pw[0][i], pw[1][i]};
        }
    };

    const int a_rd = half * A_PLANE + (wave_m * 64 + l31) * 16;
    const int w_rd = W_BASE + half * W_PLANE + (wave_n * (BN / 2) + l31) * 16;
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
        const int nw = n0 + wave_n * (BN / 2);
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

    request(0);
    request_vectors(0);
    request(1);
    request_vectors(1);
    split_half(0, 0);
    split_half(0, 1);
    write_parts(smem);
    __syncthreads();
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
        auto interleave = [&]() {
#pragma unroll
            for (int i = 0; i < 6 * JN; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
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
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
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
        if (t < BM && m0 + t < g.M) g.partial[(m0 + t) * g.n_tiles + tn] = red[t] + red[BM + t];
    }
}

template <int AMODE, int EPI, int BN>
static hipError_t launch_one(const GemmArgs &g, hipStream_t st)
{
    constexpr int smem = 2 * 6 * (128 + BN) * 16;
    const int64_t blocks = (g.m_tiles + 7) / 8 * 8 * g.n_tiles;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    gemm_split_kernel<AMODE, EPI, BN><<<(unsigned)blocks, 256, smem, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_split(int amode, int epi, GemmArgs g, int n_groups, hipStream_t st)
{
    const int bn = g.N % 128 == 0 ? 128 : 64;
    if (g.M <= 0) return hipSuccess;
    if (g.N % bn != 0 || g.K <= 0 || g.K % 32 != 0 || !g.bias || g.N / bn % n_groups != 0) return hipErrorInvalidValue;
    g.m_tiles = (g.M + 127) / 128;
    g.n_tiles = n_groups;
    g.n_loop = g.N / bn / n_groups;
    if (bn == 128) {
        if (amode == AMODE_LOAD)
            return epi == EPI_STORE ? launch_one<AMODE_LOAD, EPI_STORE, 128>(g, st) : launch_one<AMODE_LOAD, EPI_SCORE, 128>(g, st);
        return epi == EPI_STORE ? launch_one<AMODE_GENV, EPI_STORE, 128>(g, st) : launch_one<AMODE_GENV, EPI_SCORE, 128>(g, st);
    }
    if (amode == AMODE_LOAD)
        return epi == EPI_STORE ? launch_one<AMODE_LOAD, EPI_STORE, 64>(g, st) : launch_one<AMODE_LOAD, EPI_SCORE, 64>(g, st);
    return epi == EPI_STORE ? launch_one<AMODE_GENV, EPI_STORE, 64>(g, st) : launch_one<AMODE_GENV, EPI_SCORE, 64>(g, st);
}

}  // namespace ab
