// C = A * B^T where the whole product is a fraction of the chip's work (a job, a few hundred rows): one 32 x 32 tile per
// work-group, its four wavefronts share the summed index.
//
// Such a product is bound by latency: what it reads was written by other XCDs and comes from the Infinity Cache, at 1 - 2 us
// a round trip, and a tile that walks its slabs with one slab requested ahead pays that trip once per slab (256 x 1024 x
// 1024 in bf16 on 64 x 64 tiles: 10.9 us, 16.5 us with a generated operand; here 4.8 and 6.3 - 6.8).  Here wavefront w takes slabs w, w + 4, ...
// of 128 bytes a row and requests up to NS of them (both operands) at once by DMA into an LDS ring of its own, so K = 1024
// in bf16 is one round trip, and there is no barrier before the four partial tiles meet in LDS.  The small tile gives four
// times the work-groups at twice the bytes, which a product that leaves most CUs idle does not notice.
//
// With GEN the first operand is the first hidden layer, relu(a_term[s] + wp xp + wc xc) (gemm_core.hpp, factored form):
// the a_term chunks, wp and wc come by DMA as well and the fragment is formed when it is read.  With 32 or more rows a
// scenario a tile touches at most two of them (GEN_PAIR): one request a slab brings both scenarios' terms, wp and wc, and a
// row picks its scenario's (one job on the 1024-wide network, a call: 27.7 us with every row's terms, 26.0 so).  With fewer
// rows a scenario (GEN_ROWS) every row's terms come, in bf16 eight requests more a slab.
#include "stream_util.hpp"

namespace ab {

enum { GEN_NONE = 0, GEN_ROWS = 1, GEN_PAIR = 2 };

template <typename T, int GEN>
struct SlimShape {
    static constexpr int BK = TileTraits<T>::BK;
    static constexpr int A_BYTES = GEN == GEN_ROWS ? 32 * BK * 4 : GEN == GEN_PAIR ? 0 : 4096, B_BYTES = 4096, W_BYTES = GEN ? 1024 : 0;
    static constexpr int SLAB = A_BYTES + B_BYTES + W_BYTES;
    static constexpr int REQ = SLAB / 1024;                  // DMA requests of a slab
    static constexpr int NS = GEN == GEN_ROWS && sizeof(T) == 2 ? 3 : 4; // slabs in flight a wavefront (160 KB of LDS)
    static constexpr int TABLES = 512;                       // xp, xc of the tile's rows, bias and output weights of its columns
};

template <int REQ>
__device__ __forceinline__ void wait_slabs(int left)         // at most `left` slabs' requests outstanding
{
    if (left >= 3)      asm volatile("s_waitcnt vmcnt(%0)" ::"i"(3 * REQ) : "memory");
    else if (left == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(2 * REQ) : "memory");
    else if (left == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(REQ) : "memory");
    else                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <typename T, int GEN, int EPI>
__global__ __launch_bounds__(256) void gemm_slim_kernel(const GemmArgs g, int stages)
{
    typedef SlimShape<T, GEN> Z;
    constexpr int ES = sizeof(T), BK = Z::BK;
    touch_arguments<sizeof(GemmArgs) + 4>();
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, l31 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // consecutive work-groups go to consecutive XCDs: a column tile of B (the larger operand) stays with one of them
    const int tn = (int)(blockIdx.x % (unsigned)g.n_tiles);
    const int64_t m0 = (int64_t)(blockIdx.x / (unsigned)g.n_tiles) * 32;
    // rows and candidates fit 32 bits (the launcher checks): 64-bit divisions are a good part of the way to the first request
    // (one job on the 1024-wide network, a call: 26.1 us with them, 25.9 so; 300 jobs with V 113.3 -> 112.0)
    const unsigned um0 = (unsigned)m0, uC = (unsigned)g.C, uM = (unsigned)g.M;
    const int n0 = tn * 32;
    const int area = stages * Z::SLAB + Z::TABLES;
    unsigned char *ring = smem + wave * area, *tab = ring + stages * Z::SLAB;

    // tables: lanes 0..31 and 32..63 of one request each
    if constexpr (GEN) {
        const unsigned r = min(um0 + l31, uM - 1);
        const unsigned x = g.x_per_row ? r : r % uC;
        dma4((half ? g.xc : g.xp) + x, tab);
    }
    dma4((half && EPI == EPI_SCORE ? g.w_out : g.bias) + n0 + l31, tab + 256);

    // DMA sources.  128-byte rows: chunk c of row r sits at c ^ ((r >> 1) & 7); 256-byte rows (a_term of a bf16 slab): c ^ (r & 15)
    constexpr int AROW = Z::A_BYTES / 32, ACH = AROW / 16, A_REQ = Z::A_BYTES / 1024;
    const unsigned char *pa = nullptr, *pb = (const unsigned char *)g.B + (int64_t)n0 * g.ldb * ES;
    int32_t off_a[A_REQ ? A_REQ : 1], off_b[4];
    const float *pv = nullptr;                               // vectors of a generated operand: this lane's piece of a request
    int second = 0;                                          // GEN_PAIR: this lane's row is of the tile's second scenario
    auto place = [](int row, int c) { return AROW == 256 ? c ^ (row & 15) : c ^ ((row >> 1) & 7); };
    if constexpr (GEN == GEN_PAIR) {
        // a_term of the two scenarios (the last one twice at the end), wp, wc: BK / 4 lanes each (fp32: the rest repeats them)
        const int64_t s0 = um0 / uC, s1 = min(s0 + 1, (int64_t)((uM - 1) / uC));
        const int part = (lane / (BK / 4)) & 3;
        pv = (part == 0 ? g.a_term + s0 * g.ldt : part == 1 ? g.a_term + s1 * g.ldt : part == 2 ? g.wp : g.wc) + (lane & (BK / 4 - 1)) * 4;
        second = m0 + l31 >= (s0 + 1) * g.C;
    } else if constexpr (GEN == GEN_ROWS) {
        // wp, wc: lanes 0 .. BK/4 - 1, then as many (the rest of the request repeats them)
        pv = (lane & (BK / 4) ? g.wc : g.wp) + (lane & (BK / 4 - 1)) * 4;
        const int64_t s0 = um0 / uC;
        pa = (const unsigned char *)(g.a_term + s0 * g.ldt);
#pragma unroll
        for (int i = 0; i < A_REQ; ++i) {
            const int row = i * (64 / ACH) + lane / ACH;
            const int64_t s = min(um0 + row, uM - 1) / uC - s0;
            off_a[i] = (int32_t)s * g.ldt * 4 + place(row, lane & (ACH - 1)) * 16;
        }
    } else {
        pa = (const unsigned char *)g.A + m0 * g.lda * ES;
#pragma unroll
        for (int i = 0; i < A_REQ; ++i) {
            const int row = i * 8 + (lane >> 3);
            off_a[i] = (int32_t)(min((int64_t)row, g.M - 1 - m0) * g.lda) * ES + place(row, lane & 7) * 16;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = i * 8 + (lane >> 3);
        off_b[i] = (int32_t)(row * g.ldb) * ES + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    auto fetch = [&](int i, unsigned char *dst) {            // slab wave + 4 i
        const int kt = wave + 4 * i;
#pragma unroll
        for (int q = 0; q < A_REQ; ++q) dma16<false>(pa + kt * AROW + off_a[q], dst + q * 1024);
#pragma unroll
        for (int q = 0; q < 4; ++q) dma16<false>(pb + kt * 128 + off_b[q], dst + Z::A_BYTES + q * 1024);
        if constexpr (GEN) dma16<false>(pv + kt * BK, dst + Z::A_BYTES + Z::B_BYTES);
    };
    const int slabs = g.K / BK, n = (slabs - wave + 3) >> 2;
    for (int i = 0; i < stages && i < n; ++i) fetch(i, ring + i * Z::SLAB);

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    unsigned char *slot = ring;
    float xp = 0.f, xc = 0.f;
    for (int i = 0; i < n; ++i) {
        wait_slabs<Z::REQ>(min(stages - 1, n - 1 - i));
        if constexpr (GEN) {
            if (i == 0) { xp = ((const float *)tab)[l31]; xc = ((const float *)tab)[32 + l31]; }
        }
        i32x4 fa[4], fb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = q * 2 + half;
            fb[q] = *(const i32x4 *)(slot + Z::A_BYTES + l31 * 128 + ((c ^ ((l31 >> 1) & 7)) << 4));
            if constexpr (!GEN) {
                fa[q] = *(const i32x4 *)(slot + l31 * 128 + (place(l31, c) << 4));
            } else {
                const float *vec = (const float *)(slot + Z::A_BYTES + Z::B_BYTES), *w = GEN == GEN_PAIR ? vec + 2 * BK : vec;
                float h[16 / ES];
#pragma unroll
                for (int p = 0; p < 4 / ES; ++p) {
                    const int ch = c * (4 / ES) + p;         // chunk of four floats
                    const f32x4 a = GEN == GEN_PAIR ? *(const f32x4 *)(vec + second * BK + ch * 4)
                                                    : *(const f32x4 *)(slot + l31 * AROW + (place(l31, ch) << 4));
                    const f32x4 wp = *(const f32x4 *)(w + ch * 4), wc = *(const f32x4 *)(w + BK + ch * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[4 * p + e] = relu_keep_nan(fmaf(wc[e], xc, fmaf(wp[e], xp, a[e])));
                }
                if constexpr (ES == 2) fa[q] = i32x4{(int)pack_bf16x2(h[0], h[1]), (int)pack_bf16x2(h[2], h[3]),
                                                     (int)pack_bf16x2(h[4], h[5]), (int)pack_bf16x2(h[6], h[7])};
                else fa[q] = __builtin_bit_cast(i32x4, f32x4{h[0], h[1], h[2], h[3]});
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot is read
        if (i + stages < n) fetch(i + stages, slot);
#pragma unroll
        for (int q = 0; q < 4; ++q) mma_chunk<T>(fa[q], fb[q], acc);
        slot = slot + Z::SLAB == tab ? ring : slot + Z::SLAB;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (a wavefront without slabs: its tables)

    // the four partial tiles, [row][32 columns], each over its wavefront's own ring
#pragma unroll
    for (int r = 0; r < 16; ++r) lds_write4(ring + ((r >> 2) * 8 + half * 4 + (r & 3)) * 128 + l31 * 4, acc[r]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int row = t >> 3, c4 = (t & 7) * 4;
    f32x4 v = *(const f32x4 *)(smem + row * 128 + c4 * 4);
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *(const f32x4 *)(smem + w * area + row * 128 + c4 * 4);
    v += *(const f32x4 *)(tab + 256 + c4 * 4);
    const bool in = m0 + row < g.M;
    if constexpr (EPI == EPI_STORE) {
        if (g.relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = relu_keep_nan(v[e]);
        }
        if (!in) return;
        const int64_t o = (m0 + row) * g.ldo + n0 + c4;
        if (ES == 4 || g.out_f32) *(f32x4 *)((float *)g.out + o) = v;
        else *(uint2 *)((uint16_t *)g.out + o) = uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else {
        const f32x4 w = *(const f32x4 *)(tab + 384 + c4 * 4);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fmaf(relu_keep_nan(v[e]), w[e], s);
        s += dpp_move<0xB1>(s);
        s += dpp_move<0x4E>(s);
        s += dpp_move<0x141>(s);
        if (in && (t & 7) == 0) g.partial[(m0 + row) * g.n_tiles + tn] = s;
    }
}

template <typename T, int GEN, int EPI>
static hipError_t launch_slim(const GemmArgs &g, hipStream_t st)
{
    typedef SlimShape<T, GEN> Z;
    auto kern = gemm_slim_kernel<T, GEN, EPI>;
    static DeviceOnce once;
    hipError_t e = ensure_dynamic_lds((const void *)kern, 4 * (Z::NS * Z::SLAB + Z::TABLES), once);
    if (e != hipSuccess) return e;
    const int per_wave = (g.K / Z::BK + 3) / 4, stages = per_wave < Z::NS ? per_wave : Z::NS;
    kern<<<(unsigned)(g.m_tiles * g.n_tiles), 256, 4 * (stages * Z::SLAB + Z::TABLES), st>>>(g, stages);
    return hipGetLastError();
}

template <typename T, int GEN>
static hipError_t launch_slim_as(int epi, const GemmArgs &g, hipStream_t st)
{
    return epi == EPI_STORE ? launch_slim<T, GEN, EPI_STORE>(g, st) : launch_slim<T, GEN, EPI_SCORE>(g, st);
}

template <typename T>
static hipError_t launch_slim_of(bool gen, int epi, const GemmArgs &g, hipStream_t st)
{
    if (!gen) return launch_slim_as<T, GEN_NONE>(epi, g, st);
    return g.C >= 32 ? launch_slim_as<T, GEN_PAIR>(epi, g, st) : launch_slim_as<T, GEN_ROWS>(epi, g, st);
}

hipError_t launch_gemm_slim(int dtype, int amode, int epi, const GemmArgs &g, hipStream_t st)
{
    if (!g.bias || g.out_t || (epi != EPI_STORE && epi != EPI_SCORE) || g.m_tiles * g.n_tiles > 0x7fffffffLL || g.M > 0x7fffff00LL) return hipErrorInvalidValue;
    const bool gen = amode != AMODE_LOAD;
    return dtype == AB_BF16 ? launch_slim_of<bf16_t>(gen, epi, g, st) : launch_slim_of<float>(gen, epi, g, st);
}

}  // namespace ab
