// First hidden layer over candidate rows whose 256-row tiles span several scenarios: C = A * W^T with the generated
// operand A[r, k] = relu(a_term[s, k] + wp[k] * xp + wc[k] * xc), row r = (scenario s = r / C, candidate r % C), for
// candidate counts that are no multiple of 256 (gemm_big.hip has the kernel for those, a tile = one scenario).
//
// Same walk over the tiles, W ring, fragment layout, generation (a thread owns one 8-wide k chunk of four adjacent
// rows) and epilogues as gemm_stream_gen_kernel there; what differs:
//   - a tile touches up to SEGS = 8 scenarios (rows per scenario C >= 37), so the scenario terms do not fit LDS as whole
//     rows: they come slab by slab, wavefront w fetching the 64 values of the tile's w-th scenario (one 256-byte
//     request per wavefront and slab, a ring of two, three slabs ahead of the multiplication);
//   - xp / xc are gathered per row (4-byte transfers, the lane's own address);
//   - a group of four adjacent rows may cross into the next scenario.  ROWS4 says what is known of the groups:
//       2: one scenario, one xp (the grid's credit count is a multiple of 4): the inner term is shared by the rows
//       1: one scenario (C is a multiple of 4)
//       0: nothing: a second set of scenario terms is read and the rows behind the border select it
//   - the last row tile may be ragged.
// Memory operations of a wavefront, in order: last quarter of slab j: W(j+2) x4, scenario terms (j+3) x1; at a tile
// border behind them the stores (x16, or x1 in wavefronts 0..3) and the gather (x1).  Inside a tile the wait in front of
// a slab's barrier is for everything; at a tile's first slab the stores and the gather may stay in flight, unless the
// tile has two slabs only: then the next slab already needs the gather.
//
// Bound by the matrix cores.  Before this kernel these shapes took the generic 256 x 256 tile, whose operand loads are
// waited for one by one: 198135 rows x 1024 x 1024 (777 scenarios x 255 candidates) took 1237 us a launch, 419 - 430 us
// here; the whole pass of that network (three hidden products) 1872 -> 1010 us, others of these shapes 1.2 - 2.3 times faster.
#include "stream_util.hpp"
#include <type_traits>

namespace ab {

static constexpr int SEGS = 8;

// n / C for n < 2^31 on the scalar unit: (n * mul) >> shift with mul = ceil(2^shift / C), shift = 31 + ceil(log2 C)
struct DivC { uint32_t mul, shift; };

template <int EPI, int ROWS4, int PARTS>                  // PARTS: of the last round's tiles, as in gemm_big.hip
__device__ __forceinline__ void stream_span_tiles(const GemmArgs &g, const DivC &dc)
{
    constexpr int BM = 256, BK = 64;
    constexpr int SLAB = BM * 128;
    constexpr int W_BASE = 2 * SLAB;
    constexpr int V_WP = 4 * SLAB, V_WC = V_WP + 4096, V_AT = V_WC + 4096, V_XP = V_AT + 2 * SEGS * 256;
    constexpr int V_BIAS = V_XP + 4096, V_WOUT = V_BIAS + 4096;   // fp32 [4][256] each, + 4096: 155648
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wave_m = wave >> 2, wave_n = wave & 3;
    const int half = lane >> 5, l31 = lane & 31;
    const int KT = g.K / BK;
    auto opaque_lane = [&]() { int v = lane; asm volatile("" : "+v"(v)); return v; };

    const unsigned G8 = gridDim.x >> 3, xcd = blockIdx.x & 7, l0 = blockIdx.x >> 3;
    const unsigned n_tiles = (unsigned)g.n_tiles;
    const unsigned panels = (unsigned)g.m_tiles > xcd ? ((unsigned)g.m_tiles - xcd + 7) / 8 : 0;
    const unsigned n_local = panels * n_tiles;
    const LastRound last = last_round<PARTS>(n_local, G8, l0);
    const unsigned n_my = last.n_my;
    if (n_my == 0) return;
    const unsigned C = (unsigned)g.C, M = (unsigned)g.M;
    auto div_c = [&](unsigned n) { return (unsigned)(((uint64_t)n * dc.mul) >> dc.shift); };
    // first row of a tile or part, for what is read (a part may lie past the end as a whole)
    auto tile_row0 = [&](unsigned qq) {
        const unsigned r = ((last.tile(qq, l0, G8) / n_tiles) * 8 + xcd) * (unsigned)BM;
        return PARTS > 1 ? min(r + last.row(qq), M - 1) : r;
    };

    // ---- W slabs by DMA
    const unsigned char *w_base;
    uint32_t w_off[4];
    auto set_w = [&](unsigned q) {
        const unsigned local = last.tile(q, l0, G8);
        w_base = (const unsigned char *)g.B + (int64_t)(local % n_tiles) * 256 * g.ldb * 2;
        const int ln = opaque_lane();
        const int dma_cc = (ln & 7) ^ ((wave & 1) * 4 + (ln >> 4)), dma_r0 = wave * 8 + (ln >> 3);
#pragma unroll
        for (int i = 0; i < 4; ++i) w_off[i] = (uint32_t)(dma_r0 + 64 * i) * (uint32_t)g.ldb * 2u + dma_cc * 16;
    };
    unsigned wq = 0;
    int wkt = 0;
    auto dma_w_rows = [&](int slot, int i0) {
        unsigned char *sb = smem + W_BASE + slot * SLAB;
        dma16<false>(w_base + w_off[i0], sb + (wave + 8 * i0) * 1024);
        dma16<false>(w_base + w_off[i0 + 1], sb + (wave + 8 * (i0 + 1)) * 1024);
    };
    auto advance_w = [&]() {
        w_base += BK * 2;
        if (++wkt == KT) { wkt = 0; if (wq + 1 < n_my) ++wq; set_w(wq); }
    };

    // ---- scenario terms by DMA: this wavefront's scenario of the tile (past the last one: the last one again)
    const float *at_base;
    unsigned atq = 0;
    int atkt = 0, at_slot = 0;
    auto set_at = [&](unsigned q) {
        unsigned s = div_c(tile_row0(q)) + (unsigned)wave;
        const unsigned s_last = div_c(M - 1);
        if (s > s_last) s = s_last;
        at_base = g.a_term + (int64_t)s * g.ldt;
    };
    auto dma_at = [&]() { dma4(at_base + lane, smem + V_AT + at_slot * (SEGS * 256) + wave * 256); };
    auto advance_at = [&]() {
        at_base += BK;
        at_slot ^= 1;
        if (++atkt == KT) { atkt = 0; if (atq + 1 < n_my) ++atq; set_at(atq); }
    };

    // o / C for o < 2^9: by a multiply (exact: o * (C * ceil(2^20 / C) - 2^20) < 512 * 256 < 2^20), C > 255: one border at most
    const unsigned c_magic = C < 256 ? ((1u << 20) + C - 1) / C : 0;
    auto seg_of = [&](unsigned o) { return C < 256 ? (o * c_magic) >> 20 : (o >= C ? 1u : 0u); };

    // ---- candidate values of a tile's rows: wavefronts 0..3 gather xp, 4..7 xc (past the end the last tile's again)
    auto fetch_x = [&](unsigned qq) {
        const int b = (int)(qq & 1);
        if (qq > n_my - 1) qq = n_my - 1;
        const int ln = opaque_lane();
        const unsigned m0 = tile_row0(qq), c0 = m0 - div_c(m0) * C, left = M - 1 - m0;
        unsigned row = (unsigned)((wave & 3) * 64 + ln);
        if (row > left) row = left;
        const unsigned i = g.x_per_row ? m0 + row : c0 + row - seg_of(c0 + row) * C;
        dma4((wave < 4 ? g.xp : g.xc) + i, smem + V_XP + b * 2048 + (wave >> 2) * 1024 + (wave & 3) * 256);
    };
    auto fetch_wp_wc = [&]() {                              // 4 requests per wavefront, once
        const int ln = opaque_lane();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int i = wave + 8 * h;
            if (i > KT - 1) i = KT - 1;
            dma4(g.wp + i * 64 + ln, smem + V_WP + i * 256);
            dma4(g.wc + i * 64 + ln, smem + V_WC + i * 256);
        }
    };

    // ---- generation: thread -> k chunk t & 7 of the four (of a part: IM = 2 or 1) adjacent rows 4 (t >> 3) + i
    typedef std::integral_constant<int, 4> full_tag;
    typedef std::integral_constant<int, 4 / PARTS> part_tag;
    const int gcc = t & 7;
    int gen_st[4];
    auto own_rows = [&](auto im_tag) {
        constexpr int IM = decltype(im_tag)::value;
#pragma unroll
        for (int i = 0; i < IM; ++i) {
            const int row = (t >> 3) * IM + i;
            gen_st[i] = row * 128 + ((gcc ^ ((row >> 1) & 7)) << 4);
        }
    };
    own_rows(full_tag{});
    f32x4 gxp, gxc;
    int seg0 = 0, seg3 = 0, border = 4;                    // byte offsets of the group's scenario terms; rows from `border` on take seg3's
    auto load_group = [&](auto im_tag, unsigned q) {       // what belongs to the group's rows in tile q
        constexpr int IM = decltype(im_tag)::value;
        const float *px = (const float *)(smem + V_XP + (q & 1) * 2048) + (t >> 3) * IM, *pc = px + 256;
        if constexpr (IM == 4) {
            gxp = *(const f32x4 *)px;
            gxc = *(const f32x4 *)pc;
        } else {
#pragma unroll
            for (int i = 0; i < IM; ++i) { gxp[i] = px[i]; gxc[i] = pc[i]; }
        }
        if (q > n_my - 1) q = n_my - 1;
        const unsigned m0 = tile_row0(q), c0 = m0 - div_c(m0) * C, left = M - 1 - m0;
        const unsigned r0 = ((unsigned)(opaque_lane() >> 3) + wave * 8) * IM, r3 = r0 + IM - 1;
        const unsigned s0 = seg_of(c0 + (r0 < left ? r0 : left));
        seg0 = (int)s0 * 256;
        if constexpr (ROWS4 == 0) {
            const unsigned s3 = seg_of(c0 + (r3 < left ? r3 : left));
            seg3 = (int)s3 * 256;
            border = (int)((s0 + 1) * C) - (int)(c0 + r0);     // (beyond 3 where the group has one scenario)
        }
    };
    f32x4 va[2], vb[ROWS4 == 0 ? 2 : 1], vp[2], vc[2];
    auto load_slices = [&](int slot, int gk) {             // slot: ring slot of the scenario terms, gk: slab within the tile
        const int o = (gk * 64 + gcc * 8) * 4;
        const unsigned char *at = smem + V_AT + slot * (SEGS * 256) + gcc * 32;
        va[0] = *(const f32x4 *)(at + seg0);
        va[1] = *(const f32x4 *)(at + seg0 + 16);
        if constexpr (ROWS4 == 0) {
            vb[0] = *(const f32x4 *)(at + seg3);
            vb[1] = *(const f32x4 *)(at + seg3 + 16);
        }
        vp[0] = *(const f32x4 *)(smem + V_WP + o);
        vp[1] = *(const f32x4 *)(smem + V_WP + o + 16);
        vc[0] = *(const f32x4 *)(smem + V_WC + o);
        vc[1] = *(const f32x4 *)(smem + V_WC + o + 16);
    };
    auto gen_chunk = [&](int slot, int i) {
        const float xp = ROWS4 == 2 ? gxp[0] : gxp[i], xc = gxc[i];
        float h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float a = va[e >> 2][e & 3];
            if constexpr (ROWS4 == 0) { if (i > 0) a = i >= border ? vb[e >> 2][e & 3] : a; }
            h[e] = relu_keep_nan(fmaf(vc[e >> 2][e & 3], xc, fmaf(vp[e >> 2][e & 3], xp, a)));
        }
        i32x4 v;
        v.x = (int)pack_bf16x2(h[0], h[1]);
        v.y = (int)pack_bf16x2(h[2], h[3]);
        v.z = (int)pack_bf16x2(h[4], h[5]);
        v.w = (int)pack_bf16x2(h[6], h[7]);
        lds_write16(smem + slot * SLAB + gen_st[i], v);
    };

    // ---- fragment read offsets
    const int sw = (l31 >> 1) & 7;
    int rd[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) rd[q] = l31 * 128 + ((((q << 1) | half) ^ sw) << 4);
    const int w_rd = W_BASE + wave_n * 64 * 128;

    f32x16 acc[2][4];
    i32x4 fa[2][4], fw[2][2];
    auto load_frags = [&](auto im_tag, int a_slot, int w_slot, int q, int set) {
        constexpr int IM = decltype(im_tag)::value;
        const unsigned char *sa = smem + a_slot * SLAB + wave_m * (IM * 4096);
        const unsigned char *sw_ = smem + w_slot * SLAB + w_rd;
#pragma unroll
        for (int jn = 0; jn < 2; ++jn) fw[set][jn] = *(const i32x4 *)(sw_ + jn * 4096 + rd[q]);
#pragma unroll
        for (int im = 0; im < IM; ++im) fa[set][im] = *(const i32x4 *)(sa + im * 4096 + rd[q]);
    };
    auto mma = [&](auto im_tag, int set) {
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
#pragma unroll
            for (int im = 0; im < decltype(im_tag)::value; ++im)
                acc[jn][im] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, fw[set][jn]), __builtin_bit_cast(bf16x8, fa[set][im]),
                    acc[jn][im], 0, 0, 0);
    };
    // A tile's first quarter: the accumulators start at the bias, which waits in those of row block 0 (in their layout,
    // the same for all four row blocks), so block 0 goes last.
    auto mma_first = [&](auto im_tag, int set) {
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
#pragma unroll
            for (int im = decltype(im_tag)::value - 1; im >= 0; --im)
                acc[jn][im] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, fw[set][jn]), __builtin_bit_cast(bf16x8, fa[set][im]),
                    acc[jn][0], 0, 0, 0);
    };

    // bias and output weights of all columns -> LDS, once, by DMA in front of everything else
    int64_t m0 = 0;
    int n0 = 0;
    unsigned tn = 0;
    {
        const int ln = opaque_lane();
#pragma unroll
        for (int h = 0; h < 2; ++h) {                       // pieces of 64 columns (past the last one: that one again)
            const int i = min(wave + 8 * h, (int)n_tiles * 4 - 1);
            dma4(g.bias + i * 64 + ln, smem + V_BIAS + i * 256);
            if constexpr (EPI == EPI_SCORE) dma4(g.w_out + i * 64 + ln, smem + V_WOUT + i * 256);
        }
    }
    auto load_bias = [&]() {
        const int hf = opaque_lane() >> 5;
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const f32x4 b4 = *(const f32x4 *)(smem + V_BIAS + ((int)tn * 256 + wave_n * 64 + jn * 32 + rg * 8 + hf * 4) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[jn][0][rg * 4 + e] = b4[e];
            }
    };
    auto begin_tile = [&](unsigned q) {
        const unsigned local = last.tile(q, l0, G8);
        tn = local % n_tiles;
        n0 = (int)tn * 256;
        m0 = (int64_t)((local / n_tiles) * 8 + xcd) * BM;
        if constexpr (PARTS > 1) m0 += last.row(q);
    };

    // ---- prologue
    set_w(0);
    set_at(0);
    fetch_wp_wc();
    fetch_x(0);
    fetch_x(1);
    dma_at(); advance_at();                                // scenario terms of slabs 0 and 1
    dma_at(); advance_at();
    dma_w_rows(0, 0); dma_w_rows(0, 2); advance_w();
    dma_w_rows(1, 0); dma_w_rows(1, 2); advance_w();
    begin_tile(0);
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                          // vectors, scenario terms, column tables and W(0) are there for everybody
    AB_FENCE();
    load_bias();
    load_group(full_tag{}, 0);
    load_slices(0, 0);
    gen_chunk(0, 0); gen_chunk(0, 1); gen_chunk(0, 2); gen_chunk(0, 3);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                          // A(0) is complete, slot 0 of the scenario terms is free
    AB_FENCE();
    dma_at(); advance_at();                                // slab 2's
    load_frags(full_tag{}, 0, 0, 0, 0);

    int a_slot = 0, w_slot = 0;
    unsigned gq = 0;                                       // tile that is being generated
    unsigned q = 0;
    // One slab (kt = its place in the tile); wave priorities as in gemm_stream_gen_kernel.
    auto slab = [&](auto im_tag, auto first_tag, int kt) {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr int IM = decltype(im_tag)::value;
        const int nxt = a_slot ^ 1;                        // retired one slab ago: slab j+1 is generated there
        int gk = kt + 1;                                   // its place in its tile
        if (gk == KT) { gk = 0; ++gq; load_group(im_tag, gq); }
        load_slices(nxt, gk);                              // (the rings of A and of the scenario terms run in step)
        AB_FENCE();
        if (wave_m) __builtin_amdgcn_s_setprio(3); else __builtin_amdgcn_s_setprio(0);
        load_frags(im_tag, a_slot, w_slot, 1, 1);
        gen_chunk(nxt, 0);
        if constexpr (IM > 1) gen_chunk(nxt, 1);
        if constexpr (FIRST) mma_first(im_tag, 0); else mma(im_tag, 0);
        if constexpr (IM == 4) AB_INTERLEAVE_6(); else AB_INTERLEAVE_PART(IM, 0);
        AB_FENCE();
        __builtin_amdgcn_s_setprio(1);
        load_frags(im_tag, a_slot, w_slot, 2, 0);
        if constexpr (IM == 4) gen_chunk(nxt, 2);
        mma(im_tag, 1);
        if constexpr (IM == 4) AB_INTERLEAVE_6(); else AB_INTERLEAVE_PART(IM, 0);
        AB_FENCE();
        __builtin_amdgcn_s_setprio(0);
        load_frags(im_tag, a_slot, w_slot, 3, 1);
        if constexpr (IM == 4) gen_chunk(nxt, 3);
        mma(im_tag, 0);
        if constexpr (IM == 4) AB_INTERLEAVE_6(); else AB_INTERLEAVE_PART(IM, 0);
        AB_FENCE();
        if (!FIRST || q == 0 || KT == 2) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else if constexpr (EPI == EPI_STORE) {
            asm volatile("s_waitcnt vmcnt(17)" ::: "memory");          // 16 stores + the gather
        } else {
            if (wave < 4) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");   // 1 store of partial sums + the gather
            else          asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
        }
        // own LDS traffic of this slab is done (fragment reads, generated chunks); then meet: slab j+1 is
        // complete and visible to everybody and slab j's stages may be refilled
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        AB_FENCE();
        __builtin_amdgcn_s_setprio(2);
        const int nw = w_slot ^ 1;
        load_frags(im_tag, nxt, nw, 0, 0);
        dma_w_rows(w_slot, 0);
        dma_w_rows(w_slot, 2);
        mma(im_tag, 1);
        if constexpr (IM == 4) AB_INTERLEAVE_6_V4(); else AB_INTERLEAVE_PART(IM, 4);
        AB_FENCE();
        dma_at();
        AB_FENCE();
        advance_w();
        advance_at();
        a_slot = nxt;
        w_slot = nw;
    };
    auto tile = [&](auto im_tag) {
        constexpr int IM = decltype(im_tag)::value;
        slab(im_tag, std::true_type{}, 0);
        for (int kt = 1; kt < KT; ++kt) slab(im_tag, std::false_type{}, kt);
        {
            // ------------------------------------------------------------ epilogue of tile q
            unsigned char *stage = smem + (a_slot ^ 1) * SLAB;            // the A stage retired by the last barrier
            const bool ragged = m0 + IM * 64 > g.M;
            const int ln = opaque_lane();
            const int half = ln >> 5, l31 = ln & 31, sw = (l31 >> 1) & 7;
            if constexpr (EPI == EPI_STORE) {
                unsigned char *mine = stage + wave * 4096;
                const int rrow = ln >> 3, rch = ln & 7;
                uint16_t *dst = (uint16_t *)g.out + (m0 + wave_m * (IM * 32) + rrow) * g.ldo + n0 + wave_n * 64 + rch * 8;
#pragma unroll
                for (int im = 0; im < IM; ++im) {
#pragma unroll
                    for (int jn = 0; jn < 2; ++jn)
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg) {
                            float v[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = relu_keep_nan(acc[jn][im][rg * 4 + e]);
                            uint2 pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                            lds_write8(mine + l31 * 128 + (((jn * 4 + rg) ^ sw) << 4) + half * 8, pk);
                        }
                    i32x4 o[4];
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const int row = rrow + 8 * it;
                        o[it] = *(const i32x4 *)(mine + row * 128 + ((rch ^ ((row >> 1) & 7)) << 4));
                    }
                    uint16_t *d = dst + (int64_t)(im * 32) * g.ldo;
                    if (!ragged) {
#pragma unroll
                        for (int it = 0; it < 4; ++it)
                            __builtin_nontemporal_store(o[it], (i32x4 *)(d + (int64_t)(8 * it) * g.ldo));
                    } else {
#pragma unroll
                        for (int it = 0; it < 4; ++it)
                            if (m0 + wave_m * (IM * 32) + im * 32 + rrow + 8 * it < g.M)
                                __builtin_nontemporal_store(o[it], (i32x4 *)(d + (int64_t)(8 * it) * g.ldo));
                    }
                }
            } else {   // EPI_SCORE: the output unit as a per-lane dot product, reduced over the four column wavefronts
                float ps[IM];
#pragma unroll
                for (int im = 0; im < IM; ++im) ps[im] = 0.f;
#pragma unroll
                for (int jn = 0; jn < 2; ++jn)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const f32x4 w4 = *(const f32x4 *)(smem + V_WOUT + ((int)tn * 256 + wave_n * 64 + jn * 32 + rg * 8 + half * 4) * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int im = 0; im < IM; ++im)
                                ps[im] += relu_keep_nan(acc[jn][im][rg * 4 + e]) * w4[e];
                    }
                float *red = (float *)stage;               // [4 column-waves][256 rows]
#pragma unroll
                for (int im = 0; im < IM; ++im) {
                    const float v = ps[im] + __shfl_xor(ps[im], 32, 64);
                    if (half == 0) lds_write4(red + wave_n * BM + wave_m * (IM * 32) + l31 + im * 32, v);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                if (wave < IM) {
                    const int tt = wave * 64 + ln;
                    const float v = (red[tt] + red[BM + tt]) + (red[2 * BM + tt] + red[3 * BM + tt]);
                    if (!ragged) g.partial[(m0 + tt) * g.n_tiles + tn] = v;
                    else if (m0 + tt < g.M) g.partial[(m0 + tt) * g.n_tiles + tn] = v;
                }
            }
            // a ragged tile may have issued fewer stores than the counts assume: drain instead
            if (ragged) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    };
    while (true) {
        if constexpr (PARTS > 1) {
            if (q == last.q_part) {                        // (its first slab was generated as a whole tile's)
                own_rows(part_tag{});
                load_group(part_tag{}, q);
                load_frags(part_tag{}, a_slot, w_slot, 0, 0);
                tile(part_tag{});
                break;
            }
        }
        tile(full_tag{});
        if (q + 1 == n_my) break;
        ++q;
        {
            begin_tile(q);
            load_bias();                                   // (a fixed table: its reads may return under the wait below)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();                  // everybody has read the staging room back
            AB_FENCE();
            fetch_x(q + 1);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no DMA may still target LDS when the group ends
}

template <int EPI, int ROWS4>
__global__ __launch_bounds__(512) void gemm_stream_span_kernel(const GemmArgs g, const DivC dc) { touch_arguments<sizeof(GemmArgs) + sizeof(DivC)>(); stream_span_tiles<EPI, ROWS4, 1>(g, dc); }
template <int EPI, int ROWS4, int PARTS>
__global__ __launch_bounds__(512) void gemm_parts_span_kernel(const GemmArgs g, const DivC dc) { touch_arguments<sizeof(GemmArgs) + sizeof(DivC)>(); stream_span_tiles<EPI, ROWS4, PARTS>(g, dc); }

template <int EPI, int ROWS4>
static hipError_t launch_span_one(const GemmArgs &g, hipStream_t st)
{
    constexpr int smem = 4 * 256 * 128 + 2 * 4096 + 2 * SEGS * 256 + 4096 + 8192;
    StreamGrid gr;
    hipError_t e = stream_grid(g, &gr);
    if (e != hipSuccess || gr.blocks == 0) return e;
    static DeviceOnce once[3];
    auto kern = gr.parts == 1 ? gemm_stream_span_kernel<EPI, ROWS4> : gr.parts == 2 ? gemm_parts_span_kernel<EPI, ROWS4, 2> : gemm_parts_span_kernel<EPI, ROWS4, 4>;
    e = ensure_dynamic_lds((const void *)kern, smem, once[gr.parts >> 1]);
    if (e != hipSuccess) return e;
    DivC dc{0, 31};
    while ((1LL << (dc.shift - 31)) < g.C) ++dc.shift;
    dc.mul = (uint32_t)(((1ull << dc.shift) + (uint32_t)g.C - 1) / (uint32_t)g.C);
    kern<<<gr.blocks, 512, smem, st>>>(g, dc);
    return hipGetLastError();
}

// 256 rows touch at most 1 + ceil(255 / C) scenarios: at most SEGS for C >= 37.  The tables of bias and output weights
// hold four column tiles, those of wp and wc 1024 inputs; the rings need two slabs.
bool gemm_span_shape(int32_t C, int H_in, int H_out)
{
    return C >= 37 && H_in % 64 == 0 && H_in >= 128 && H_in <= 1024 && H_out % 256 == 0 && H_out <= 1024;
}

hipError_t launch_gemm_span(int epi, GemmArgs g, hipStream_t st)
{
    if (!gemm_span_shape(g.C, g.K, g.N) || g.M <= 0 || g.M > 0x7fffff00LL || g.ldt % 4 != 0 || g.ldb % 8 != 0 || !g.bias ||
        !g.relu || !g.wp || !g.wc || !g.xp || !g.xc || (epi == EPI_STORE && (g.out_f32 || g.out_t || g.ldo % 8 != 0)))
        return hipErrorInvalidValue;
    g.m_tiles = (g.M + 255) / 256;
    g.n_tiles = g.N / 256;
    const int rows4 = g.C % 4 ? 0 : g.xp_runs4 ? 2 : 1;
    if (epi == EPI_STORE)
        return rows4 == 2 ? launch_span_one<EPI_STORE, 2>(g, st) : rows4 == 1 ? launch_span_one<EPI_STORE, 1>(g, st)
                                                                             : launch_span_one<EPI_STORE, 0>(g, st);
    return rows4 == 2 ? launch_span_one<EPI_SCORE, 2>(g, st) : rows4 == 1 ? launch_span_one<EPI_SCORE, 1>(g, st)
                                                                         : launch_span_one<EPI_SCORE, 0>(g, st);
}

}  // namespace ab
