// fp32 values in three bf16 parts, and weights laid out in them for gemm_split.hip.
#pragma once
#include "gemm_core.hpp"

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

// Weights W[N, K] in their parts, in the order in which the slabs of a column tile of `tile` columns go to LDS:
// out[tile][slab of 16 k][part][half][column], eight k of 2 bytes each; 6 bytes a weight.
struct SplitWeights { const float *W; i32x4 *out; int32_t N, K, tile; };
enum { kMostSplitWeights = 3 };
struct SplitWeightsArgs { SplitWeights w[kMostSplitWeights]; int32_t n; uint32_t from; };     // from: the first work-group of them
inline int64_t split_weights_items(const SplitWeightsArgs &a)
{
    int64_t n = 0;
    for (int i = 0; i < a.n; ++i) n += (int64_t)a.w[i].N * (a.w[i].K / 8);
    return n;
}
__device__ __forceinline__ void split_weights_item(const SplitWeightsArgs &a, int64_t id)
{
    for (int i = 0; i < a.n; ++i) {
        const SplitWeights &w = a.w[i];
        const int64_t items = (int64_t)w.N * (w.K / 8);
        if (id >= items) { id -= items; continue; }
        const int q = (int)(id / w.N), n = (int)(id - (int64_t)q * w.N);       // eight k of one column; adjacent lanes, adjacent columns
        const float *src = w.W + (int64_t)n * w.K + q * 8;
        const f32x4 lo = *(const f32x4 *)src, hi = *(const f32x4 *)(src + 4);
        uint32_t p[4][3];
        split3(lo[0], lo[1], p[0]);
        split3(lo[2], lo[3], p[1]);
        split3(hi[0], hi[1], p[2]);
        split3(hi[2], hi[3], p[3]);
        i32x4 *out = w.out + (((int64_t)(n / w.tile) * (w.K / 16) + q / 2) * 6 + (q & 1)) * w.tile + n % w.tile;
#pragma unroll
        for (int j = 0; j < 3; ++j) out[j * 2 * w.tile] = i32x4{(int)p[0][j], (int)p[1][j], (int)p[2][j], (int)p[3][j]};
        return;
    }
}

}  // namespace ab
