// What the streaming GEMM kernels (gemm_big.hip, gemm_span.hip) share: global->LDS transfers, LDS stores that are not
// ordered behind them, scalar loads, and the scheduling hints of a slab's quarters.
#pragma once
#include "internal.hpp"

namespace ab {

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;
typedef float f32x8_unaligned __attribute__((ext_vector_type(8), aligned(4)));

typedef __attribute__((address_space(4))) f32x8_unaligned const_f32x8;   // read-only for the whole launch: scalar loads
// Eight consecutive floats at a wave-uniform address, fetched through the scalar cache into scalar registers.
__device__ __forceinline__ f32x8_unaligned scalar_load8(const float *p)
{
    f32x8_unaligned v = *(const const_f32x8 *)(uintptr_t)p;
    asm volatile("" : "+s"(v));
    return v;
}

// 64 lanes x 16 bytes; lane l's data lands at lds_uniform_dst + 16*l.  STREAM marks the access
// non-temporal: activation panels and outputs pass through L2 once per XCD and should not push the
// weight matrix (re-read by every tile) out of it.
template <bool STREAM>
__device__ __forceinline__ void dma16(const void *gsrc, void *lds_uniform_dst)
{
    __builtin_amdgcn_global_load_lds((global_void *)gsrc, (lds_void *)lds_uniform_dst, 16, 0, STREAM ? 2 : 0);
}
__device__ __forceinline__ void dma4(const void *gsrc, void *lds_uniform_dst)   // 64 lanes x 4 bytes
{
    __builtin_amdgcn_global_load_lds((global_void *)gsrc, (lds_void *)lds_uniform_dst, 4, 0, 0);
}

// LDS stores the compiler does not see as such: it orders every LDS store it knows of behind all
// global->LDS DMA in flight (a full vmcnt drain), which the staging writes of the epilogue must not do;
// the stage they go to has been retired by the barrier before.  LDS operations of a wavefront execute
// in order, so the reads that follow see the data.
__device__ __forceinline__ void lds_write8(void *p, uint2 v)
{
    asm volatile("ds_write_b64 %0, %1" ::"v"((uint32_t)(uintptr_t)(lds_void *)p), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_write4(void *p, float v)
{
    asm volatile("ds_write_b32 %0, %1" ::"v"((uint32_t)(uintptr_t)(lds_void *)p), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_write16(void *p, i32x4 v)
{
    asm volatile("ds_write_b128 %0, %1" ::"v"((uint32_t)(uintptr_t)(lds_void *)p), "v"(v) : "memory");
}

// Scheduling hints: keep the source order of the phases (fence) and, inside a phase, alternate one
// matrix instruction with one LDS fragment read so the reads for the next quarter are issued under
// the current quarter's matrix work instead of being sunk in front of their first use.
#define AB_FENCE() __builtin_amdgcn_sched_barrier(0)
#define AB_MFMA_DS_PAIR() do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); \
                               __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); } while (0)
#define AB_INTERLEAVE_6() do { AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); \
                               AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); \
                               __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); } while (0)
// Scheduling inside a quarter that also issues slab fetches: 8 matrix instructions, 6 fragment reads and
// 2 (or 4) DMA requests, spread evenly.
#define AB_MFMA_VMEM_PAIR() do { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); \
                                 __builtin_amdgcn_sched_group_barrier(0x010, 1, 0); } while (0)
#define AB_INTERLEAVE_6_V2() do { AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); \
                                  AB_MFMA_DS_PAIR(); AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_DS_PAIR(); } while (0)
#define AB_INTERLEAVE_6_V4() do { __builtin_amdgcn_sched_group_barrier(0x100, 2, 0); \
                                  AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); \
                                  AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); AB_MFMA_VMEM_PAIR(); AB_MFMA_DS_PAIR(); } while (0)
// The same for a part of a tile: IM row blocks a wavefront, 2 IM matrix instructions and 2 + IM fragment reads a quarter, REQS DMA
// requests (4 or IM).
#define AB_INTERLEAVE_PART(IM, REQS) do { \
        if constexpr ((REQS) > 0) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0); \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); \
        if constexpr ((REQS) > 0) __builtin_amdgcn_sched_group_barrier(0x010, ((REQS) + 1) / 2, 0); \
        __builtin_amdgcn_sched_group_barrier(0x100, (REQS) > 0 ? (IM) : 2, 0); \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); \
        if constexpr ((REQS) > 1) __builtin_amdgcn_sched_group_barrier(0x010, (REQS) / 2, 0); \
        if constexpr ((REQS) == 0) __builtin_amdgcn_sched_group_barrier(0x100, (IM), 0); \
        if constexpr ((IM) > 1) __builtin_amdgcn_sched_group_barrier(0x008, 2 * (IM) - 2, 0); } while (0)

// The last round of a streaming kernel's tiles, per XCD: work-group l0 of G8 takes tiles l0 + q G8, q < n_my.  With PARTS > 1 and
// a last round of at most G8 / PARTS tiles, those are shared out among PARTS work-groups each (item q_part, rows from row(q) on).
struct LastRound {
    unsigned n_my, q_part, part_tile, part_row;
    __device__ __forceinline__ unsigned tile(unsigned q, unsigned l0, unsigned G8) const { return q == q_part ? part_tile : l0 + q * G8; }
    __device__ __forceinline__ unsigned row(unsigned q) const { return q == q_part ? part_row : 0; }
};
template <int PARTS>
__device__ __forceinline__ LastRound last_round(unsigned n_local, unsigned G8, unsigned l0)
{
    const unsigned rounds = n_local / G8, left = n_local - rounds * G8;
    LastRound r{rounds + (l0 < left ? 1u : 0u), ~0u, 0, 0};
    if constexpr (PARTS > 1) {
        if (left * PARTS <= G8) {
            const bool mine = l0 < left * PARTS;
            r = LastRound{rounds + (mine ? 1u : 0u), rounds, rounds * G8 + l0 / PARTS, l0 % PARTS * (256 / PARTS)};
        }
    }
    return r;
}

// The grid of a streaming launch (a work-group a CU) and into how many parts its last round's tiles go: by the XCD with the most.
struct StreamGrid { unsigned blocks; int parts; };
inline StreamGrid stream_grid_on(int cus, int64_t m_tiles, int n_tiles)
{
    const int64_t ids = (m_tiles + 7) / 8 * 8 * n_tiles;
    const int64_t most = cus / 8 * 8 < 8 ? 8 : cus / 8 * 8, per_xcd = ids / 8, left = per_xcd % (most / 8);
    const int parts = left == 0 || n_tiles > 4 ? 1 : left * 4 <= most / 8 ? 4 : left * 2 <= most / 8 ? 2 : 1;
    return StreamGrid{(unsigned)(ids < most && parts == 1 ? ids : most), parts};
}
inline hipError_t stream_grid(const GemmArgs &g, StreamGrid *out)
{
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    if ((g.m_tiles + 7) / 8 * 8 * g.n_tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    *out = stream_grid_on(cus, g.m_tiles, g.n_tiles);
    return hipSuccess;
}

}  // namespace ab
