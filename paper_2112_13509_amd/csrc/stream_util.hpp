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

}  // namespace ab
