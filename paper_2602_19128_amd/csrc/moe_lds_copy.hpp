// Direct global -> LDS copies, as the grouped GEMMs and the router's logits issue them, and the waits for them.
#pragma once
#include "moe_internal.hpp"

namespace moe {
namespace {

#define MOE_WAIT_VMCNT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory")

// Direct global -> LDS copies, one instruction per wavefront: lane l moves 16 (or 4) bytes from its
// own global address to LDS byte address lds_base + 16*l (4*l).  Written as inline assembly so that
// the compiler's wait-count bookkeeping of the ordinary LDS reads stays exact (it otherwise falls
// back to full waits whenever such a copy is pending); the copies are tracked by hand with
// MOE_WAIT_VMCNT.  lds_base must be wavefront-uniform.
__device__ __forceinline__ uint32_t lds_addr_of(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)(p);
}
// m0 (the LDS base of such a copy) is named as clobbered so that the compiler never carries a value of
// its own in m0 across these statements; clang notes that it does not save reserved registers, which
// is what is wanted here.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT>
__device__ __forceinline__ void copy16_to_lds(const void *g, uint32_t lds_base)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds_base), "v"(g) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(g) : "memory", "m0");
}
__device__ __forceinline__ void copy4_to_lds(const void *g, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_base), "v"(g) : "memory", "m0");
}
// The same with a wavefront-uniform base and a 32-bit offset per lane.
template <bool NT>
__device__ __forceinline__ void copy16_to_lds_at(const void *base, uint32_t off, uint32_t lds_base)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_base), "v"(off), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace
}  // namespace moe
