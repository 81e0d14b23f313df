// wf_lds_dma.h -- memory-to-LDS copies and the explicit waits of the kernels
// that pipeline them (gfx950).  Internal header; not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace wf {

#define WF_LDS(T) __attribute__((address_space(3))) T

template <int N>
using ic = std::integral_constant<int, N>;

// 32-bit LDS byte address of a __shared__ object.
__device__ __forceinline__ unsigned lds_addr(const void *p) {
    return (unsigned)(uintptr_t)(const WF_LDS(char) *)p;
}

// s_waitcnt vmcnt(n) for the few counts the pipeline needs (n must be a
// compile-time immediate).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt immediate out of range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// HBM -> LDS copy of 16 bytes per lane: lane L's 16 bytes, addressed as a
// wave-uniform 64-bit base (SGPRs) plus a 32-bit per-lane byte offset, land
// at LDS byte lds + 16*L (lds wave-uniform).  Written as inline assembly so
// the compiler does not know these loads write LDS: it would otherwise make
// every LDS read wait for all of them.  Completion is tracked by the
// explicit vmcnt waits of the pipeline.
// NT: with the non-temporal hint, for tiles that only this workgroup reads.
template <bool NT = false>
__device__ __forceinline__ void lds_dma16_so(const char *base, unsigned voff, unsigned lds) {
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, %1 nt"
                     :
                     : "v"(voff), "s"(base), "s"(lds)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(voff), "s"(base), "s"(lds)
                     : "memory", "m0");
}

// The same with a 64-bit address per lane, for sources whose rows can lie
// 4 GB apart.
template <bool NT = false>
__device__ __forceinline__ void lds_dma16(const char *src, unsigned lds) {
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, off nt"
                     :
                     : "v"(src), "s"(lds)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %0, off"
                     :
                     : "v"(src), "s"(lds)
                     : "memory", "m0");
}

}  // namespace wf
