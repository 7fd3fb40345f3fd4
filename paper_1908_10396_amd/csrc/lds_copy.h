// Copies from memory straight to LDS whose end the kernel waits for itself.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace avq {

// 16 bytes a lane from `src` to dst + 16 lane (dst: LDS, the same for the whole wave). As an instruction of its own rather
// than the builtin: before any read of LDS that might alias the target of a copy known to it the compiler waits for all loads
// in flight, those of a later stage too. The caller waits (s_waitcnt vmcnt; loads end in order) before it reads the place, and has
// read what was there before it calls this. (M0 holds the place; a wait state lies between its write and its use.)
__device__ __forceinline__ void lds_copy16(const void *src, void *dst)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"((uint64_t)(uintptr_t)src) : "m0", "memory");
}

// 4 bytes a lane, to dst + 4 lane.
__device__ __forceinline__ void lds_copy4(const void *src, void *dst)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(at), "v"((uint64_t)(uintptr_t)src) : "m0", "memory");
}

// 16 bytes a lane of what is read once and had better not displace what the caches hold.
__device__ __forceinline__ void lds_copy16_once(const void *src, void *dst)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "s"(at), "v"((uint64_t)(uintptr_t)src) : "m0", "memory");
}

} // namespace avq
