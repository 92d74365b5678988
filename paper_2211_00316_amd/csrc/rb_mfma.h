// Device helpers shared by the contraction kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

// Output row held by (lane, register i) of a 32x32 MFMA tile.
__device__ __forceinline__ int mfma_row(int lane, int i) {
    return (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
}

// 16 bytes per lane from the buffer to LDS: lane l writes lds + 16 l (lds wave-uniform).
template <typename T>
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, T *lds, uint32_t off,
                                           uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (__attribute__((address_space(3))) void *)lds, 16, (int)off, (int)soff, 0, 0);
}

// Wait until at most N global loads of this wave are outstanding and its LDS operations are
// done, then meet the other waves. Loads return in order, so the older step's operands are in
// LDS; after the barrier every wave's are.
template <int N>
__device__ __forceinline__ void lr_sync() {
    static_assert(N >= 0 && N < 64, "vmcnt");
    if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
