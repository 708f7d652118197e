// Buffer accesses, LDS reads by address, an LDS-only barrier and the LDS limit, shared by the kernels on the 6-bit matrix instruction.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hq_int_gemm_kernel.h"

namespace {

// Barrier that orders LDS only: __syncthreads() would also wait for the wave's global loads (weights requested
// ahead) and stores.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Buffer accesses: uniform base and bound in scalar registers, a 32-bit offset per lane; loads beyond the bound
// return zeros, stores beyond it are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, static_cast<int>(bytes), 0x00027000);
}
__device__ __forceinline__ v4i buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off) {
    return __builtin_bit_cast(
        v4i, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(lane_off), static_cast<int>(uniform_off), 0));
}
__device__ __forceinline__ void buffer_store16(const v4i &v, __amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, static_cast<int>(lane_off),
                                           static_cast<int>(uniform_off), 0);
}

// LDS reads at an address that is already one of LDS (no base to add)
typedef int v2i __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v4i lds_v4i(int address, int offset = 0) {
    return *reinterpret_cast<const __attribute__((address_space(3))) v4i *>(static_cast<uint32_t>(address) + offset);
}
__device__ __forceinline__ v2i lds_v2i(int address, int offset = 0) {
    return *reinterpret_cast<const __attribute__((address_space(3))) v2i *>(static_cast<uint32_t>(address) + offset);
}

constexpr int kLdsPerCu = 163840;

// Dynamic LDS beyond the default limit has to be allowed once per kernel and device.
inline hq_status allow_lds(const void *fn, std::atomic<uint64_t> &done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return HQ_ERR_LAUNCH;
    if ((done.load(std::memory_order_acquire) >> dev) & 1) return HQ_OK;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu) != hipSuccess) return HQ_ERR_LAUNCH;
    done.fetch_or(1ull << dev, std::memory_order_release);
    return HQ_OK;
}

}  // namespace
