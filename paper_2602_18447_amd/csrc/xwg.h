// Hand-over of values between workgroups inside one launch: device-scope relaxed atomic stores and loads, which are
// written through to, and served from, the memory side of the per-XCD L2 caches, and an arrival counter that is bumped
// only after the stores are acknowledged.  Nobody waits for anybody: the workgroup that arrives last does the rest.
#pragma once
#include <hip/hip_runtime.h>

namespace cs {

__device__ inline void xwg_store(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The same with 16 bytes per lane (there is no atomic access of that width; each 4-byte part is one on its own, which is all
// a hand-over needs): the store in assembly.  Loads, of 16 or 8 bytes, are buffer loads at device scope from wave-uniform `base` plus a
// byte offset per lane; offsets at or past `bytes` read zeros.
typedef __attribute__((ext_vector_type(4))) float xwg_f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned xwg_u32x4;
__device__ inline void xwg_store4(xwg_f32x4 *p, xwg_f32x4 v) { asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory"); }
struct XwgLoads {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ XwgLoads(const void *base, unsigned bytes) : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000)) {}
    __device__ xwg_f32x4 load4(unsigned off) const {
        constexpr int SC1 = 1 << 4;
        return __builtin_bit_cast(xwg_f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, SC1));
    }
    __device__ float2 load2(unsigned off) const {
        constexpr int SC1 = 1 << 4;
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)off, 0, SC1));
    }
};
// Every thread calls it after its hand-over stores: waits until they are acknowledged, then counts the workgroup in.
// Returns true (to all threads) for the workgroup that arrives last of n; that one also clears the counter.
__device__ inline bool xwg_arrive_last(int32_t *cnt, int n, volatile int *flag, int tid) {
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    if (tid == 0) {
        int last = atomicAdd(cnt, 1) == n - 1;
        if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = last;
    }
    __syncthreads();
    return *flag != 0;
}

}  // namespace cs
