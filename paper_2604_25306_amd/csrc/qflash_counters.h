// Counters in LDS by which the wavefronts of a workgroup tell each other what has landed there.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace {

typedef __attribute__((address_space(3))) int lds_int;

// Wait until the counter at flag_addr (LDS) has reached target.  The LDS serves the requests of a
// wavefront in order, so the reads that follow in program order see what was written before the
// counter was; the empty statement only keeps the compiler from moving them up.
__device__ __forceinline__ void wait_count(int flag_addr, int target) {
    lds_int* f = (lds_int*)(size_t)flag_addr;
    while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target) __builtin_amdgcn_s_sleep(2);
    asm volatile("" ::: "memory");
}
// Add 1 to a counter after the loads it stands for have landed (the caller has waited for them).
// Written as an instruction of its own: the compiler would otherwise make every LDS access that it
// cannot tell apart from the destination of a direct load wait for all direct loads still in flight.
__device__ __forceinline__ void count_up(int flag_addr) {
    const int one = 1;
    asm volatile("ds_add_u32 %0, %1" ::"v"(flag_addr), "v"(one) : "memory");
}

}  // namespace
