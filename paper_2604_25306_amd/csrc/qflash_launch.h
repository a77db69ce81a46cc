// Host side of a forward launch, shared by every kernel family: per-process and per-device set-up of a
// kernel on its first launch, then the launch itself.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

#include "qflash_internal.h"

// Launches KERN on the current device (args.device).  First launch per process and device: raise the
// dynamic LDS limit, make sure that the kernel has no static LDS in front of the dynamic one (the index
// into the weight table is used as an LDS address; static_lds_ok for kernels without dynamic LDS), and
// look the kernel up by its symbol once: a launch by function handle costs the host 2.4 us, by symbol 2.6.
template <class Args, void (*KERN)(const Args)>
int qflash_launch_function(const QflashKernelArgs& args, unsigned grid, unsigned threads, size_t lds, int lds_limit,
                         hipStream_t stream, bool static_lds_ok) {
    static std::once_flag once[kQflashMaxDevices];
    static int status[kQflashMaxDevices];
    static hipFunction_t func[kQflashMaxDevices];
    const int dev = args.device;
    if (dev < 0 || dev >= kQflashMaxDevices) return (int)hipErrorInvalidDevice;
    std::call_once(once[dev], [&] {
        hipFuncAttributes fa;
        hipError_t e = hipFuncGetAttributes(&fa, (const void*)KERN);
        if (e == hipSuccess && fa.sharedSizeBytes != 0 && !static_lds_ok) e = hipErrorInvalidValue;
        if (e == hipSuccess && !static_lds_ok)
            e = hipFuncSetAttribute((const void*)KERN, hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit);
        if (e == hipSuccess) e = hipGetFuncBySymbol(&func[dev], (const void*)KERN);
        status[dev] = (int)e;
    });
    if (status[dev] != 0) return status[dev];
    void* params[] = {const_cast<Args*>(static_cast<const Args*>(&args))};
    return (int)hipModuleLaunchKernel(func[dev], grid, 1, 1, threads, 1, 1, (unsigned)lds, stream, params, nullptr);
}

// The kernel takes all arguments or those of a launch with one set of constants.
template <void (*KERN)(const QflashKernelArgs)>
int qflash_launch_kernel(const QflashKernelArgs& args, unsigned grid, unsigned threads, size_t lds, int lds_limit,
                         hipStream_t stream, bool static_lds_ok = false) {
    return qflash_launch_function<QflashKernelArgs, KERN>(args, grid, threads, lds, lds_limit, stream, static_lds_ok);
}
template <void (*KERN)(const QflashLaunchArgs)>
int qflash_launch_kernel(const QflashKernelArgs& args, unsigned grid, unsigned threads, size_t lds, int lds_limit,
                         hipStream_t stream, bool static_lds_ok = false) {
    return qflash_launch_function<QflashLaunchArgs, KERN>(args, grid, threads, lds, lds_limit, stream, static_lds_ok);
}
