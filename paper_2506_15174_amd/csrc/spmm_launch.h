// Kernel launches of the executors (internal).
#ifndef SPMM_LAUNCH_H
#define SPMM_LAUNCH_H

#include <hip/hip_runtime.h>

#include <type_traits>

// Launches `kernel` and answers whether that worked.  Short products follow each other as fast as the host launches them,
// and what `<<< >>>` does besides, handing the runtime the launch's shape in one call and taking it back in a second, and asking for the
// last error in a third, is 0.25 us of the 2.5 that a launch of an empty kernel then takes (this one 2.2).
template <typename... P> inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, unsigned threads, unsigned lds, hipStream_t stream, std::remove_const_t<P>... args)
{
    void *pointers[] = {&args...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, dim3(threads), pointers, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();  // the answer says it: not to be found by whoever asks next
    return e;
}

#endif
