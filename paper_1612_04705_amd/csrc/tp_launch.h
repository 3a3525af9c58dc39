// Kernel launches that return their own status.  The <<< >>> form drops it, and
// the runtime's last error is the whole process's: an error that another call
// left unread stands there after a good launch.
#pragma once

#include <hip/hip_runtime.h>

namespace tpk {

template <typename T> struct Same { typedef T t; };

template <typename... P>
hipError_t launch(void (*kernel)(P...), unsigned grid, unsigned block, size_t lds, hipStream_t st,
                  typename Same<P>::t... args)
{
    void *a[] = { const_cast<void *>(static_cast<const void *>(&args))... };
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), a, lds, st);
}

}  // namespace tpk
