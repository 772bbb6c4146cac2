// Kernel launch without the runtime's configuration stack, which <<<>>> and hipLaunchKernelGGL push and pop around the same
// call (2.4 us of host time a launch with it, 2.2 without; a KiB of arguments costs 0.1, eight arguments more 0.05).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <tuple>
#include <utility>

namespace kvb {

template <typename Args, std::size_t... I>
inline hipError_t launch_packed(const void *kernel, dim3 grid, dim3 block, hipStream_t stream, Args &args, std::index_sequence<I...>)
{
    void *ptrs[] = {(void *)&std::get<I>(args)...};
    return hipLaunchKernel(kernel, grid, block, ptrs, 0, stream);
}

// The arguments are converted to the kernel's parameter types; an error is left for hipGetLastError as well.
template <typename... P, typename... A>
inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t stream, const A &...args)
{
    static_assert(sizeof...(P) == sizeof...(A), "one argument per parameter");
    std::tuple<typename std::remove_cv<P>::type...> packed(static_cast<P>(args)...);
    return launch_packed((const void *)kernel, grid, block, stream, packed, std::index_sequence_for<P...>{});
}

}  // namespace kvb
