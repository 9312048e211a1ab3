// Pointers that kernels take out of tables in memory (tile pointers, product descriptors).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nnt {

// The same pointer, known to point into device memory.  A kernel sees a pointer it has loaded as a generic one and
// would use it with FLAT instructions, which count as LDS accesses too: every wait for an LDS read or a scalar load
// then also waits for all such loads in flight, so nothing prefetched from memory ever overlaps with work on LDS.
// Tile data is always device memory, and through this its accesses are GLOBAL instructions.
template <typename T>
__device__ __forceinline__ T* in_global(T* p) {
    return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;      // (by way of an integer: a plain pair of casts is folded away)
}
template <typename T>
__device__ __forceinline__ T* global_as(void* p) { return in_global(static_cast<T*>(p)); }
template <typename T>
__device__ __forceinline__ T* global_as(const void* p) { return in_global(static_cast<T*>(p)); }

}  // namespace nnt
