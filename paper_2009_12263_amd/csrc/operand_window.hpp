// How much of a plain operand a buffer descriptor covers.  Plain integer arithmetic without HIP: a CPU test compiles this header.
#pragma once
#include <stdint.h>

#ifndef FG_HOST_DEVICE
#ifdef __HIP__
#define FG_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FG_HOST_DEVICE inline
#endif
#endif

namespace fg {

// The byte offset of a lane that is to load zeros: beyond every descriptor that such a lane is loaded through.
constexpr uint32_t kOutOfRange = 0x80000000u;

// Size of a descriptor from which `rest` bytes of the operand are left: those, at most 2 GiB - 1.  The host keeps every offset that a
// lane forms below that, and a larger one would reach kOutOfRange: lanes beyond K then fetched what lies 2 GiB further on.
constexpr uint32_t kLargestWindow = 0x7fffffffu;
FG_HOST_DEVICE uint32_t window_bytes(int64_t rest) { return rest < 0 ? 0u : rest > (int64_t)kLargestWindow ? kLargestWindow : (uint32_t)rest; }

}  // namespace fg
