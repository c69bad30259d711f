// limits.h -- bounds of the kernels' index arithmetic (host code, no HIP).
#pragma once
#include <stdint.h>

namespace lbem {

// Whether the byte offset of every one of `count` consecutive elements of `bytes`
// bytes fits 32 unsigned bits.
constexpr bool offsets32(int64_t count, int64_t bytes) { return count <= ((int64_t)1 << 32) / bytes; }

}  // namespace lbem
