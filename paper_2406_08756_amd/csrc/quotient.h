// Division of tile indices by numbers that the host knows.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace lynx {

// x / d (x >= 0, d > 0) by inv = inverse(d, most), x <= most: two scalar instructions, where a division takes about 25, and
// a wavefront issues one in 4 to 5 clocks before it can ask for its first operands (with the other instructions
// that went at the same time, before the first loads: a layer of 768 tokens of h 512, 22 launches, 121.0 -> 118.6 us).
// With inv = ceil(2^31 / d), x inv / 2^31 is above x / d by less than 1 / d as long as x d < 2^31; elsewhere inv is 0,
// and quotient() divides.
inline uint32_t inverse(long long d, long long most) {
  return most * d < (1ll << 31) ? static_cast<uint32_t>(((1ll << 31) + d - 1) / d) : 0u;
}
__host__ __device__ __forceinline__ int quotient(int x, int d, uint32_t inv) {
  return inv != 0 ? static_cast<int>((static_cast<uint64_t>(static_cast<uint32_t>(x) << 1) * inv) >> 32) : x / d;
}

}  // namespace lynx
