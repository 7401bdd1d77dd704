// Conversion of fp32 to bf16 bits on the device.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dmrg {

__device__ inline uint16_t f2bf(float x) {
  // round to nearest even
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);  // inf / nan
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

}  // namespace dmrg
