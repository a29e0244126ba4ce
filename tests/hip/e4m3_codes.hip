// The low plane's conversion on the device against f32_to_e4m3, over every float up to 448.
#include "e4m3.h"

using namespace et;

constexpr uint32_t TOP = 0x43E00000u;  // 448
constexpr uint32_t VALUES = TOP + 1;   // bit patterns of one sign

// Four values of a thread: pattern i and those a quarter of the range on each, signs alternating
// (other codes in every byte).  bad: [0] the number of differing codes, [1] a pattern of one.
__global__ void __launch_bounds__(256) k_codes(uint32_t sign, uint32_t* bad) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < VALUES; i += (uint64_t)gridDim.x * 256) {
    float x[4];
    for (int k = 0; k < 4; ++k) {
      const uint32_t u = (uint32_t)((i + (uint64_t)k * (VALUES / 4 + 1)) % VALUES);
      x[k] = __uint_as_float(u | ((sign ^ (uint32_t)k) & 1u) << 31);
    }
    const uint32_t got = pack_e4m3(x);
    for (int k = 0; k < 4; ++k) {
      const uint32_t g = got >> (8 * k) & 0xFFu, want = f32_to_e4m3(x[k]);
      if (g != want && !((g & 0x7Fu) == 0u && want == 0u)) {
        atomicAdd(&bad[0], 1u);
        bad[1] = __float_as_uint(x[k]);
      }
    }
  }
}

// bad: two words on the device, zeroed by the caller.  Returns the HIP status.
extern "C" int e4m3_codes(uint32_t* bad) {
  for (uint32_t sign = 0; sign < 2; ++sign)
    hipLaunchKernelGGL(k_codes, dim3(8192), dim3(256), 0, nullptr, sign, bad);
  const hipError_t e = hipGetLastError();
  return (int)(e != hipSuccess ? e : hipDeviceSynchronize());
}
