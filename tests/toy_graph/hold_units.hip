// hold_units.hip - holds compute units for a while (test program, not part of the library): every block takes the whole
// LDS of a unit, so that nothing else that needs LDS runs there.  A block ends after `ticks` of the 100 MHz clock, and
// in any case after a million looks at it.
#include <hip/hip_runtime.h>
#include <stdint.h>

static __global__ __launch_bounds__(64) void hold_units_kernel(uint64_t ticks, uint32_t* looks) {
  extern __shared__ uint32_t s_all[];
  const uint64_t begin = wall_clock64();
  uint32_t n = 0;
  while (n < 1000000u && wall_clock64() - begin < ticks) {
    __builtin_amdgcn_s_sleep(64);
    ++n;
  }
  if (threadIdx.x == 0) {
    s_all[0] = n;
    looks[blockIdx.x] = s_all[0];
  }
}

// looks: device uint32_t [blocks].
extern "C" int hold_units(uint32_t blocks, uint64_t ticks, uint32_t* looks, void* hip_stream) {
  constexpr int kLds = 160 * 1024;
  hipError_t rc = hipFuncSetAttribute((const void*)hold_units_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (rc != hipSuccess) return (int)rc;
  hold_units_kernel<<<dim3(blocks), dim3(64), kLds, (hipStream_t)hip_stream>>>(ticks, looks);
  return (int)hipGetLastError();
}
