// Holds CUs for a while: `blocks` blocks, of which no two fit a CU, that sleep
// until `ms` milliseconds have passed and then end.  Launched on `stream`.
#include <hip/hip_runtime.h>
#include <stdint.h>

__global__ void __launch_bounds__(1024) k_hold(uint64_t ticks, uint32_t* out) {
  __shared__ uint32_t lds[24 * 1024];  // 96 of 160 KiB
  for (int i = threadIdx.x; i < 24 * 1024; i += 1024) lds[i] = i;
  __syncthreads();
  const uint64_t t0 = wall_clock64();
  while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(64);
  out[blockIdx.x] = lds[(threadIdx.x * 7u + (uint32_t)ticks) % (24u * 1024u)];
}

extern "C" int hold_cus(int device, int blocks, double ms, uint32_t* out, void* stream) {
  int khz = 0;
  if (blocks < 1 || blocks > 256 || !(ms > 0.0) || ms > 2000.0) return -1;
  if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) != hipSuccess || khz < 1) return -2;
  hipLaunchKernelGGL(k_hold, dim3(blocks), dim3(1024), 0, (hipStream_t)stream, (uint64_t)(ms * khz), out);
  return (int)hipGetLastError();
}
