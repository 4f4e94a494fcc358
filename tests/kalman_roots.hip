// The filter's short square root, reciprocal and quotient compared, on the GPU,
// with the compiler's correctly rounded sqrtf and division (test_gpu_kalman_roots.py).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tpc_kalman.h"

using namespace tpc_kf;

namespace {

__device__ __forceinline__ uint64_t mix(uint64_t z) {  // splitmix64
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// a float of the given 23 bits of mantissa and binary exponent
__device__ __forceinline__ float make(uint32_t mantissa, int exponent) {
  return __uint_as_float((uint32_t(exponent + 127) << 23) | (mantissa & 0x7FFFFFu));
}

enum { SQRT, RCP, DIV_RCP, DIV_RSQ };

__global__ void __launch_bounds__(256) k_check(int what, uint64_t first, uint64_t count, unsigned long long *out) {
  unsigned long long bad = 0;
  for (uint64_t j = uint64_t(blockIdx.x) * 256 + threadIdx.x; j < count; j += uint64_t(gridDim.x) * 256) {
    const uint64_t i = first + j;
    float got, want;
    if (what == SQRT) {  // i: the bits of x
      const float x = __uint_as_float(uint32_t(i));
      float rs;
      got = sqrt_n(x, rs);
      want = sqrtf(x);
    } else if (what == RCP) {
      const float x = __uint_as_float(uint32_t(i));
      got = rcp_n(x);
      want = 1.f / x;
    } else {  // i: number of a pair
      const uint64_t h = mix(i), g = mix(~i);
      const float a = make(uint32_t(h), int(h >> 32 & 63) - 40) * (h >> 63 ? -1.f : 1.f);  // 2^-40 .. 2^24
      const float b = make(uint32_t(g), int(g >> 32 & 63) - 40);
      if (what == DIV_RCP) {
        got = div_by(a, b, rcp_n(b));
        want = a / b;
      } else {  // the divisor a root, its reciprocal from the root's own approximation
        float rs;
        const float c = sqrt_n(b, rs);
        got = div_by(a, c, refine_rcp(c, rs));
        want = a / c;
      }
    }
    bad += __float_as_uint(got) != __float_as_uint(want);
  }
  if (bad) atomicAdd(out, bad);
}

}  // namespace

// The number of values first .. first + count - 1 that differ; negative on a failure of the runtime.
extern "C" long long kalman_roots(int what, unsigned long long first, unsigned long long count) {
  unsigned long long *d = nullptr, n = 0;
  if (hipMalloc(&d, sizeof n) != hipSuccess) return -1;
  bool ok = hipMemcpy(d, &n, sizeof n, hipMemcpyHostToDevice) == hipSuccess;
  if (ok) {
    hipLaunchKernelGGL(k_check, dim3(8192), dim3(256), 0, nullptr, what, uint64_t(first), uint64_t(count), d);
    ok = hipGetLastError() == hipSuccess && hipMemcpy(&n, d, sizeof n, hipMemcpyDeviceToHost) == hipSuccess;
  }
  ok = hipFree(d) == hipSuccess && ok;
  return ok ? (long long)n : -1;
}
