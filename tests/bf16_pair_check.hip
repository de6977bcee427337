// Test helper (test_gpu_bf16_pair.py): the paired BF16 rounding of two increments
// beside the single one, on the same values, by the kernels' own functions.
#include "../paper_2308_06196_amd/csrc/bgk_device.hpp"

using namespace bgk;

__global__ void k_pair(const float* o, const float* base, int n, uint32_t* word, uint32_t* want,
                       float* stored, float* stored_want) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float o0 = o[2 * i], o1 = o[2 * i + 1], b0 = base[2 * i], b1 = base[2 * i + 1];
  float s0, s1, t0, t1;
  word[i] = bf16_increment2(o0, o1, b0, b1, s0, s1);
  const uint32_t lo = bf16_increment(o0, b0, t0), hi = bf16_increment(o1, b1, t1);
  want[i] = lo | hi << 16;
  stored[2 * i] = s0;
  stored[2 * i + 1] = s1;
  stored_want[2 * i] = t0;
  stored_want[2 * i + 1] = t1;
}

// Device arrays: o, base, stored, stored_want of 2 n values, word, want of n.
extern "C" int bf16_pair_check(const float* o, const float* base, int n, uint32_t* word,
                               uint32_t* want, float* stored, float* stored_want) {
  if (n <= 0) return 1;
  hipLaunchKernelGGL(k_pair, dim3((n + 255) / 256), dim3(256), 0, nullptr, o, base, n, word, want,
                     stored, stored_want);
  return hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess ? 0 : 1;
}
