// The append of one token to its ring slot as a launch of its own: word for
// word, one wave per item.  The read kernels append the token themselves; this
// one runs before them where their output takes the place of the token's
// arrays, which their other workgroups may still be reading.
#include <hip/hip_runtime.h>

#include "../args.h"

namespace skssm {

__global__ __launch_bounds__(64) void append_token_kernel(const AppendArgs a) {
  const size_t item = blockIdx.x, slot = item * (size_t)a.W + a.n;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const uint32_t w = a.words[f];
    for (uint32_t i = threadIdx.x; i < w; i += 64) a.dst[f][slot * w + i] = a.src[f][item * w + i];
  }
}

int run_append_token(const AppendArgs& a, size_t items, void* stream) {
  hipLaunchKernelGGL(append_token_kernel, dim3((unsigned)items), dim3(64), 0, static_cast<hipStream_t>(stream), a);
  return 0;
}

}  // namespace skssm
