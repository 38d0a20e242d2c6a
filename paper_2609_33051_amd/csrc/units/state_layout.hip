// Conversion of the recurrent state between the row layout X[v][k] (X = S^T,
// the transpose of the paper's K x V state, per item) and the tile-major
// layout the kernels read and write: 16 x 16 tiles (vt, kt), vt-major, each
// 1 KB contiguous with lane l of a wave holding X[16 vt + l%16][16 kt +
// 4 (l/16) + i] at 4 l + i (the register layout of the flush's MFMA
// accumulators).
//
// Sixteen rows of X (a stripe: 64 K bytes) and their K / 16 tiles are the same
// contiguous run in both layouts, so the conversion permutes float4s within
// runs of 4 or 8 KB.  One wave per stripe reads it in 1 KB runs, permutes it
// through LDS and writes it in 1 KB runs; a stripe is read once and, being the
// whole of what the wave holds, in flight only briefly.  Reading the row side
// straight in the tiles' order (16 pieces of 64 bytes a load) moved 2 GiB at
// 4.6 TB/s.  The reads are non-temporal at every size: what reads the tiles next
// (the initial sketch) finds more of them in the last-level cache.  Conversion and
// offline-map sketch, K = V = 128, with ordinary reads / these: 64 MiB of states
// 53.3 / 42.7 us, 128 MiB 93.5 / 78.0 (rows not in cache), 38.4 / 36.6 and 71.1 /
// 66.5 (rows just written); alone and repeated on rows that stay in cache the
// conversion of 64 MiB takes 20.1 / 22.8.
#include <hip/hip_runtime.h>

#include "../args.h"
#include "../device.h"

namespace skssm {

template <int K, bool TO_TILES>
__global__ __launch_bounds__(64) void state_layout_kernel(const float4* src, float4* dst) {
  constexpr int N = K / 16, KQ = K / 4;  // float4s per lane; float4s per row
  __shared__ float4 buf[16 * KQ];
  const int lane = threadIdx.x;
  const size_t base = (size_t)blockIdx.x * (16 * KQ);
  float4 x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = ld_nt(src + base + 64 * i + lane);
  // LDS holds the stripe in tile order with the low three bits of the position
  // exchanged by the channel group's, so that both sides hit different banks
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int f = 64 * i + lane;
    if constexpr (TO_TILES) {
      const int r = f / KQ, c = f % KQ;  // row, channel group
      buf[((c >> 2) * 64 + r + 16 * (c & 3)) ^ (c & 7)] = x[i];
    } else {
      buf[f ^ ((f >> 4) & 7)] = x[i];    // (tile f / 64, group f / 16 % 4: channel group f / 16)
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int f = 64 * i + lane;
    float4 y;
    if constexpr (TO_TILES) {
      y = buf[f ^ ((f >> 4) & 7)];
    } else {
      const int r = f / KQ, c = f % KQ;
      y = buf[((c >> 2) * 64 + r + 16 * (c & 3)) ^ (c & 7)];
    }
    dst[base + f] = y;
  }
}

int run_state_layout(const float* src, float* dst, size_t items, int K, int V, int to_tiles, void* stream) {
  if ((K != 64 && K != 128) || V % 16) return -2;
  const dim3 grid((unsigned)(items * (size_t)(V / 16)));  // < 2^26 (the ABI bounds the items)
  hipStream_t s = static_cast<hipStream_t>(stream);
  const float4* a = reinterpret_cast<const float4*>(src);
  float4* b = reinterpret_cast<float4*>(dst);
  if (K == 128) {
    if (to_tiles) hipLaunchKernelGGL((state_layout_kernel<128, true>), grid, dim3(64), 0, s, a, b);
    else hipLaunchKernelGGL((state_layout_kernel<128, false>), grid, dim3(64), 0, s, a, b);
  } else {
    if (to_tiles) hipLaunchKernelGGL((state_layout_kernel<64, true>), grid, dim3(64), 0, s, a, b);
    else hipLaunchKernelGGL((state_layout_kernel<64, false>), grid, dim3(64), 0, s, a, b);
  }
  return 0;
}

}  // namespace skssm
