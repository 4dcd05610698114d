// The end of the vocabulary products in which a wavefront has a block of 32 columns: logits, and the retrieve stage's statistics of the block.
#pragma once
#include "lsq_internal.h"

namespace lsq {

// Lane: row m, columns 8 vg + 4 (lane >> 5) + 0..3 of the block; value(vg, e) says what they are, store(n, v) keeps columns n .. n + 3.
// stats (may be null): [row][groups] pairs (largest, sum of exponentials), in the order of gemm_f16_skinny_kernel, whose wavefronts have eight columns each.
// EXACT: its bits too.
template <bool EXACT, typename V, typename S>
__device__ __forceinline__ void vocabulary_block(V&& value, S&& store, float* stats, int groups, int m, int block, int M, int N, int lane) {
  auto merge = [](float& m1, float& z1, float m2, float z2) {
    if constexpr (EXACT) merge_stat_exact(m1, z1, m2, z2);
    else merge_stat(m1, z1, m2, z2);
  };
  float mx = -INFINITY, z = 0.f;
#pragma unroll
  for (int vg = 0; vg < 4; ++vg) {
    const int n = block * 32 + vg * 8 + (lane >> 5) * 4;
    float v[4], vm = -INFINITY, vz = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = value(vg, e);
    if (m < M && n < N) store(n, v);
    if (!stats) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) vm = fmaxf(vm, v[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) vz += __expf(v[e] - vm);
    const float m2 = lane_xor<32>(vm), z2 = lane_xor<32>(vz);
    merge(vm, vz, m2, z2);
    if (vg == 0) { mx = vm; z = vz; }
    else merge(mx, z, vm, vz);
  }
  if (stats && lane < 32 && m < M) {
    float* st = stats + ((size_t)m * groups + block) * 2;
    st[0] = mx;
    st[1] = z;
  }
}

}  // namespace lsq
