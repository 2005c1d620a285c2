// Split weights in the order in which the layer-fused inference (fused_forward.hip) reads them, for launches that write them.
#pragma once

#include "kernels.h"
#include "split_bf16.h"

namespace rslx {

// One layer's weights [K, N]: [64 columns][step of 32][column block][part][lane] units of 16 bytes, rows past K zero, columns past
// N those of the last.  Lane (m, kq) of column block cb holds column 4 m + cb at contraction indices 8 kq .. + 7 of the step.
constexpr int FP_STEP = 12 * 64;             // units of a step

__host__ __device__ inline int fused_pack_columns(int N) { return (N + 63) / 64 * 64; }
__host__ __device__ inline int fused_pack_steps(int K) { return (K + 31) / 32; }
__host__ __device__ inline long fused_pack_units(int K, int N) { return (long)(fused_pack_columns(N) / 64) * fused_pack_steps(K) * FP_STEP; }

__device__ __forceinline__ void fused_pack_unit(const FusedPackJob& J, int e) {
  const int cols = fused_pack_columns(J.N), steps = fused_pack_steps(J.K);
  const int kg = e / cols, c = e - kg * cols;
  if (kg >= 4 * steps) return;
  const float* src = J.src + min(c, J.N - 1);
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = src[(long)min(8 * kg + i, J.K - 1) * J.N];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = 8 * kg + i < J.K ? SPLIT_SCALE * v[i] : 0.f;
  uint4 part[3];
  split_pair(v[0], v[1], part[0].x, part[1].x, part[2].x);
  split_pair(v[2], v[3], part[0].y, part[1].y, part[2].y);
  split_pair(v[4], v[5], part[0].z, part[1].z, part[2].z);
  split_pair(v[6], v[7], part[0].w, part[1].w, part[2].w);
  uint4* dst = reinterpret_cast<uint4*>(J.dst) + (long)((c >> 6) * steps + (kg >> 2)) * FP_STEP + (c & 3) * 192 + (kg & 3) * 16 + ((c & 63) >> 2);
#pragma unroll
  for (int s = 0; s < 3; ++s) dst[64 * s] = part[s];
}

}  // namespace rslx
