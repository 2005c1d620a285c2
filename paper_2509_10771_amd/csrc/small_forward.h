// Layer-fused inference of networks with hidden layers of up to 128 units for up to 2048 rows: the chain of one workgroup is what a
// call takes, so everything is made to shorten it.  One workgroup (8 wavefronts) carries 16 rows of one network; a wavefront owns 16
// columns of every layer, so no sums are exchanged and a layer costs one barrier.  All weights and biases of its columns, and the
// noise of the Gaussian head, are requested or formed before the rows arrive.  Operands, LDS layout and the handling of values
// without a split are those of small_step.h; weights are split in registers.
// act() in the wider kernel (fused_forward.hip, 32 rows) and here, us; with two rounds of workgroups the wider one is faster:
//   [48, 128, 128, 12]    64 rows 14.4,  8.1    2048 rows 15.3,  9.1    3000 rows 15.4, 17
//   [235, 128, 128, 12]   64 rows 19.1, 11.9    2048 rows 19.8, 12.6
//   [100, 128, 4]         64 rows 10.6,  8.4
#pragma once

#include "small_step.h"

namespace rslx {

namespace {

constexpr int SF_HIDDEN = 128, SF_IN = 256, SF_OUT = 64;
constexpr int SF_STEPS = SF_HIDDEN / 32;

// Columns 16 t + m of the weights, contraction indices 32 s + 8 kq .. + 7 of STEPS steps.  Rows and columns past the end repeat the
// last ones: the former meet zeros, the latter's sums are dropped.
template <int STEPS>
__device__ __forceinline__ void sf_request(const float* W, int K, int N, int wave, int m, int kq, float (&w)[STEPS][8]) {
  const uint32_t col = (uint32_t)min(16 * wave + m, N - 1);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (32 * s >= K) break;
#pragma unroll
    for (int i = 0; i < 8; ++i) w[s][i] = W[(uint32_t)min(32 * s + 8 * kq + i, K - 1) * (uint32_t)N + col];
  }
}

template <int STEPS>
__device__ __forceinline__ void sf_split(const float (&w)[STEPS][8], int K, SsWeights<STEPS>& p) {
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (32 * s >= K) break;
    uint32_t q[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair(SPLIT_SCALE * w[s][2 * i], SPLIT_SCALE * w[s][2 * i + 1], q[0][i], q[1][i], q[2][i]);
#pragma unroll
    for (int i = 0; i < 3; ++i) p.u[s][i] = make_uint4(q[i][0], q[i][1], q[i][2], q[i][3]);
  }
}

// LDS: the activations of two layers, then outputs, noise and sigma of the head.  IN: contraction steps of 32 of the first layer.
template <int IN>
struct SfLds {
  static constexpr int COLS = 32 * (IN > SF_STEPS ? IN : SF_STEPS), C = 3 * SS_PLANE * COLS;
  static constexpr int TOTAL = 2 * C + 4 * (2 * SF_OUT * SS_ROWS + 2 * SF_OUT);
};
constexpr int SF_MAX_LDS = SfLds<SF_IN / 32>::TOTAL;

// Rows 16 block .. of a network of L layers; lds: SfLds<IN>::TOTAL bytes.
template <int IN, int L>
__device__ __forceinline__ void small_forward(const FusedForwardArgs& args, const FusedNet& net, int block, char* lds) {
  constexpr int COLS = SfLds<IN>::COLS;
  char* const C[2] = {lds, lds + SfLds<IN>::C};
  float* const out = reinterpret_cast<float*>(lds + 2 * SfLds<IN>::C);
  float* const noise = out + SF_OUT * SS_ROWS;
  float* const sig = noise + SF_OUT * SS_ROWS;
  const int row0 = block * SS_ROWS;
  if (row0 >= args.n_rows) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kq = lane >> 4;
  int dim[L + 1];
  const float* W[L + 1];             // the last one: log_std
  W[0] = net.params;
#pragma unroll
  for (int l = 0; l <= L; ++l) {
    dim[l] = net.dims[l];
    if (l > 0) W[l] = W[l - 1] + (long)(dim[l - 1] + 1) * dim[l];
  }
  const int A = dim[L];

  // ---- requests: rows, weights, biases ----
  const int lrow = tid & 15, lj = tid >> 4, row = row0 + lrow;
  const bool row_ok = row < args.n_rows;
  const int D = dim[0], Dc = ss_pad(D, 32);
  constexpr int PASSES = (IN * 8 * SS_ROWS + SS_THREADS - 1) / SS_THREADS;
  float x[PASSES][4];
  {
    const bool vec = net.col_map == nullptr && (D & 3) == 0 && (net.ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(net.x) & 15) == 0;
    const float* xr = net.x + (long)min(row, args.n_rows - 1) * net.ldx;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int c = 4 * (lj + 32 * i);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[i][k] = 0.f;
      if (!row_ok || c >= D) continue;
      if (vec) {
        const float4 q = *reinterpret_cast<const float4*>(xr + c);
        x[i][0] = q.x; x[i][1] = q.y; x[i][2] = q.z; x[i][3] = q.w;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (c + k < D) x[i][k] = xr[net.col_map != nullptr ? net.col_map[c + k] : c + k];
      }
    }
  }
  float w0[IN][8], w[L - 1][SF_STEPS][8], bias[L][4];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    if (16 * wave < dim[l + 1]) {
      if (l == 0) sf_request<IN>(W[0], D, dim[1], wave, m, kq, w0);
      else sf_request<SF_STEPS>(W[l], dim[l], dim[l + 1], wave, m, kq, w[l > 0 ? l - 1 : 0]);
#pragma unroll
      for (int r = 0; r < 4; ++r) bias[l][r] = (W[l + 1] - dim[l + 1])[min(16 * wave + 4 * kq + r, dim[l + 1] - 1)];
    }
  }
  if (net.head) {
    if (tid < A) {
      const float ls = W[L][tid];
      sig[2 * tid] = ls;
      sig[2 * tid + 1] = expf(ls);
    }
    for (int e = tid; e < SS_ROWS * A; e += SS_THREADS) {
      const int r = e & 15;
      const long o = (long)(row0 + r) * A + (e >> 4);
      float eps = 0.f;
      if (!args.deterministic && row0 + r < args.n_rows) {
        if (args.eps != nullptr) {
          eps = args.eps[o];
        } else {
          const uint64_t nb = args.step_dev != nullptr ? ff_mix64(args.noise_pre ^ (uint64_t)*args.step_dev) : args.noise_base;
          const uint64_t h = ff_mix64(nb ^ (uint64_t)o);
          const float u1 = (float)((uint32_t)(h >> 40) + 1u) * 5.9604644775390625e-08f;
          const float u2 = (float)((uint32_t)(h >> 8) & 0xFFFFFFu) * 5.9604644775390625e-08f;
          eps = sqrtf(-2.0f * logf(u1)) * cospif(2.0f * u2);
        }
      }
      noise[e] = eps;
    }
  }
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    const int c = 4 * (lj + 32 * i);
    if (c < Dc) ss_put_c(C[0], COLS, c, lrow, ss_split(x[i]));
  }
  SsWeights<IN> p0;
  if (16 * wave < dim[1]) sf_split<IN>(w0, D, p0);
  __syncthreads();

  // ---- layers ----
  SsWeights<SF_STEPS> p;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int K = dim[l], N = dim[l + 1];
    const char* from = C[l & 1];
    if (16 * wave < N) {
      f32x4 acc;
      if (l == 0) acc = ss_product<IN>(p0, K, from, COLS, m, kq);
      else acc = ss_product<SF_STEPS>(p, K, from, COLS, m, kq);
      const int c = 16 * wave + 4 * kq;
      if (ss_any_nonfinite(acc)) ss_repeat(W[l], N, 1, K, 16 * wave, N, from, COLS, m, kq, acc);
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = acc[r] + bias[l][r];
      if (l + 1 < L) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = c + r < N ? ff_elu(v[r], net.alpha) : 0.f;
        ss_put_c(C[(l + 1) & 1], COLS, c, m, ss_split(v));
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (net.head) out[(c + r) * SS_ROWS + m] = v[r];
          if (c + r < N && row0 + m < args.n_rows) net.out[(long)(row0 + m) * N + c + r] = v[r];
        }
      }
    } else if (l + 1 < L && 16 * wave < ss_pad(N, 32)) {          // zeros up to the next whole step
      ss_put_c(C[(l + 1) & 1], COLS, 16 * wave + 4 * kq, m, Parts{});
    }
    if (l + 1 < L && 16 * wave < dim[l + 2 <= L ? l + 2 : L]) sf_split<SF_STEPS>(w[l], N, p);
    if (l + 1 < L || net.head) __syncthreads();
  }

  // ---- Gaussian head (actor only): lanes of (row, component), and one lane per row for its log-density ----
  if (!net.head) return;
  for (int e = tid; e < SS_ROWS * A; e += SS_THREADS) {
    const int r = e & 15, j = e >> 4;
    if (row0 + r >= args.n_rows) continue;
    const long o = (long)(row0 + r) * A + j;
    args.actions[o] = out[e] + sig[2 * j + 1] * noise[e];
    args.sigma[o] = sig[2 * j + 1];
  }
  if (wave == SS_WAVES - 1 && lane < SS_ROWS && row0 + lane < args.n_rows) {
    float zz = 0.f, sum_ls = 0.f;
#pragma unroll 4
    for (int j = 0; j < A; ++j) {
      const float mean = out[j * SS_ROWS + lane], sg = sig[2 * j + 1];
      const float act = mean + sg * noise[j * SS_ROWS + lane];
      const float z = (act - mean) / sg;
      zz += __fmul_rn(z, z);         // rounded by itself, as the wider kernel's
      sum_ls += sig[2 * j];
    }
    args.logp[row0 + lane] = -0.5f * zz - sum_ls - 0.5f * (float)A * FF_LOG_2PI;
  }
}

template <int IN, int L>
__global__ __launch_bounds__(SS_THREADS, 2) void small_forward_kernel(const FusedForwardArgs args) {
  __shared__ __align__(16) char lds[SfLds<IN>::TOTAL];
  small_forward<IN, L>(args, args.net[blockIdx.y], blockIdx.x, lds);
}

// The same for a network of any sizes that small_forward_takes; lds: SF_MAX_LDS bytes.
template <int IN>
__device__ __forceinline__ void small_forward_depth(const FusedForwardArgs& args, const FusedNet& net, int block, char* lds) {
  if (net.n_layers == 2) small_forward<IN, 2>(args, net, block, lds);
  else if (net.n_layers == 3) small_forward<IN, 3>(args, net, block, lds);
  else small_forward<IN, 4>(args, net, block, lds);
}
__device__ __forceinline__ void small_forward_any(const FusedForwardArgs& args, const FusedNet& net, int block, char* lds) {
  if (net.dims[0] <= 64) small_forward_depth<2>(args, net, block, lds);
  else if (net.dims[0] <= 128) small_forward_depth<4>(args, net, block, lds);
  else small_forward_depth<8>(args, net, block, lds);
}

// Two networks of different depths.  (A template so that its code lies behind the other kernels'.)
template <int = 0>
__global__ __launch_bounds__(SS_THREADS, 2) void small_uneven_kernel(const FusedForwardArgs args) {
  __shared__ __align__(16) char lds[SF_MAX_LDS];
  small_forward_any(args, args.net[blockIdx.y], blockIdx.x, lds);
}

template <int IN>
void launch_small_in(const FusedForwardArgs& a, hipStream_t stream) {
  const dim3 grid((a.n_rows + SS_ROWS - 1) / SS_ROWS, a.n_nets), block(SS_THREADS);
  switch (a.net[0].n_layers) {
    case 2: hipLaunchKernelGGL((small_forward_kernel<IN, 2>), grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL((small_forward_kernel<IN, 3>), grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL((small_forward_kernel<IN, 4>), grid, block, 0, stream, a); break;
  }
}

// Networks that this takes; the choice is made per network and by the row count alone.
bool small_forward_takes(const FusedNet& n, int n_rows) {
  if (n.n_layers < 2 || n.n_layers > 4 || n.dims[0] > SF_IN || n.dims[n.n_layers] > SF_OUT || n_rows > 2048) return false;
  for (int l = 1; l < n.n_layers; ++l)
    if (n.dims[l] > SF_HIDDEN) return false;
  return true;
}

hipError_t launch_small_forward(const FusedForwardArgs& a, hipStream_t stream) {
  int widest = 0;
  for (int i = 0; i < a.n_nets; ++i) widest = std::max(widest, a.net[i].dims[0]);
  if (widest <= 64) launch_small_in<2>(a, stream);
  else if (widest <= 128) launch_small_in<4>(a, stream);
  else launch_small_in<8>(a, stream);
  return hipGetLastError();
}

hipError_t launch_small_uneven(const FusedForwardArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((small_uneven_kernel<0>), dim3((a.n_rows + SS_ROWS - 1) / SS_ROWS, 2), dim3(SS_THREADS), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

}  // namespace rslx
