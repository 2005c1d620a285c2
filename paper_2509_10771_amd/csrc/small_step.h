// Gradients of small networks over small minibatches in one launch: forward pass, loss and backward pass of an optimiser step.
// Where the launches per layer have a few workgroups each, a step is the sum of their latencies: 41 us in six launches (13.6 the
// loss head) at 384 rows and [48, 128, 128, 12] twice; this one takes 19.  It is a chain of some twenty phases of 0.3 to 1.9 us between
// barriers (2.5 the gathered rows, 1.6 the loss, 1.9 the widest weight gradient), bound by the latency of each.
//
// One workgroup (8 wavefronts) carries 16 rows of one network through everything and leaves its share of the weight gradients as
// one split of the partial sums that launch_reduce_partials adds up.  The products run on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16) with operands split in three (see gemm.hip); the weights come split from memory
// (launch_pack_weights), each unit used by one wavefront only, requested a phase ahead; values that stay in the workgroup are
// split when they are made and lie in LDS in two layouts:
//   C[part][column / 8][row][8 columns]   operand of the contractions over columns (forward, input gradient)
//   R[part][row / 8][column][8 rows]      operand of the contraction over the rows (weight gradient)
// C holds the layer that is being read, R the inputs of all layers and the gradient that is being read.  Sixteen rows fill half of
// a contraction of 32 in the weight gradients; the other half meets zeros.  Lane (m, kq) of a product holds outputs
// 16 t + 4 kq .. + 3 of row m: four consecutive columns, one 8-byte write per part to C.
#pragma once

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "ppo_row.h"
#include "split_bf16.h"

namespace rslx {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int SS_ROWS = 16, SS_THREADS = 512, SS_WAVES = SS_THREADS / 64;
constexpr int SS_MAX_OUT = 32;
constexpr int SS_PLANE = 2 * SS_ROWS;                     // LDS bytes of one part of one column, either layout
constexpr float SS_LOG_2PI = 1.8378770664093453f;

__host__ __device__ inline int ss_pad(int n, int m) { return (n + m - 1) / m * m; }

__host__ __device__ inline int ss_r_bytes(int n) { return 3 * SS_PLANE * ss_pad(n, 16); }

// LDS plan (bytes): R of the layers' inputs, R of a gradient, C, then small arrays.
struct SsLds {
  int r_dz, c, c_cols, small, total;                 // R of layer l's input lies behind those of the layers before, from 0
  __host__ __device__ SsLds(const int32_t* dims, int n_layers) {
    int o = 0, dz = SS_MAX_OUT;
    c_cols = SS_MAX_OUT;
    for (int l = 0; l < n_layers; ++l) {
      o += ss_r_bytes(dims[l]);
      c_cols = ss_pad(dims[l], 32) > c_cols ? ss_pad(dims[l], 32) : c_cols;
      if (l > 0) dz = ss_pad(dims[l], 16) > dz ? ss_pad(dims[l], 16) : dz;
    }
    r_dz = o; o += 3 * SS_PLANE * dz;
    c = o; o += 3 * SS_PLANE * c_cols;
    small = o; o += 4 * (2 * SS_MAX_OUT * SS_ROWS + 2 * SS_MAX_OUT) + 8 * SS_WAVES;
    total = o;
  }
};

struct Parts { uint32_t p[3][2]; };       // three parts of four values

// Parts of SPLIT_SCALE * v.  Values without a split (2^111 and above, infinite, NaN) have NaN for their first part and the two
// halves of their bits for the others: their products come out NaN, and ss_value finds the value for the repetition in fp32.
__device__ __forceinline__ Parts ss_split(const float (&v)[4]) {
  Parts q;
  float most = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    split_pair(SPLIT_SCALE * v[2 * i], SPLIT_SCALE * v[2 * i + 1], q.p[0][i], q.p[1][i], q.p[2][i]);
    most = fmaxf(most, fmaxf(fabsf(v[2 * i]), fabsf(v[2 * i + 1])));
  }
  if (most >= 0x1p111f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!(fabsf(v[i]) >= 0x1p111f)) continue;
      const uint32_t bits = __float_as_uint(v[i]), keep = 0xffff0000u >> (16 * (i & 1));
      const int sh = 16 * (i & 1);
      q.p[0][i / 2] = (q.p[0][i / 2] & keep) | (0x7fc0u << sh);
      q.p[1][i / 2] = (q.p[1][i / 2] & keep) | ((bits >> 16) << sh);
      q.p[2][i / 2] = (q.p[2][i / 2] & keep) | ((bits & 0xffffu) << sh);
    }
  }
  return q;
}

// The value whose parts (of negated values where `neg`) lie at u, `step` bytes apart; NaN for NaN.
__device__ __forceinline__ float ss_value(const char* u, int step, bool neg) {
  uint32_t p[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) p[s] = *reinterpret_cast<const uint16_t*>(u + s * step) ^ (neg ? 0x8000u : 0u);
  if ((p[0] & 0x7fffu) > 0x7f80u) return __uint_as_float((p[1] << 16) | p[2]);
  return (__uint_as_float(p[2] << 16) + __uint_as_float(p[1] << 16) + __uint_as_float(p[0] << 16)) * (1.0f / SPLIT_SCALE);
}

// Four columns c .. c + 3 (c % 4 == 0) of a row to C, negated in odd rows (see split_scale).
__device__ __forceinline__ void ss_put_c(char* C, int cols, int c, int row, const Parts& q) {
  const uint32_t flip = row & 1 ? 0x80008000u : 0u;
  char* u = C + ((c >> 3) * SS_ROWS + row) * 16 + (c & 4) * 2;
#pragma unroll
  for (int s = 0; s < 3; ++s) *reinterpret_cast<uint2*>(u + s * SS_PLANE * cols) = make_uint2(q.p[s][0] ^ flip, q.p[s][1] ^ flip);
}
// The same to R; `odd`: parity of the columns that are negated, 2 = none.
__device__ __forceinline__ void ss_put_r(char* R, int cols, int c, int row, const Parts& q, int odd) {
  char* u = R + ((row >> 3) * cols + c) * 16 + (row & 7) * 2;
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<uint16_t*>(u + s * SS_PLANE * cols + i * 16) = (uint16_t)((q.p[s][i / 2] >> (16 * (i & 1))) ^ ((i & 1) == odd ? 0x8000u : 0u));
}

__device__ __forceinline__ bool ss_any_nonfinite(const f32x4& a) {
  float z = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) z = fmaf(a[r], 0.f, z);
  return __any(!(z == 0.f));
}

__device__ __forceinline__ bf16x8 ss_unit(const char* u) { return *reinterpret_cast<const bf16x8*>(u); }

// Split weights of output column `col` for all contraction steps (layout of launch_pack_weights): all requested together.
template <int STEPS>
struct SsWeights { uint4 u[STEPS][3]; };
template <int STEPS>
__device__ __forceinline__ void ss_load_weights(const uint16_t* pack, int K, int cols, int col, int kq, SsWeights<STEPS>& w) {
  const uint4* P = reinterpret_cast<const uint4*>(pack);
  const int steps16 = (K + 15) / 16;
  const int c = min(col, cols - 1);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (32 * s >= K) break;
    const int at = min(2 * s + (kq >> 1), steps16 - 1);           // past the end: the last step again, which meets zeros
#pragma unroll
    for (int p = 0; p < 3; ++p) w.u[s][p] = P[(at * 6 + 2 * p + (kq & 1)) * cols + c];
  }
}

// Sums over K of weights x C for the tile's 16 columns and the 16 rows.  Every step's products start from zero, the smallest first, and
// the steps are added up in pairs: the matrix instructions cut low bits of what they add to a larger sum.  Error of act() on
// [48, 128, 128, 12] at 64 rows against 64 bits (relative norm of the means and of the values, geometric mean over 60 seeds): 1.02e-7
// and 1.05e-7; one sum that runs on over all steps 2.29e-7 and 2.35e-7, a running sum each for the small products and the large ones
// 1.07e-7 and 1.09e-7; the wider kernel (fused_forward.hip) 1.04e-7 and 1.06e-7.
template <int STEPS>
__device__ __forceinline__ f32x4 ss_product(const SsWeights<STEPS>& w, int K, const char* C, int cols, int m, int kq) {
  constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  const char* u = C + (kq * SS_ROWS + m) * 16;
  auto step = [&](int s) {
    bf16x8 b[3];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < 3; ++p) b[p] = ss_unit(u + p * SS_PLANE * cols + s * 4 * SS_ROWS * 16);
#pragma unroll
    for (int q = 0; q < 6; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w.u[s][PA[q]]), b[PB[q]], acc, 0, 0, 0);
    return acc;
  };
#pragma unroll
  for (int s = 0; s < STEPS; s += 2) {
    if (32 * s >= K) break;
    f32x4 acc = step(s);
    if (32 * (s + 1) < K) acc += step(s + 1);
    sum += acc;
  }
  return sum * split_unscale(m);
}

// Puts sums of fp32 products (v_mfma_f32_16x16x4_f32) in place of the non-finite ones (see gemm.hip): weights W[k * sk + c * sc] of
// the tile's columns c0 .. c0 + 15.
__device__ __forceinline__ void ss_repeat(const float* W, long sk, long sc, int K, int c0, int N, const char* C, int cols, int m, int kq, f32x4& acc) {
  constexpr int AHEAD = 4;           // products whose operands are requested together
  const float* w0 = W + min(c0 + m, N - 1) * sc;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int k0 = 0; k0 < K; k0 += 4 * AHEAD) {
    float w[AHEAD], x[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int k = k0 + 4 * i + kq, at = min(k, K - 1);
      w[i] = w0[at * sk];
      x[i] = ss_value(C + ((at >> 3) * SS_ROWS + m) * 16 + (at & 7) * 2, SS_PLANE * cols, m & 1);
      if (k >= K) w[i] = x[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], x[i], s, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (!__builtin_isfinite(acc[r])) acc[r] = s[r];
}

// Sums over the 16 lanes of a group, in all of them.
template <int N>
__device__ __forceinline__ float ss_turn(float v) {                       // lane i's value from lane i + N of its 16, cyclically
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x120 + 16 - N, 0xf, 0xf, true));
}
__device__ __forceinline__ float ss_sum16(float v) {
  v += ss_turn<8>(v); v += ss_turn<4>(v); v += ss_turn<2>(v); v += ss_turn<1>(v);
  return v;
}
template <int N>
__device__ __forceinline__ double ss_turn(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + 16 - N, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + 16 - N, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double ss_sum16(double v) {
  v += ss_turn<8>(v); v += ss_turn<4>(v); v += ss_turn<2>(v); v += ss_turn<1>(v);
  return v;
}

// STEPS: contraction steps of 32 of the widest layer.  L: layers; the loops over them are unrolled, so that what describes them is
// fetched once and a layer's outputs stay in registers for the backward pass.
template <int STEPS, int L>
__global__ __launch_bounds__(SS_THREADS, 2) void small_step_kernel(const SmallStepArgs args) {
  constexpr int TILES = STEPS * 32 / 16 / SS_WAVES;         // output tiles of a layer per wavefront
  extern __shared__ __align__(16) char lds[];
  const SmallNet& net = args.net[blockIdx.y];
  int dim[L + 1];
#pragma unroll
  for (int l = 0; l <= L; ++l) dim[l] = net.dims[l];
  const SsLds at(dim, L);
  char* C = lds + at.c;
  char* Rz = lds + at.r_dz;
  float* out = reinterpret_cast<float*>(lds + at.small);                  // [SS_MAX_OUT][16] outputs
  float* act = out + SS_MAX_OUT * SS_ROWS;                                // [SS_MAX_OUT][16] actions
  float* cst = act + SS_MAX_OUT * SS_ROWS;                                // [SS_MAX_OUT][2] log_std, 1 / sigma
  double* wsum = reinterpret_cast<double*>(cst + 2 * SS_MAX_OUT);         // [SS_WAVES]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kq = lane >> 4;
  const int split = blockIdx.x, turn = split & 1;
  const int row0 = split * SS_ROWS;
  const int A = dim[L];

  // Weights of the wavefront's first tile in product `ph` (forward through the layers, then the input gradients from the last one
  // down), requested AHEAD products before they are used: they come from beyond the L2 where the optimiser has just written them.
  constexpr int AHEAD = STEPS <= 4 ? 2 : 1;
  SsWeights<STEPS> w[AHEAD];
  auto request = [&](int ph) {
    const int l = ph < L ? ph : 2 * L - 1 - ph;
    if (l < 1 && ph > 0) return;
    if (ph < L) ss_load_weights<STEPS>(net.pack + net.fwd[l], dim[l], dim[l + 1], 16 * wave + m, kq, w[ph % AHEAD]);
    else ss_load_weights<STEPS>(net.pack + net.dx[l], dim[l + 1], dim[l], 16 * wave + m, kq, w[ph % AHEAD]);
  };

  // ---- rows of the minibatch; lane (row, j) also holds component j of the row's quantities for the loss ----
  const int lrow = tid & 15, lj = tid >> 4;
  const bool row_ok = row0 + lrow < args.rows;
  const long src = row_ok ? args.idx[row0 + lrow] : 0;
  request(0);
  float v_act = 0.f, v_mu = 0.f, v_sigma = 1.f, adv = 0.f, ret = 0.f, v_old = 0.f, logp_old = 0.f;   // a regression's target comes in v_act
  float ls = 0.f;
  {
    const int D = dim[0], Dr = ss_pad(D, 16), Dc = ss_pad(D, 32);
    const bool vec = (D & 3) == 0 && (net.ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(net.x) & 15) == 0;
    const float* x = net.x + src * net.ldx;
    constexpr int PASSES = STEPS * 8 * SS_ROWS / SS_THREADS;
    float v[PASSES][4];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int c = 4 * (lj + 32 * i);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[i][k] = 0.f;
      if (row_ok && c < D) {
        if (vec) {
          const float4 q = *reinterpret_cast<const float4*>(x + c);
          v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (c + k < D) v[i][k] = x[c + k];
        }
      }
    }
    // what the loss reads is requested behind the rows and waited for after them
    if (net.role != SMALL_CRITIC && row_ok && lj < A) {
      v_act = args.actions[src * A + lj];
      if (net.role == SMALL_ACTOR) {
        v_mu = args.mu_old[src * A + lj];
        v_sigma = args.sigma_old[src * A + lj];
      }
    }
    if (net.role == SMALL_ACTOR && lj < A) ls = args.log_std[lj];
    if (net.role == SMALL_ACTOR && row_ok) { adv = args.adv[src]; logp_old = args.logp_old[src]; }
    if (net.role == SMALL_CRITIC && row_ok) { ret = args.returns[src]; v_old = args.v_old[src]; }
    if (AHEAD > 1) request(1);
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int c = 4 * (lj + 32 * i);
      if (c >= Dc) continue;
      const Parts q = ss_split(v[i]);
      ss_put_c(C, at.c_cols, c, lrow, q);
      if (c < Dr) ss_put_r(lds, Dr, c, lrow, q, 1 - turn);
    }
  }
  const float inv = expf(-ls);
  if (net.role == SMALL_ACTOR) {
    act[lj * SS_ROWS + lrow] = v_act;
    if (lrow == 0) { cst[2 * lj] = ls; cst[2 * lj + 1] = inv; }
  }
  __syncthreads();

  // ---- forward ----
  float h[L][TILES][4];              // outputs of the hidden layers
  int r_at[L];                       // LDS offset of R of a layer's input
  r_at[0] = 0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int K = dim[l], N = dim[l + 1], tiles = (N + 15) / 16;
    const float* W = net.params + net.weights[l];
    const float* bias = W + (long)K * N;
    f32x4 acc[TILES];
    float bv[TILES][4];
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
      const int t = wave + SS_WAVES * i;
      acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r) bv[i][r] = 0.f;
      if (t < tiles) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[i][r] = bias[min(16 * t + 4 * kq + r, N - 1)];
        if (i > 0) ss_load_weights<STEPS>(net.pack + net.fwd[l], K, N, 16 * t + m, kq, w[l % AHEAD]);
        acc[i] = ss_product<STEPS>(w[l % AHEAD], K, C, at.c_cols, m, kq);
        if (ss_any_nonfinite(acc[i])) ss_repeat(W, N, 1, K, 16 * t, N, C, at.c_cols, m, kq, acc[i]);
      }
    }
    request(l + AHEAD);
    if (l + 1 < L) {
      r_at[l + 1 < L ? l + 1 : 0] = r_at[l] + ss_r_bytes(K);
      const int Nr = ss_pad(N, 16), Nc = ss_pad(N, 32);
      Parts q[TILES];
#pragma unroll
      for (int i = 0; i < TILES; ++i) {
        const int c = 16 * (wave + SS_WAVES * i) + 4 * kq;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[i][r] + bv[i][r], e = net.alpha * (__expf(v) - 1.0f);
          h[l][i][r] = c + r < N ? (v > 0.f ? v : e) : 0.f;
        }
        q[i] = ss_split(h[l][i]);
      }
      __syncthreads();               // C has been read
#pragma unroll
      for (int i = 0; i < TILES; ++i) {
        const int c = 16 * (wave + SS_WAVES * i) + 4 * kq;
        if (c < Nc) ss_put_c(C, at.c_cols, c, m, q[i]);
        if (c < Nr) ss_put_r(lds + r_at[l + 1 < L ? l + 1 : 0], Nr, c, m, q[i], 1 - turn);
      }
    } else if (wave < tiles) {
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(16 * wave + 4 * kq + r) * SS_ROWS + m] = acc[0][r] + bv[0][r];
    }
    __syncthreads();
  }

  // ---- loss; lane (row, component).  Every lane of a row forms the row's sums by itself: reading them over costs less than two
  //      more exchanges ----
  float d = 0.f;                     // gradient of the output
  if (net.role == SMALL_ACTOR) {
    float dl = 0.f, z = 0.f;
    double kl = 0.0, surr = 0.0, clipped = 0.0;
    if (row_ok) {
      float zz = 0.f, sum_ls = 0.f;
#pragma unroll 4
      for (int j = 0; j < A; ++j) {
        const float zj = (act[j * SS_ROWS + lrow] - out[j * SS_ROWS + lrow]) * cst[2 * j + 1];
        zz += zj * zj;
        sum_ls += cst[2 * j];
      }
      const float cl = sum_ls + 0.5f * (float)A * SS_LOG_2PI;
      float d_v;
      const RowTerms t = ppo_row(args.terms, -0.5f * zz - cl, logp_old, adv, 0.f, 0.f, 0.f, 1.0f / (float)args.rows, &dl, &d_v);
      surr = t.surr; clipped = t.clipped;
      if (lj < A) {
        const float mean = out[lj * SS_ROWS + lrow], inv2 = 0.5f * inv * inv;
        z = (v_act - mean) * inv;
        kl = (double)((ls - logf(v_sigma)) + (v_sigma * v_sigma + (v_mu - mean) * (v_mu - mean)) * inv2 - 0.5f);
        d = dl * z * inv;
      }
    }
    double* part = args.loss_partials + (long)split * (PPO_NPART_FIXED + A);
    const double g = ss_sum16(row_ok ? (double)(dl * (z * z - 1.0f)) : 0.0);
    if (lrow == 0 && lj < A) part[PPO_NPART_FIXED + lj] = g;
    kl = ss_sum16(kl);
    kl += __shfl_xor(kl, 16, 64);
    kl += __shfl_xor(kl, 32, 64);
    if (lane == 0) wsum[wave] = kl;  // added up behind the next barrier
    if (wave == 0) {
      surr = ss_sum16(surr); clipped = ss_sum16(clipped);
      if (tid == 0) { part[0] = surr; part[3] = clipped; part[4] = 0.0; }
    }
  } else if (net.role == SMALL_CRITIC) {
    if (tid < SS_ROWS) {
      double vloss = 0.0;
      if (row_ok) {
        float dl;
        const RowTerms t = ppo_row(args.terms, 0.f, 0.f, 0.f, out[lrow], v_old, ret, 1.0f / (float)args.rows, &dl, &d);
        vloss = t.vloss;
      }
      vloss = ss_sum16(vloss);
      if (tid == 0) args.loss_partials[(long)split * (PPO_NPART_FIXED + args.terms.A) + 1] = vloss;
    }
  } else {
    double q = 0.0;
    if (row_ok && lj < A) {
      const float e = out[lj * SS_ROWS + lrow] - v_act;
      d = 2.0f / (float)((long)args.rows * A) * e;
      q = (double)e * (double)e;
    }
    q = ss_sum16(q);
    q += __shfl_xor(q, 16, 64);
    q += __shfl_xor(q, 32, 64);
    if (lane == 0) wsum[wave] = q;
  }
  // the gradient of the outputs to C and R (32 columns, zeros behind the outputs), its column sums to the bias gradient
  {
    const float v[4] = {d, 0.f, 0.f, 0.f};
    const Parts q = ss_split(v);
    const int Ar = ss_pad(A, 16);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const uint32_t p = q.p[s][0] & 0xffffu;
      *reinterpret_cast<uint16_t*>(C + s * SS_PLANE * at.c_cols + ((lj >> 3) * SS_ROWS + lrow) * 16 + (lj & 7) * 2) = (uint16_t)(p ^ (lrow & 1 ? 0x8000u : 0u));
      if (lj < Ar) *reinterpret_cast<uint16_t*>(Rz + s * SS_PLANE * Ar + ((lrow >> 3) * Ar + lj) * 16 + (lrow & 7) * 2) = (uint16_t)p;
    }
    const float s = ss_sum16(d);
    if (lrow == 0 && lj < A) net.partials[net.part_off[L - 1] + split * net.pitch[L - 1] + (long)dim[L - 1] * A + lj] = s;
  }
  __syncthreads();
  if (tid == 0 && net.role != SMALL_CRITIC) {
    double s = wsum[0];
    for (int i = 1; i < SS_WAVES; ++i) s += wsum[i];
    args.loss_partials[net.role == SMALL_ACTOR ? (long)split * (PPO_NPART_FIXED + A) + 2 : split] = s;
  }

  // ---- backward ----
#pragma unroll
  for (int l = L - 1; l >= 0; --l) {
    const int K = dim[l], N = dim[l + 1], Kr = ss_pad(K, 16), Nr = ss_pad(N, 16);
    const int tk = Kr / 16, tn = Nr / 16;
    const char* R = lds + r_at[l];
    f32x4 acc[TILES];
    if (l > 0) {
      const float* W = net.params + net.weights[l];
#pragma unroll
      for (int i = 0; i < TILES; ++i) {
        const int t = wave + SS_WAVES * i;
        acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (t < tk) {
          if (i > 0) ss_load_weights<STEPS>(net.pack + net.dx[l], N, K, 16 * t + m, kq, w[(2 * L - 1 - l) % AHEAD]);
          acc[i] = ss_product<STEPS>(w[(2 * L - 1 - l) % AHEAD], N, C, at.c_cols, m, kq);
          if (ss_any_nonfinite(acc[i])) ss_repeat(W, 1, N, N, 16 * t, K, C, at.c_cols, m, kq, acc[i]);
        }
      }
      request(2 * L - 1 - l + AHEAD);
    }
    // weight gradient: a wavefront keeps the operand of the wider side and walks along the other.  Lane (m, kq) of a tile holds
    // outputs 4 kq .. + 3 of input m: one 16-byte store where the rows allow it
    {
      float* P = net.partials + net.part_off[l] + split * net.pitch[l];
      const bool by_n = tn >= tk, whole = (N & 3) == 0;
      const int own = by_n ? tn : tk, walk = by_n ? tk : tn;
      const int rg = kq & 1;
      const char* kept = by_n ? Rz + (rg * Nr + m) * 16 : R + (rg * Kr + m) * 16;
      const char* other = by_n ? R + (rg * Kr + m) * 16 : Rz + (rg * Nr + m) * 16;
      const int kept_step = SS_PLANE * (by_n ? Nr : Kr), other_step = SS_PLANE * (by_n ? Kr : Nr);
      const float unscale = split_unscale(m + turn);
#pragma unroll 1
      for (int o = wave; o < own; o += SS_WAVES) {
        bf16x8 u[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {                       // the half of a contraction that has no rows meets zeros in this operand
          const bf16x8 x = ss_unit(kept + p * kept_step + o * 256);
          u[p] = kq < 2 ? x : __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
        }
        auto tiles = [&](int t0, auto count) {
          constexpr int T = decltype(count)::value;
          bf16x8 v[T][3];
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) v[i][p] = ss_unit(other + p * other_step + min(t0 + i, walk - 1) * 256);
          constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
          f32x4 g[T];
#pragma unroll
          for (int i = 0; i < T; ++i) g[i] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (by_n) {
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
              for (int i = 0; i < T; ++i) g[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[PA[q]], v[i][PB[q]], g[i], 0, 0, 0);
          } else {
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
              for (int i = 0; i < T; ++i) g[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[i][PA[q]], u[PB[q]], g[i], 0, 0, 0);
          }
          float zero = 0.f;          // becomes NaN with any non-finite sum
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              g[i][r] *= unscale;
              zero = fmaf(g[i][r], 0.f, zero);
            }
          const bool repeat = __any(!(zero == 0.f));
#pragma unroll
          for (int i = 0; i < T; ++i) {
            if (t0 + i >= walk) break;
            const int k = 16 * (by_n ? t0 + i : o) + m, n = 16 * (by_n ? o : t0 + i) + 4 * kq;
            if (repeat) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                if (__builtin_isfinite(g[i][r])) continue;
                float s = 0.f;
#pragma unroll 1
                for (int y = 0; y < SS_ROWS; ++y)
                  s = fmaf(ss_value(R + ((y >> 3) * Kr + k) * 16 + (y & 7) * 2, SS_PLANE * Kr, ((m + turn) & 1) != 0),
                           ss_value(Rz + ((y >> 3) * Nr + n + r) * 16 + (y & 7) * 2, SS_PLANE * Nr, false), s);
                g[i][r] = s;
              }
            }
            if (k < K) {
              float* to = P + (long)k * N + n;
              if (whole) {
                if (n < N) *reinterpret_cast<float4*>(to) = make_float4(g[i][0], g[i][1], g[i][2], g[i][3]);
              } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                  if (n + r < N) to[r] = g[i][r];
              }
            }
          }
        };
        int t = 0;
        for (; t + 2 < walk; t += 4) tiles(t, std::integral_constant<int, 4>{});
        for (; t < walk; ++t) tiles(t, std::integral_constant<int, 1>{});
      }
    }
    if (l == 0) break;
    // the layer below: times ELU' of its outputs
    const int Kc = ss_pad(K, 32);
    float v[TILES][4];
    Parts q[TILES];
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
      const int c = 16 * (wave + SS_WAVES * i) + 4 * kq;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float y = h[l > 0 ? l - 1 : 0][i][r];
        v[i][r] = c + r < K ? acc[i][r] * (y > 0.f ? 1.0f : y + net.alpha) : 0.f;
      }
      q[i] = ss_split(v[i]);
    }
    __syncthreads();                 // C and the gradient's R have been read
    float* bias_grad = net.partials + net.part_off[l > 0 ? l - 1 : 0] + split * net.pitch[l > 0 ? l - 1 : 0] + (long)dim[l > 0 ? l - 1 : 0] * K;
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
      const int c = 16 * (wave + SS_WAVES * i) + 4 * kq;
      if (c < Kc) ss_put_c(C, at.c_cols, c, m, q[i]);
      if (c < Kr) {
        ss_put_r(Rz, Kr, c, m, q[i], 2);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float s = ss_sum16(v[i][r]);
          if (m == 0 && c + r < K) bias_grad[c + r] = s;
        }
      }
    }
    __syncthreads();
  }
}

template <int STEPS, int L>
hipError_t launch_steps(const SmallStepArgs& a, int lds, hipStream_t stream) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(small_step_kernel<STEPS, L>), hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_MAX_LDS);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((small_step_kernel<STEPS, L>), dim3(small_step_blocks(a.rows), a.n_nets), dim3(SS_THREADS), lds, stream, a);
  return hipGetLastError();
}

template <int STEPS>
hipError_t launch_layers(const SmallStepArgs& a, int lds, hipStream_t stream) {
  switch (a.net[0].n_layers) {
    case 2: return launch_steps<STEPS, 2>(a, lds, stream);
    case 3: return launch_steps<STEPS, 3>(a, lds, stream);
    default: return launch_steps<STEPS, 4>(a, lds, stream);
  }
}

}  // namespace

int small_step_blocks(int32_t rows) { return (rows + SS_ROWS - 1) / SS_ROWS; }

bool small_step_supported(const int32_t* dims, int32_t n_layers) {
  if (n_layers < 2 || n_layers > SMALL_MAX_LAYERS || dims[n_layers] > SS_MAX_OUT) return false;
  for (int l = 0; l < n_layers; ++l)
    if (dims[l] > SMALL_MAX_DIM) return false;
  return SsLds(dims, n_layers).total <= SMALL_MAX_LDS;
}

hipError_t launch_small_step(const SmallStepArgs& a, hipStream_t stream) {
  int widest = 0, lds = 0;
  double flops = 0.0;
  for (int i = 0; i < a.n_nets; ++i) {
    const SmallNet& n = a.net[i];
    lds = std::max(lds, SsLds(n.dims, n.n_layers).total);
    for (int l = 0; l <= n.n_layers; ++l) {
      if (l < n.n_layers) flops += (l > 0 ? 6.0 : 4.0) * a.rows * n.dims[l] * (double)n.dims[l + 1];
      widest = std::max(widest, n.dims[l]);
    }
  }
  TraceScope ts(stream, "small_step", flops, 0.0);
  return widest <= 128 ? launch_layers<4>(a, lds, stream) : launch_layers<8>(a, lds, stream);
}

}  // namespace rslx
