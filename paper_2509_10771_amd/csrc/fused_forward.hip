// Layer-fused MLP inference for gfx950: the latency-critical path of act() and of the RND reward, where the
// batch is a few thousand rows and per-layer launches would cost more than the arithmetic.
//
// One workgroup (8 wavefronts, two per SIMD) carries 32 batch rows of one network through every layer.  The products
// run on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16) with both operands split in three, six products each (see
// gemm.hip): 96 matrix-core cycles per 32 contraction indices of a 16 x 16 block, where fp32 instructions take 256.
// Activations stay in LDS, split, 16 bytes holding one part of eight consecutive contraction indices of a row; weights
// are not staged at all but streamed from L2 as fp32 and split in registers (each is used by one wavefront of a
// workgroup only), or streamed as a launch ahead has split them.  A layer is cut into tasks of 64 output columns; when a layer has fewer than 8 such groups the
// contraction range of a group is split over 2, 4 or 8 wavefronts, so all 8 stay busy down to the narrow output layer.
// Lane (m, kq) of a task owns columns col0 + 4 m .. + 3 at contraction indices 8 kq .. + 7 of a step of 32: eight
// 16-byte loads per step, of which the 16 lanes of a row read 256 contiguous bytes.  Partial sums meet in LDS; all 512
// lanes then add them up in a fixed order, apply bias and ELU and leave the split result in place of the layer's
// input.  The last layer is also written to global memory; for the actor the Gaussian head (noise, action,
// log-density) runs in the same launch, one lane per (row, action component).
#include "kernels.h"
#include "split_bf16.h"
#include "fused_pack.h"
#include <algorithm>
#include <type_traits>

namespace rslx {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FF_ROWS = 32;
constexpr int FF_THREADS = 512;
constexpr int FF_WAVES = FF_THREADS / 64;
constexpr int FF_GROUP = 64;                   // output columns per task
constexpr int FF_STEP = 32;                    // contraction indices per step
constexpr int FF_MAX_DIM = 512;
constexpr int FF_PART = FF_MAX_DIM * FF_ROWS * 2;   // LDS bytes of one part of an activation matrix
constexpr int FF_SUMS = FF_WAVES * FF_GROUP * FF_ROWS * 4;   // LDS bytes of all partial sums
constexpr int FF_LDS = 3 * FF_PART + FF_SUMS;  // 160 KB
constexpr float FF_LOG_2PI = 1.8378770664093453f;

__device__ __forceinline__ uint64_t ff_mix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// LDS position of output (column c, row) among fp32 sums: the two 16-row halves are interleaved, so that a lane writes
// its two rows with one 8-byte access and 16 lanes write 128 contiguous bytes.
__device__ __forceinline__ int ff_at(int c, int row) { return c * FF_ROWS + ((row & 15) << 1) + (row >> 4); }
// LDS byte offset of part 0 of activations 8 g .. 8 g + 7 of a row.
__device__ __forceinline__ int ff_unit(int g, int row) { return (g * FF_ROWS + row) * 16; }

// ELU with the hardware exponential: alpha (e^x - 1) for x <= 0.  The absolute error (about 1e-7) is what
// matters for a value that feeds the next layer's sums; the relative error near zero does not.
__device__ __forceinline__ float ff_elu(float x, float alpha) { return x > 0.f ? x : alpha * (__expf(x) - 1.0f); }

// Splits eight consecutive activations of a row and writes them to LDS.  Values without a split (2^111 and above,
// infinite) have NaN for their first part and the two halves of their bits for the others: their row's sums come out NaN,
// and ff_value finds the value for the repetition in fp32.
__device__ __forceinline__ void ff_put(char* acts, int g, int row, const float (&v)[8]) {
  uint32_t p[3][4];
  const float scale = split_scale(row);
  float most = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    split_pair(scale * v[2 * i], scale * v[2 * i + 1], p[0][i], p[1][i], p[2][i]);
    most = fmaxf(most, fmaxf(fabsf(v[2 * i]), fabsf(v[2 * i + 1])));
  }
  if (most >= 0x1p111f) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (!(fabsf(v[i]) >= 0x1p111f)) continue;
      const uint32_t bits = __float_as_uint(v[i]);
      const int sh = 16 * (i & 1);
      const uint32_t keep = 0xffff0000u >> sh;
      p[0][i / 2] = (p[0][i / 2] & keep) | (0x7fc0u << sh);
      p[1][i / 2] = (p[1][i / 2] & keep) | ((bits >> 16) << sh);
      p[2][i / 2] = (p[2][i / 2] & keep) | ((bits & 0xffffu) << sh);
    }
  }
#pragma unroll
  for (int s = 0; s < 3; ++s)
    *reinterpret_cast<uint4*>(acts + s * FF_PART + ff_unit(g, row)) = make_uint4(p[s][0], p[s][1], p[s][2], p[s][3]);
}

// Activation k of a row as ff_put was given it (NaN for NaN).
__device__ __forceinline__ float ff_value(const char* acts, int k, int row) {
  const char* u = acts + ff_unit(k >> 3, row) + 2 * (k & 7);
  uint32_t p[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) p[i] = *reinterpret_cast<const uint16_t*>(u + i * FF_PART);
  if ((p[0] & 0x7fffu) > 0x7f80u) return __uint_as_float((p[1] << 16) | p[2]);
  return (__uint_as_float(p[2] << 16) + __uint_as_float(p[1] << 16) + __uint_as_float(p[0] << 16)) * (SPLIT_UNSCALE * split_scale(row));
}

// Work of one wavefront in one layer: 64 columns from col0 and contraction steps [s_begin, s_end).  Activations
// between K and the next multiple of 32 are kept at zero in LDS, so no step needs a partial form.
struct FfTask {
  int col0, kpart, parts, s_begin, s_end;   // parts: how many wavefronts share a group's contraction
  bool active;
};

__host__ __device__ inline int ff_groups(int N) { return (N + FF_GROUP - 1) / FF_GROUP; }

// The split of a layer is planned on the host (it needs integer divisions): see FusedNet::split_*.
__device__ __forceinline__ FfTask ff_task(const FusedNet& net, int l, int wave) {
  const int K = net.dims[l], N = net.dims[l + 1];
  const int shift = net.split_shift[l], per = net.split_steps[l];
  FfTask t;
  const int group = wave >> shift;
  t.kpart = wave & ((1 << shift) - 1);
  t.col0 = group * FF_GROUP;
  t.parts = net.split_parts[l];
  const int steps = (K + FF_STEP - 1) / FF_STEP;
  t.s_begin = min(steps, t.kpart * per);
  t.s_end = min(steps, t.s_begin + per);
  t.active = group < ff_groups(N) && t.kpart < t.parts;
  return t;
}

// Weight stream of a task.  Register 4 i + cb of the chunk of step s is W[32 s + 8 kq + i][col0 + 4 m + cb].
// Rows and columns are clamped into the matrix: rows past K meet zero activations, columns past N only feed
// accumulator rows that are dropped later.
constexpr int FF_CHUNK = 32;
struct FfWeights {
  const float* W;
  int ldw, K, m, kq;
  bool vec;             // rows are 16-byte aligned and N % 4 == 0: one 16-byte load per contraction index
  int col[4];           // clamped columns col0 + 4 m + cb

  __device__ __forceinline__ void setup(const float* W_, int K_, int N, int col0, int m_, int kq_) {
    W = W_; ldw = N; K = K_; m = m_; kq = kq_;
    vec = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(W_) & 15) == 0;
    const int c = vec ? min(col0 + 4 * m, N - 4) : col0 + 4 * m;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) col[cb] = min(c + cb, N - 1);
  }
  template <bool VEC>
  __device__ __forceinline__ void load(int s, float (&dst)[FF_CHUNK]) const {
    // byte offsets of the lane from the uniform base: one product for the step (both factors fit 24 bits, FF_MAX_DIM),
    // rows past the end clamped by their offset
    const uint32_t ldb = 4u * (uint32_t)ldw, c0 = VEC ? 4u * (uint32_t)col[0] : 0u;
    const uint32_t first = __umul24((uint32_t)(FF_STEP * s + 8 * kq), ldb) + c0, end = (uint32_t)(K - 1) * ldb + c0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t row = min(first + (uint32_t)i * ldb, end);
      const char* base = reinterpret_cast<const char*>(W);
      if constexpr (VEC) {
        const float4 v = *reinterpret_cast<const float4*>(base + row);
        dst[4 * i + 0] = v.x; dst[4 * i + 1] = v.y; dst[4 * i + 2] = v.z; dst[4 * i + 3] = v.w;
      } else {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) dst[4 * i + cb] = *reinterpret_cast<const float*>(base + (row + 4u * (uint32_t)col[cb]));
      }
    }
  }
};

// acc[cb][h] += W[:, col0 + 4 m + cb]^T (A operand) x activations of row half h (B operand) over the task's
// contraction range.  `w0` arrives holding the task's first chunk, fetched by the caller ahead of time.  A step has two
// halves of 24 matrix instructions, two column blocks each; under each the other pair of column blocks is split, so the
// scaling and splitting (104 vector instructions per half) hide behind the matrix cores.  The chunk after next is requested as
// soon as a step's weights have been split.
template <bool VEC>
__device__ __forceinline__ void ff_contract(const FfWeights& wt, const FfTask& task, const char* acts,
                                            float (&w0)[FF_CHUNK], f32x4 (&acc)[4][2]) {
  float w1[FF_CHUNK];
  const char* bp = acts + ff_unit(wt.kq, wt.m);
  bf16x8 b[3][2];
  auto read_b = [&](int s) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        b[p][h] = *reinterpret_cast<const bf16x8*>(bp + p * FF_PART + s * (FF_STEP / 8 * FF_ROWS * 16) + h * 256);
  };
  struct Pair { uint4 part[2][3]; };       // two column blocks, three parts
  auto split = [&](const float (&w)[FF_CHUNK], int cb0, Pair& a) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int cb = cb0 + c;
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = SPLIT_SCALE * w[4 * i + cb];
      split_pair(v[0], v[1], a.part[c][0].x, a.part[c][1].x, a.part[c][2].x);
      split_pair(v[2], v[3], a.part[c][0].y, a.part[c][1].y, a.part[c][2].y);
      split_pair(v[4], v[5], a.part[c][0].z, a.part[c][1].z, a.part[c][2].z);
      split_pair(v[6], v[7], a.part[c][0].w, a.part[c][1].w, a.part[c][2].w);
    }
  };
  auto multiply = [&](const Pair& a, int cb0) {
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          acc[cb0 + c][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.part[c][PA[q]]), b[PB[q]][h],
                                                                    acc[cb0 + c][h], 0, 0, 0);
  };
  Pair lo, hi;
  const int last = task.s_end - 1;
  auto step = [&](int s, float (&w)[FF_CHUNK], float (&wn)[FF_CHUNK]) {
    read_b(s);
    split(w, 2, hi);
    multiply(lo, 0);
    wt.load<VEC>(s + 2, w);                // clamped: past the range it reads valid weights that nobody uses
    split(wn, 0, lo);
    multiply(hi, 2);
  };
  if (last == task.s_begin) {              // narrow layers: nothing is fetched and split for a step that does not come
    read_b(last);
    split(w0, 0, lo);
    split(w0, 2, hi);
    multiply(lo, 0);
    multiply(hi, 2);
  } else {
    wt.load<VEC>(task.s_begin + 1, w1);
    split(w0, 0, lo);
    for (int s = task.s_begin;; s += 2) {
      step(s, w0, w1);
      if (s + 1 > last) break;
      step(s + 1, w1, w0);
      if (s + 2 > last) break;
    }
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int h = 0; h < 2; ++h) acc[cb][h] *= split_unscale(wt.m);     // batch rows m and 16 + m
}

// The same from weights that come split (fused_pack.h), the same bits: no vector instruction beside the matrix instructions but
// addresses, and the step is bound by the weights' way from L2 (6 bytes a weight, 1.1 MB per workgroup of [48, 512, 256, 128, 12]):
// two such networks at 4096 rows 31 us instead of 36.  p is the lane's unit of the task's first step, w0 holds that step.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void ff_load_packed(const u32x4* p, u32x4 (&w)[12]) {
#pragma unroll
  for (int i = 0; i < 12; ++i) w[i] = p[64 * i];
}

__device__ __forceinline__ void ff_contract_packed(const u32x4* p, const FfTask& task, const char* acts, int m, int kq, u32x4 (&w0)[12], f32x4 (&acc)[4][2]) {
  u32x4 w1[12];
  const char* bp = acts + ff_unit(kq, m);
  const int last = task.s_end - 1;
  auto step = [&](int s, u32x4 (&w)[12]) {
    bf16x8 b[3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        b[q][h] = *reinterpret_cast<const bf16x8*>(bp + q * FF_PART + s * (FF_STEP / 8 * FF_ROWS * 16) + h * 256);
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          acc[cb][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[3 * cb + PA[q]]), b[PB[q]][h], acc[cb][h], 0, 0, 0);
    ff_load_packed(p + (long)min(s + 2 - task.s_begin, last - task.s_begin) * FP_STEP, w);
  };
  if (last > task.s_begin) ff_load_packed(p + FP_STEP, w1);
  for (int s = task.s_begin;; s += 2) {
    step(s, w0);
    if (s + 1 > last) break;
    step(s + 1, w1);
    if (s + 2 > last) break;
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int h = 0; h < 2; ++h) acc[cb][h] *= split_unscale(m);
}

// Puts the sums of fp32 products (v_mfma_f32_16x16x4_f32, from the fp32 weights and the activations' values) in place of
// the non-finite ones of a task (see gemm.hip): such inputs have no split.  The other rows keep their sums.
__device__ __forceinline__ void ff_repeat_fp32(const float* W, int K, int N, const FfTask& task, const char* acts, int m, int kq,
                                               f32x4 (&acc)[4][2]) {
  f32x4 c[4][2];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int h = 0; h < 2; ++h) c[cb][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int k_end = min(K, task.s_end * FF_STEP);
  constexpr int AHEAD = 4;             // contraction indices per lane whose operands are requested together
#pragma unroll 1
  for (int k0 = task.s_begin * FF_STEP; k0 < k_end; k0 += 4 * AHEAD) {
    float w[AHEAD][4];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int k = k0 + 4 * i + kq;
        w[i][cb] = k < K ? W[(long)k * N + min(task.col0 + 4 * m + cb, N - 1)] : 0.f;
      }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      float x[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) x[h] = ff_value(acts, k0 + 4 * i + kq, m + 16 * h);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int h = 0; h < 2; ++h) c[cb][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][cb], x[h], c[cb][h], 0, 0, 0);
    }
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (!__builtin_isfinite(acc[cb][h][r])) acc[cb][h][r] = c[cb][h][r];
}

// First weight chunk of a task.
__device__ __forceinline__ void ff_first_chunk(const float* __restrict__ W, int K, int N, const FfTask& task, int m,
                                               int kq, float (&w)[FF_CHUNK]) {
  if (!task.active) return;
  FfWeights wt;
  wt.setup(W, K, N, task.col0, m, kq);
  if (wt.vec) wt.load<true>(task.s_begin, w);
  else wt.load<false>(task.s_begin, w);
}

// The lane's unit of a task's first step; layer: the layer's first unit.
__device__ __forceinline__ const u32x4* ff_task_units(const u32x4* layer, int K, const FfTask& task, int lane) {
  return layer + (long)((task.col0 / FF_GROUP) * fused_pack_steps(K) + task.s_begin) * FP_STEP + lane;
}

namespace {
__device__ void small_forward_any(const FusedForwardArgs& args, const FusedNet& net, int block, char* lds);      // small_forward.h
}

// UNEVEN: two networks of which the second takes the kernel of small_forward.h, side by side in one launch: each in the form that its
// own sizes call for, with the bits that it has by itself.  The launch takes as long as the wider network, whose workgroups are
// dispatched first; two launches take the sum.  act(), both networks through the wider kernel, two launches and this, us at 1024 rows:
// [48, 128, 128] beside [48, 256, 128] 16.4, 24.6 and 16.2, [48, 512, 256, 128] beside [48, 128, 128] 34.6, 41.2 and 34.0; two narrow
// networks of different depths (small_uneven_kernel), [48, 64] beside [48, 64, 32], 11.7, 11.1 and 7.5.
template <bool PACK, bool UNEVEN>
__global__ __launch_bounds__(FF_THREADS) void fused_forward_kernel(const FusedForwardArgs args) {
  extern __shared__ __align__(16) char lds[];
  if constexpr (UNEVEN) {
    if (blockIdx.y == 1) {
      small_forward_any(args, args.net[1], blockIdx.x, lds);
      return;
    }
  }
  const FusedNet& net = args.net[UNEVEN ? 0 : blockIdx.y];
  const int row0 = blockIdx.x * FF_ROWS;
  if (row0 >= args.n_rows) return;
  const int tid = threadIdx.x, lane = tid & 63;
  // the wavefront index decides which columns and contraction range a wavefront works on: held in a scalar
  // register, every test on it is a scalar branch
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int m = lane & 15, kq = lane >> 4;
  char* acts = lds;                                          // [3 parts][K / 8][32 rows][8]
  float* sums = reinterpret_cast<float*>(lds + 3 * FF_PART);  // [part][column][32 rows], see ff_at

  // The first weight chunk of the first layer and the head's per-component inputs do not depend on any
  // activation: they are requested before the input rows, so their latency passes under the staging.
  float wpre[FF_CHUNK];
  u32x4 upre[12];
  const u32x4* layer = reinterpret_cast<const u32x4*>(net.pack);
  FfTask task = ff_task(net, 0, wave);
  if constexpr (PACK) {
    if (task.active) ff_load_packed(ff_task_units(layer, net.dims[0], task, lane), upre);
  } else {
    ff_first_chunk(net.params, net.dims[0], net.dims[1], task, m, kq, wpre);
  }
  const int A = net.dims[net.n_layers];
  float head_ls = 0.f, head_eps = 0.f;
  if (net.head && tid < FF_ROWS * A) {
    long woff_ls = 0;
    for (int l = 0; l < net.n_layers; ++l) woff_ls += (long)net.dims[l] * net.dims[l + 1] + net.dims[l + 1];
    head_ls = net.params[woff_ls + (tid >> 5)];
    const long n = row0 + (tid & 31);
    if (!args.deterministic && args.eps != nullptr && n < args.n_rows) head_eps = args.eps[n * A + (tid >> 5)];
  }

  // Lane (row, g) finishes units of eight values: row tid % 32, units g = tid / 32 + 16 i.
  int urow = tid & 31, ug = tid >> 5;
  // ---- input rows -> LDS; values from K0 to the next multiple of 32 are zero ----
  {
    const int K0 = net.dims[0];
    const int units = (K0 + FF_STEP - 1) / FF_STEP * (FF_STEP / 8);
    const bool vec = net.col_map == nullptr && (net.ldx & 3) == 0 && (K0 & 3) == 0 && (reinterpret_cast<uintptr_t>(net.x) & 15) == 0;
    const int row = row0 + urow;
    const float* xr = net.x + (long)min(row, args.n_rows - 1) * net.ldx;
#pragma unroll
    for (int i = 0; i < FF_MAX_DIM / 8 / 16; ++i) {
      const int g = ug + 16 * i;
      if (16 * i >= units) break;
      if (g >= units) continue;
      float v[8];
      if (vec) {
#pragma unroll
        for (int c = 0; c < 8; c += 4) {
          float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
          if (8 * g + c < K0) q = *reinterpret_cast<const float4*>(xr + 8 * g + c);
          v[c] = q.x; v[c + 1] = q.y; v[c + 2] = q.z; v[c + 3] = q.w;
        }
      } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int k = 8 * g + c;
          v[c] = k < K0 ? xr[net.col_map ? net.col_map[k] : k] : 0.f;
        }
      }
      if (row >= args.n_rows) {
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = 0.f;
      }
      ff_put(acts, g, urow, v);
    }
  }
  __syncthreads();

  const float* mu = sums;        // the last layer's outputs, see ff_at
  long woff = 0;
  int K = net.dims[0], N = net.dims[1];
  for (int l = 0; l < net.n_layers; ++l) {
    // opaque from here on, or every address formed from them below would be computed once, kept for all layers and spilled
    asm volatile("" : "+v"(m), "+v"(kq), "+v"(urow), "+v"(ug));
    const float* W = net.params + woff;
    const float* bias = W + (long)K * N;
    const bool last = (l + 1 == net.n_layers);
    float* gout = last ? net.out : nullptr;
    const int plane = ff_groups(N) * FF_GROUP * FF_ROWS;     // floats between the partial sums of two parts
    const int units = (N + FF_STEP - 1) / FF_STEP * (FF_STEP / 8);

    const bool shared = task.parts > 1;
    const FfTask next = last ? task : ff_task(net, l + 1, wave);
    const int N2 = last ? 0 : net.dims[l + 2];       // read ahead like `next`: nothing waits for it between the layers
    f32x4 acc[4][2];
    if (task.active) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[cb][h] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (PACK) {
        ff_contract_packed(ff_task_units(layer, K, task, lane), task, acts, m, kq, upre, acc);
      } else {
        FfWeights wt;
        wt.setup(W, K, N, task.col0, m, kq);
        if (wt.vec) ff_contract<true>(wt, task, acts, wpre, acc);
        else ff_contract<false>(wt, task, acts, wpre, acc);
      }
      float z = 0.f;                 // becomes NaN with any non-finite sum
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r) z = fmaf(acc[cb][h][r], 0.f, z);
      if (__any(!(z == 0.f))) ff_repeat_fp32(W, K, N, task, acts, m, kq, acc);
    }
    // bias values of the outputs this lane finishes, requested before the sums are exchanged: with the contraction of
    // a group shared among wavefronts, the sums are finished by all lanes after an exchange through LDS; otherwise
    // each wavefront finishes its own accumulators in registers
    constexpr int FIN = 2;         // units per lane at most: shared layers have at most four groups of 64 columns
    float bfin[8 * FIN];
    if (shared) {
#pragma unroll
      for (int i = 0; i < FIN; ++i) {
        if (16 * i >= units) break;
#pragma unroll
        for (int c = 0; c < 8; ++c) bfin[8 * i + c] = bias[min(8 * (ug + 16 * i) + c, N - 1)];
      }
    } else if (task.active) {
#pragma unroll
      for (int c = 0; c < 16; ++c) bfin[c] = bias[min(task.col0 + 16 * kq + c, N - 1)];
    }
    // the next layer's first chunk is requested before this layer's sums are exchanged as well
    if constexpr (PACK) {
      layer += fused_pack_units(K, N);
      if (!last && next.active) ff_load_packed(ff_task_units(layer, N, next, lane), upre);
    } else {
      if (!last) ff_first_chunk(bias + N, N, N2, next, m, kq, wpre);
    }
    // accumulator register r of block cb: column col0 + 16 kq + 4 r + cb, batch rows m (half 0) and 16 + m
    if (shared && task.active) {
      float* part = sums + task.kpart * plane;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<float2*>(part + ff_at(task.col0 + 16 * kq + 4 * r + cb, m)) = make_float2(acc[cb][0][r], acc[cb][1][r]);
    }
    __syncthreads();                 // every wavefront has read its activations; the partial sums are there

    if (!shared) {
      if (task.active) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          float v[16];
#pragma unroll
          for (int c = 0; c < 16; ++c) {
            v[c] = acc[c & 3][h][c >> 2] + bfin[c];
            if (!last) v[c] = ff_elu(v[c], net.alpha);
          }
          const int c0 = task.col0 + 16 * kq;
          if (last) {
            const int row = row0 + m + 16 * h;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
              sums[ff_at(c0 + c, m + 16 * h)] = v[c];
              if (c0 + c < N && row < args.n_rows) gout[(long)row * N + c0 + c] = v[c];
            }
          } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              float x[8];
#pragma unroll
              for (int c = 0; c < 8; ++c) x[c] = c0 + 8 * u + c < N ? v[8 * u + c] : 0.f;
              ff_put(acts, (c0 >> 3) + u, m + 16 * h, x);
            }
          }
        }
      }
    } else {
      // all lanes: sum the parts in order, bias, activation
      float* muw = reinterpret_cast<float*>(acts);
      float fv[FIN][8];
#pragma unroll
      for (int i = 0; i < FIN; ++i) {
        if (16 * i >= units) break;
        const float* p0 = sums + ff_at(8 * min(ug + 16 * i, units - 1), urow);
#pragma unroll
        for (int c = 0; c < 8; ++c) fv[i][c] = p0[c * FF_ROWS];
        for (int p = 1; p < task.parts; ++p)
#pragma unroll
          for (int c = 0; c < 8; ++c) fv[i][c] += p0[p * plane + c * FF_ROWS];
      }
#pragma unroll
      for (int i = 0; i < FIN; ++i) {
        const int g = ug + 16 * i;
        if (16 * i >= units) break;
        if (g >= units) continue;
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          v[c] = fv[i][c] + bfin[8 * i + c];
          if (!last) v[c] = ff_elu(v[c], net.alpha);
          if (8 * g + c >= N) v[c] = 0.f;
        }
        if (last) {
          const int row = row0 + urow;
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            muw[ff_at(8 * g + c, urow)] = v[c];
            if (8 * g + c < N && row < args.n_rows) gout[(long)row * N + 8 * g + c] = v[c];
          }
        } else {
          ff_put(acts, g, urow, v);
        }
      }
      if (last) mu = muw;
    }
    __syncthreads();
    task = next;
    woff += (long)K * N + N;
    K = N; N = N2;
  }

  // ---- Gaussian head (actor only): `mu` holds the means; one lane per (row, action component) ----
  if (net.head) {
    const float* log_std = net.params + woff;
    float* z2 = mu == sums ? reinterpret_cast<float*>(acts) : sums;   // [A][32], in the buffer that is free by now
    float* lsb = z2 + FF_ROWS * A;         // [A] log_std, for the per-row sums
    for (int e = tid; e < FF_ROWS * A; e += FF_THREADS) {
      const int r = e & 31, jj = e >> 5;
      const long n = row0 + r;
      const float ls = e == tid ? head_ls : log_std[jj];
      if (r == 0) lsb[jj] = ls;
      float zz = 0.f;
      if (n < args.n_rows) {
        const long o = n * A + jj;
        const float sg = expf(ls);
        const float mean = mu[ff_at(jj, r)];
        float eps;
        if (args.deterministic) {
          eps = 0.f;
        } else if (args.eps != nullptr) {
          eps = e == tid ? head_eps : args.eps[o];
        } else {
          const uint64_t nb = args.step_dev != nullptr ? ff_mix64(args.noise_pre ^ (uint64_t)*args.step_dev) : args.noise_base;
          const uint64_t h = ff_mix64(nb ^ (uint64_t)o);
          const float u1 = (float)((uint32_t)(h >> 40) + 1u) * 5.9604644775390625e-08f;
          const float u2 = (float)((uint32_t)(h >> 8) & 0xFFFFFFu) * 5.9604644775390625e-08f;
          eps = sqrtf(-2.0f * logf(u1)) * cospif(2.0f * u2);
        }
        const float act = mean + sg * eps;
        const float z = (act - mean) / sg;
        zz = z * z;
        args.actions[o] = act;
        args.sigma[o] = sg;
      }
      z2[jj * FF_ROWS + r] = zz;
    }
    __syncthreads();
    if (tid < FF_ROWS && row0 + tid < args.n_rows) {
      float zz = 0.f, sum_ls = 0.f;
      for (int jj = 0; jj < A; ++jj) {
        zz += z2[jj * FF_ROWS + tid];
        sum_ls += lsb[jj];
      }
      args.logp[row0 + tid] = -0.5f * zz - sum_ls - 0.5f * (float)A * FF_LOG_2PI;
    }
  }
}

bool fused_forward_supported(const FusedForwardArgs& a) {
  if (a.max_dim > FF_MAX_DIM || a.n_nets < 1 || a.n_nets > 2) return false;
  return true;
}

static double forward_flops(const FusedForwardArgs& a) {
  double flops = 0.0;
  for (int i = 0; i < a.n_nets; ++i)
    for (int l = 0; l < a.net[i].n_layers; ++l) flops += 2.0 * a.n_rows * a.net[i].dims[l] * (double)a.net[i].dims[l + 1];
  return flops;
}

size_t fused_pack_bytes(const int32_t* dims, int32_t n_layers) {
  size_t units = 0;
  if (n_layers < 1 || n_layers > 8) return 0;                // workspace queries come before any check
  for (int l = 0; l < n_layers; ++l) {
    if (std::min(dims[l], dims[l + 1]) < 1 || std::max(dims[l], dims[l + 1]) > FF_MAX_DIM) return 0;      // no layer-fused inference
    units += fused_pack_units(dims[l], dims[l + 1]);
  }
  return units * 16;
}

// The work split of every layer among the wavefronts of wide_forward (FusedNet::split_*).
static void plan_wide(FusedNet& n) {
  for (int l = 0; l < n.n_layers; ++l) {
    const int steps = (n.dims[l] + FF_STEP - 1) / FF_STEP;
    const int groups = ff_groups(n.dims[l + 1]);
    const int shift = groups <= 1 ? 3 : groups <= 2 ? 2 : groups <= 4 ? 1 : 0;
    const int per = (steps + (1 << shift) - 1) >> shift;
    n.split_shift[l] = shift;
    n.split_steps[l] = per;
    n.split_parts[l] = std::max(1, (steps + per - 1) / per);
  }
}

static const char* wide_site(bool packed) { return packed ? "fused_forward_packed" : "fused_forward"; }

static hipError_t launch_wide_forward(const FusedForwardArgs& a, hipStream_t stream) {
  static bool attr_set = false;
  if (!attr_set) {
    for (const void* k : {reinterpret_cast<const void*>(fused_forward_kernel<true, false>), reinterpret_cast<const void*>(fused_forward_kernel<false, false>)}) {
      hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, FF_LDS);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
  const bool packed = a.net[0].pack != nullptr && (a.n_nets < 2 || a.net[1].pack != nullptr);
  TraceScope ts(stream, wide_site(packed), forward_flops(a), 0.0);
  FusedForwardArgs b = a;
  for (int i = 0; i < b.n_nets; ++i) plan_wide(b.net[i]);
  dim3 grid((b.n_rows + FF_ROWS - 1) / FF_ROWS, b.n_nets);
  if (packed)
    hipLaunchKernelGGL((fused_forward_kernel<true, false>), grid, dim3(FF_THREADS), FF_LDS, stream, b);
  else
    hipLaunchKernelGGL((fused_forward_kernel<false, false>), grid, dim3(FF_THREADS), FF_LDS, stream, b);
  return hipGetLastError();
}

}  // namespace rslx

#include "small_step.h"      // the layer-fused optimiser step, compiled with the layer-fused inference
#include "small_forward.h"

namespace rslx {

void plan_fused_pack(FusedForwardArgs& a, void* ws, FusedPackBatch& b) {
  b.count = 0;
  uint4* at = static_cast<uint4*>(ws);
  for (int i = 0; i < a.n_nets; ++i) {
    FusedNet& n = a.net[i];
    if (!small_forward_takes(n, a.n_rows)) {
      n.pack = reinterpret_cast<const uint16_t*>(at);
      const float* w = n.params;
      uint4* dst = at;
      for (int l = 0; l < n.n_layers; ++l) {
        const int K = n.dims[l], N = n.dims[l + 1];
        b.job[b.count++] = FusedPackJob{w, reinterpret_cast<uint16_t*>(dst), K, N};
        w += (long)K * N + N;
        dst += fused_pack_units(K, N);
      }
    }
    at += fused_pack_bytes(n.dims, n.n_layers) / 16;
  }
}

template <bool PACK>
static hipError_t launch_uneven_forward(const FusedForwardArgs& a, hipStream_t stream) {
  static_assert(FF_THREADS == SS_THREADS && SS_ROWS <= FF_ROWS && SF_MAX_LDS <= FF_LDS, "one launch");
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_forward_kernel<PACK, true>), hipFuncAttributeMaxDynamicSharedMemorySize, FF_LDS);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((fused_forward_kernel<PACK, true>), dim3((a.n_rows + SS_ROWS - 1) / SS_ROWS, 2), dim3(FF_THREADS), FF_LDS, stream, a);
  return hipGetLastError();
}

hipError_t launch_fused_forward(const FusedForwardArgs& a, hipStream_t stream) {
  if (a.n_rows <= 0) return hipSuccess;
  const bool small = small_forward_takes(a.net[0], a.n_rows);
  if (a.n_nets == 2 && (small != small_forward_takes(a.net[1], a.n_rows) || (small && a.net[0].n_layers != a.net[1].n_layers))) {
    FusedForwardArgs b = a;
    bool is_small[2];
    double flops[2];
    for (int i = 0; i < 2; ++i) {
      is_small[i] = small_forward_takes(a.net[i], a.n_rows);
      FusedForwardArgs one = a;
      one.net[0] = a.net[i];
      one.n_nets = 1;
      flops[i] = forward_flops(one);
    }
    // a record for each network, both over the launch
    TraceScope t0(stream, is_small[0] ? "small_forward" : wide_site(a.net[0].pack != nullptr), flops[0], 0.0);
    TraceScope t1(stream, is_small[1] ? "small_forward" : wide_site(a.net[1].pack != nullptr), flops[1], 0.0);
    if (is_small[0] && is_small[1]) return launch_small_uneven(a, stream);
    if (is_small[0]) std::swap(b.net[0], b.net[1]);
    plan_wide(b.net[0]);
    return b.net[0].pack != nullptr ? launch_uneven_forward<true>(b, stream) : launch_uneven_forward<false>(b, stream);
  }
  if (!small) return launch_wide_forward(a, stream);
  TraceScope ts(stream, "small_forward", forward_flops(a), 0.0);
  return launch_small_forward(a, stream);
}

}  // namespace rslx
