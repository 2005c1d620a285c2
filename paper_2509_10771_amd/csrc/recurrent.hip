// Recurrent memory cells (GRU, LSTM): the hidden-side contraction on the matrix cores with the gate stage (forward) or the
// gate derivatives (back-propagation through time) as its epilogue, one time step per launch or a whole roll-out, and
// the index plumbing of column-wise minibatches.  The input-side contractions and the weight gradients run in the GEMM kernel.
#include "kernels.h"
#include "split_bf16.h"
#include "fused_pack.h"

#include <algorithm>

namespace rslx {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigmoidf_(float a) { return 1.0f / (1.0f + __expf(-a)); }
// tanh through the exponential of -2|a| (never overflows): (1 - e) / (1 + e) with the sign of a
__device__ __forceinline__ float tanhf_(float a) {
  const float e = __expf(-2.0f * fabsf(a));
  const float t = (1.0f - e) / (1.0f + e);
  return a < 0.f ? -t : t;
}

__device__ __forceinline__ f4 ld4(const float* p) { return *reinterpret_cast<const f4*>(p); }
__device__ __forceinline__ void st4(float* p, f4 v) { *reinterpret_cast<f4*>(p) = v; }

// ---- fused step kernels ----------------------------------------------------------------------------------
// A workgroup of 2 x 2 wavefronts owns 32 rows and 32 hidden units: wavefront (wr, wj) takes rows 16 wr .. 16 wr + 15
// and hidden units 16 wj .. 16 wj + 15 and accumulates NTW tiles of 16 output columns with
// v_mfma_f32_16x16x4_f32, D[row, col] += sum_k A[row, k] B[k, col(tile)]; the tiles' columns come from `col0[]`
// (forward: the r, z and n columns of its 16 hidden units; backward: the 16 hidden units themselves).  Accumulator
// register q of lane l belongs to row 4 * (l / 16) + q and column l % 16 in every tile, so the gate stage finds all
// its operands in the lane's own registers.  Operands are staged through LDS in chunks of KC contraction steps; the
// next chunk's global loads are in flight while the current one is multiplied.  One step moves little data per
// workgroup and every chunk costs a full memory latency, so the chunks are long rather than many, and two
// wavefronts share each SIMD so that one's LDS reads overlap the other's matrix instructions.
constexpr int GS_JB = 32;          // hidden units per workgroup
constexpr int GS_ROWS = 32;        // rows per workgroup
constexpr int GS_THREADS = 256;

template <int NTW, int KC>
struct StepTile {
  static constexpr int NT = 2 * NTW;            // tiles per workgroup: wavefront column wj owns tiles wj * NTW ...
  static constexpr int APITCH = KC + 4;         // floats per staged A row (16-byte aligned, spreads the banks)
  static constexpr int COLS = 16 * NT, BPITCH = COLS + 8;
  static constexpr int A_VECS = GS_ROWS * KC / 4, B_VECS = KC * COLS / 4;
  static constexpr int A_PER = (A_VECS + GS_THREADS - 1) / GS_THREADS, B_PER = (B_VECS + GS_THREADS - 1) / GS_THREADS;
  static constexpr int LDS_FLOATS = GS_ROWS * APITCH + KC * BPITCH;

  // acc[u] += A[row0 + 16 wr .., 0 .. K) * B[0 .. K, col0[wj * NTW + u] .. + 16).  Rows >= n_rows read as zero and so
  // do the columns of tile t from col_end[t] on.  K, lda, ldb, col0[], col_end[] are multiples of 4 and A, B are
  // 16-byte aligned, so every 16-byte fetch is entirely inside or entirely outside.
  static __device__ __forceinline__ void mma(const float* __restrict__ A, int lda, int row0, int n_rows,
                                             const float* __restrict__ B, int ldb, const int (&col0)[NT],
                                             const int (&col_end)[NT], int K, float* smem, f4 (&acc)[NTW]) {
    float* As = smem;
    float* Bs = smem + GS_ROWS * APITCH;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 1, wj = wave >> 1;
    const int m = lane & 15, kq = lane >> 4;
    // what this lane fetches of every chunk: fixed (row, k offset) pairs of A and (k, column) pairs of B
    int a_off[A_PER], a_kc[A_PER], b_col[B_PER], b_k[B_PER];
    bool a_ok[A_PER], b_ok[B_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int v = tid + i * GS_THREADS;
      const int r = v / (KC / 4);
      a_kc[i] = (v % (KC / 4)) * 4;
      a_ok[i] = v < A_VECS && row0 + r < n_rows;
      a_off[i] = min(row0 + r, n_rows - 1) * lda;
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int v = tid + i * GS_THREADS;
      const int c4 = v % (COLS / 4), t = c4 / 4;
      b_k[i] = v / (COLS / 4);
      int c0 = col0[0], ce = col_end[0];
#pragma unroll
      for (int u = 1; u < NT; ++u) { c0 = t == u ? col0[u] : c0; ce = t == u ? col_end[u] : ce; }
      const int col = c0 + (c4 % 4) * 4;
      b_ok[i] = v < B_VECS && col < ce;
      b_col[i] = b_ok[i] ? col : 0;
    }
    // Loads are issued unconditionally from clamped (always valid) addresses and the out-of-range parts are zeroed
    // only when the chunk is written to LDS, so nothing waits on a load before the chunk is needed.
    f4 ra[A_PER], rb[B_PER];
    auto fetch = [&](int k0) {
#pragma unroll
      for (int i = 0; i < A_PER; ++i) ra[i] = ld4(A + (long)a_off[i] + min(k0 + a_kc[i], K - 4));
#pragma unroll
      for (int i = 0; i < B_PER; ++i) rb[i] = ld4(B + (long)min(k0 + b_k[i], K - 1) * ldb + b_col[i]);
    };
    auto stage = [&](int k0) {
#pragma unroll
      for (int i = 0; i < A_PER; ++i) {
        const int v = tid + i * GS_THREADS;
        const f4 x = (a_ok[i] && k0 + a_kc[i] < K) ? ra[i] : f4{0.f, 0.f, 0.f, 0.f};
        if (A_VECS % GS_THREADS == 0 || v < A_VECS) st4(As + (v / (KC / 4)) * APITCH + a_kc[i], x);
      }
#pragma unroll
      for (int i = 0; i < B_PER; ++i) {
        const int v = tid + i * GS_THREADS;
        const f4 x = (b_ok[i] && k0 + b_k[i] < K) ? rb[i] : f4{0.f, 0.f, 0.f, 0.f};
        if (B_VECS % GS_THREADS == 0 || v < B_VECS) st4(Bs + b_k[i] * BPITCH + (v % (COLS / 4)) * 4, x);
      }
    };
    fetch(0);
    const float* ap = As + (wr * 16 + m) * APITCH + kq;
    const float* bp = Bs + kq * BPITCH + wj * NTW * 16 + m;
    for (int k0 = 0; k0 < K; k0 += KC) {
      __syncthreads();               // the previous chunk has been consumed
      stage(k0);
      __syncthreads();
      fetch(k0 + KC);                // past the end this re-reads the last rows (clamped); never staged
      __builtin_amdgcn_sched_barrier(0);
      // operands of contraction step s + 1 are read from LDS while the matrix instructions of step s run
      float a_cur = ap[0], b_cur[NTW];
#pragma unroll
      for (int u = 0; u < NTW; ++u) b_cur[u] = bp[16 * u];
#pragma unroll
      for (int s4 = 0; s4 < KC / 4; ++s4) {
        float a_nxt = 0.f, b_nxt[NTW];
        if (s4 + 1 < KC / 4) {
          a_nxt = ap[4 * (s4 + 1)];
#pragma unroll
          for (int u = 0; u < NTW; ++u) b_nxt[u] = bp[4 * (s4 + 1) * BPITCH + 16 * u];
        }
#pragma unroll
        for (int u = 0; u < NTW; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_cur, b_cur[u], acc[u], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1 + NTW, 0);    // next step's LDS reads ...
        __builtin_amdgcn_sched_group_barrier(0x008, NTW, 0);        // ... then this step's matrix instructions
        if (s4 + 1 < KC / 4) {
          a_cur = a_nxt;
#pragma unroll
          for (int u = 0; u < NTW; ++u) b_cur[u] = b_nxt[u];
        }
      }
    }
  }
};

// The same accumulation for an operand pair that is contiguous along the contraction on BOTH sides: A[row, k] and
// Bt[col, k] (D[row, col] += sum_k A[row, k] Bt[col, k]).  Both are staged row-major with the contraction index
// innermost, so one 16-byte LDS read per operand feeds four matrix instructions: lane (m, kq) of group g reads
// k = 16 g + 4 kq .. + 3 and uses component i in instruction i, which then contracts over {16 g + 4 kq' + i} - the
// order of the sum inside a group of 16 is permuted, nothing else.  The backward step uses it (A = dgh of the next
// step, Bt = the rows of W_hh itself), where one instruction per contraction step would leave the LDS latency bare.
template <int NTW, int KC>
struct StepTileKK {
  static constexpr int NT = 2 * NTW;
  static constexpr int PITCH = KC + 4;
  static constexpr int BROWS = 16 * NT;
  static constexpr int A_VECS = GS_ROWS * KC / 4, B_VECS = BROWS * KC / 4;
  static constexpr int A_PER = (A_VECS + GS_THREADS - 1) / GS_THREADS, B_PER = (B_VECS + GS_THREADS - 1) / GS_THREADS;
  static constexpr int LDS_FLOATS = (GS_ROWS + BROWS) * PITCH;
  static_assert(KC % 16 == 0 && A_VECS % GS_THREADS == 0 && B_VECS % GS_THREADS == 0, "chunk shape");

  // acc[u] += A[row0 + 16 wr .., 0 .. K) * Bt[col0[wj * NTW + u] .. + 16, 0 .. K)^T.  Rows >= n_rows and Bt rows from
  // col_end[t] on read as zero; K, lda, ldbt multiples of 4, A and Bt 16-byte aligned.
  static __device__ __forceinline__ void mma(const float* __restrict__ A, int lda, int row0, int n_rows,
                                             const float* __restrict__ Bt, int ldbt, const int (&col0)[NT],
                                             const int (&col_end)[NT], int K, float* smem, f4 (&acc)[NTW]) {
    float* As = smem;
    float* Bs = smem + GS_ROWS * PITCH;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 1, wj = wave >> 1;
    const int m = lane & 15, kq = lane >> 4;
    int a_off[A_PER], a_kc[A_PER], b_off[B_PER], b_kc[B_PER];
    bool a_ok[A_PER], b_ok[B_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int v = tid + i * GS_THREADS;
      const int r = v / (KC / 4);
      a_kc[i] = (v % (KC / 4)) * 4;
      a_ok[i] = row0 + r < n_rows;
      a_off[i] = min(row0 + r, n_rows - 1) * lda;
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int v = tid + i * GS_THREADS;
      const int c = v / (KC / 4), t = c / 16;
      b_kc[i] = (v % (KC / 4)) * 4;
      int c0 = col0[0], ce = col_end[0];
#pragma unroll
      for (int u = 1; u < NT; ++u) { c0 = t == u ? col0[u] : c0; ce = t == u ? col_end[u] : ce; }
      const int col = c0 + (c % 16);
      b_ok[i] = col < ce;
      b_off[i] = min(col, ce - 1) * ldbt;           // clamped: always a valid row
    }
    f4 ra[A_PER], rb[B_PER];
    auto fetch = [&](int k0) {      // unconditional loads from clamped addresses; zeroing happens at staging time
#pragma unroll
      for (int i = 0; i < A_PER; ++i) ra[i] = ld4(A + (long)a_off[i] + min(k0 + a_kc[i], K - 4));
#pragma unroll
      for (int i = 0; i < B_PER; ++i) rb[i] = ld4(Bt + (long)b_off[i] + min(k0 + b_kc[i], K - 4));
    };
    auto stage = [&](int k0) {
#pragma unroll
      for (int i = 0; i < A_PER; ++i) {
        const int v = tid + i * GS_THREADS;
        st4(As + (v / (KC / 4)) * PITCH + a_kc[i], (a_ok[i] && k0 + a_kc[i] < K) ? ra[i] : f4{0.f, 0.f, 0.f, 0.f});
      }
#pragma unroll
      for (int i = 0; i < B_PER; ++i) {
        const int v = tid + i * GS_THREADS;
        st4(Bs + (v / (KC / 4)) * PITCH + b_kc[i], (b_ok[i] && k0 + b_kc[i] < K) ? rb[i] : f4{0.f, 0.f, 0.f, 0.f});
      }
    };
    const float* ap = As + (wr * 16 + m) * PITCH + 4 * kq;
    const float* bp = Bs + (wj * NTW * 16 + m) * PITCH + 4 * kq;
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += KC) {
      __syncthreads();               // the previous chunk has been consumed
      stage(k0);
      __syncthreads();
      fetch(k0 + KC);                // past the end this re-reads clamped addresses; never staged
      __builtin_amdgcn_sched_barrier(0);
      f4 a_cur = ld4(ap), b_cur[NTW];
#pragma unroll
      for (int u = 0; u < NTW; ++u) b_cur[u] = ld4(bp + u * 16 * PITCH);
#pragma unroll
      for (int g = 0; g < KC / 16; ++g) {
        f4 a_nxt = a_cur, b_nxt[NTW];
#pragma unroll
        for (int u = 0; u < NTW; ++u) b_nxt[u] = b_cur[u];
        if (g + 1 < KC / 16) {
          a_nxt = ld4(ap + 16 * (g + 1));
#pragma unroll
          for (int u = 0; u < NTW; ++u) b_nxt[u] = ld4(bp + u * 16 * PITCH + 16 * (g + 1));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int u = 0; u < NTW; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_cur[i], b_cur[u][i], acc[u], 0, 0, 0);
        a_cur = a_nxt;
#pragma unroll
        for (int u = 0; u < NTW; ++u) b_cur[u] = b_nxt[u];
      }
    }
  }
};

// Workgroup -> (row block, hidden-unit block).  Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each
// with an L2 of its own: all hidden-unit blocks of a row block go to one XCD, so a row block's operand rows are
// fetched into one L2 only (the weights, shared by every row block, fit in each L2).
constexpr int GS_XCDS = 8;
__device__ __forceinline__ void step_block(int id, int H, int& rb, int& jb) {
  const int jblocks = (H + GS_JB - 1) / GS_JB;
  const int xcd = id % GS_XCDS, i = id / GS_XCDS;
  rb = (i / jblocks) * GS_XCDS + xcd;
  jb = i % jblocks;
}

template <int CELL> struct CellShape;
template <> struct CellShape<CELL_GRU> { static constexpr int G = 3, KC = 128; };
template <> struct CellShape<CELL_LSTM> { static constexpr int G = 4, KC = 64; };   // shorter chunks: 8 tiles of weights in LDS

template <int CELL> using StepFwdTile = StepTile<CellShape<CELL>::G, CellShape<CELL>::KC>;

// Workgroup `id` of a network's share of the launch; smem: StepFwdTile<CELL>::LDS_FLOATS floats.
template <int CELL>
__device__ __forceinline__ void step_fwd(const StepFwdArgs& a, const StepFwdNet& n, int id, float* smem) {
  constexpr int G = CellShape<CELL>::G;
  using Tile = StepFwdTile<CELL>;
  const int H = n.H, nb = a.nb, S = CELL == CELL_LSTM ? 2 * H : H;
  int rb, jb;
  step_block(id, H, rb, jb);
  const int row0 = rb * GS_ROWS, j0 = jb * GS_JB;
  if (row0 >= nb) return;
  int col0[2 * G], col_end[2 * G];      // tile wj * G + g: gate g of hidden units j0 + 16 wj ...
#pragma unroll
  for (int t = 0; t < 2 * G; ++t) { col0[t] = (t % G) * H + j0 + (t / G) * 16; col_end[t] = (t % G) * H + H; }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = wave & 1, wj = wave >> 1;
  const int j = j0 + wj * 16 + (lane & 15), jc = min(j, H - 1);
  const int rbase = row0 + wr * 16 + 4 * (lane >> 4);
  // the gate stage's own operands do not depend on the contraction: fetch them first (clamped addresses, no
  // branches) so their latency hides behind it
  float pgi[4][G], pst[4];      // pst: the state entry the gates blend with (GRU: h, LSTM: c)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = min(rbase + q, nb - 1);
    const long og = (long)row * G * H + jc;
#pragma unroll
    for (int g = 0; g < G; ++g) pgi[q][g] = n.gi[og + g * H];
    pst[q] = n.sin[(long)row * S + (CELL == CELL_LSTM ? H : 0) + jc];
  }
  float bias[G];
#pragma unroll
  for (int g = 0; g < G; ++g) bias[g] = n.b_hh[g * H + jc];
  f4 acc[G];
#pragma unroll
  for (int t = 0; t < G; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  Tile::mma(n.sin, S, row0, nb, n.w_hh, G * H, col0, col_end, H, smem, acc);
  if (j >= H) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = rbase + q;
    if (row >= nb) continue;
    const long og = (long)row * G * H + j;
    float keep = 1.0f;
    if (n.sin_next != nullptr && a.done != nullptr) keep = a.done[a.done_idx ? a.done_idx[row] : row] ? 0.0f : 1.0f;
    if (CELL == CELL_GRU) {
      const float ghr = acc[0][q] + bias[0], ghz = acc[1][q] + bias[1], ghn = acc[2][q] + bias[2];
      const float r = sigmoidf_(pgi[q][0] + ghr);
      const float zz = sigmoidf_(pgi[q][1] + ghz);
      const float nn = tanhf_(pgi[q][2] + r * ghn);
      const float h = (1.0f - zz) * nn + zz * pst[q];
      n.h_out[(long)row * n.ld_out + j] = h;
      if (n.sin_next != nullptr) n.sin_next[(long)row * S + j] = h * keep;
      if (n.pre_out != nullptr) { n.pre_out[og] = ghr; n.pre_out[og + H] = ghz; n.pre_out[og + 2 * H] = ghn; }
    } else {
      float pre[G];
#pragma unroll
      for (int g = 0; g < G; ++g) pre[g] = pgi[q][g] + acc[g][q] + bias[g];
      const float ii = sigmoidf_(pre[0]), ff = sigmoidf_(pre[1]), gg = tanhf_(pre[2]), oo = sigmoidf_(pre[3]);
      const float c = ff * pst[q] + ii * gg;
      const float h = oo * tanhf_(c);
      n.h_out[(long)row * n.ld_out + j] = h;
      if (n.c_out != nullptr) n.c_out[(long)row * n.ld_out + j] = c;
      if (n.sin_next != nullptr) { n.sin_next[(long)row * S + j] = h * keep; n.sin_next[(long)row * S + H + j] = c * keep; }
      if (n.pre_out != nullptr) {
#pragma unroll
        for (int g = 0; g < G; ++g) n.pre_out[og + g * H] = pre[g];
      }
    }
  }
}

template <int CELL>
__global__ __launch_bounds__(GS_THREADS) void step_fwd_kernel(const StepFwdArgs a) {
  __shared__ __attribute__((aligned(16))) float smem[StepFwdTile<CELL>::LDS_FLOATS];
  step_fwd<CELL>(a, a.net[blockIdx.y], blockIdx.x, smem);
}

template <int CELL>
__global__ __launch_bounds__(GS_THREADS) void step_bwd_kernel(const StepBwdArgs a) {
  constexpr int G = CellShape<CELL>::G;
  using Tile = StepTileKK<1, 128>;
  __shared__ __attribute__((aligned(16))) float smem[Tile::LDS_FLOATS];
  const int z = blockIdx.y;
  const StepBwdNet& n = a.net[z];
  const int H = n.H, nb = a.nb, S = CELL == CELL_LSTM ? 2 * H : H;
  int rb, jb;
  step_block(blockIdx.x, H, rb, jb);
  const int row0 = rb * GS_ROWS, j0 = jb * GS_JB;
  if (row0 >= nb) return;
  const bool has_next = n.dg_next != nullptr;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = wave & 1, wj = wave >> 1;
  const int j = j0 + wj * 16 + (lane & 15), jc = min(j, H - 1);
  const int rbase = row0 + wr * 16 + 4 * (lane >> 4);
  // the gate stage's own operands, fetched ahead of the contraction (clamped addresses, no branches)
  float pgi[4][G], ppre[4][G], pst[4], pdh[4], pcarry[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = min(rbase + q, nb - 1);
    const long o = (long)row * H + jc, og = (long)row * G * H + jc;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      ppre[q][g] = n.pre[og + g * H];
      pgi[q][g] = CELL == CELL_GRU ? n.gi[og + g * H] : 0.f;
    }
    pst[q] = n.sin[(long)row * S + (CELL == CELL_LSTM ? H : 0) + jc];
    pdh[q] = n.dh_ext[o];
    pcarry[q] = has_next ? n.carry[o] : 0.f;
  }
  f4 acc[1] = {f4{0.f, 0.f, 0.f, 0.f}};
  if (has_next) {
    const int col0[2] = {j0, j0 + 16}, col_end[2] = {H, H};      // rows of W_hh = hidden units
    Tile::mma(n.dg_next, G * H, row0, nb, n.w_hh, G * H, col0, col_end, G * H, smem, acc);
  }
  if (j >= H) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = rbase + q;
    if (row >= nb) continue;
    const long o = (long)row * H + j, og = (long)row * G * H + j;
    float keep = 1.0f;
    if (has_next && a.done != nullptr) keep = a.done[a.done_idx ? a.done_idx[row] : row] ? 0.0f : 1.0f;
    if (CELL == CELL_GRU) {
      float dh = pdh[q];
      if (has_next) dh += (acc[0][q] + pcarry[q]) * keep;
      const float ghn = ppre[q][2];
      const float r = sigmoidf_(pgi[q][0] + ppre[q][0]);
      const float zz = sigmoidf_(pgi[q][1] + ppre[q][1]);
      const float nn = tanhf_(pgi[q][2] + r * ghn);
      const float dn = dh * (1.0f - zz);
      const float dz = dh * (pst[q] - nn);
      const float dn_pre = dn * (1.0f - nn * nn);
      const float dr_pre = dn_pre * ghn * r * (1.0f - r);
      const float dz_pre = dz * zz * (1.0f - zz);
      n.carry[o] = dh * zz;
      n.dgi[og] = dr_pre; n.dgi[og + H] = dz_pre; n.dgi[og + 2 * H] = dn_pre;
      n.dg[og] = dr_pre; n.dg[og + H] = dz_pre; n.dg[og + 2 * H] = dn_pre * r;
    } else {
      float dh = pdh[q], dc = 0.f;
      if (has_next) { dh += acc[0][q] * keep; dc = pcarry[q] * keep; }
      const float ii = sigmoidf_(ppre[q][0]), ff = sigmoidf_(ppre[q][1]), gg = tanhf_(ppre[q][2]), oo = sigmoidf_(ppre[q][3]);
      const float tc = tanhf_(ff * pst[q] + ii * gg);
      const float d_o = dh * tc;
      const float dct = dc + dh * oo * (1.0f - tc * tc);
      n.carry[o] = dct * ff;
      n.dg[og] = dct * gg * ii * (1.0f - ii);
      n.dg[og + H] = dct * pst[q] * ff * (1.0f - ff);
      n.dg[og + 2 * H] = dct * ii * (1.0f - gg * gg);
      n.dg[og + 3 * H] = d_o * oo * (1.0f - oo);
    }
  }
}

// ---- gate stages of the split-operand kernels --------------------------------------------------------------
// One unit of one row.  gh: hidden-side terms with their bias.  st: what the gates blend with (GRU: h, LSTM: c), replaced by
// its successor times keep.  out: the gates as the backward pass reads them (GRU r, z, n and n's hidden-side term).
template <int CELL, int G>
__device__ __forceinline__ void gates_forward(const float (&gi)[G], const float (&gh)[G], float keep, float& st, float& h, float (&out)[4]) {
  if constexpr (CELL == CELL_GRU) {
    out[0] = sigmoidf_(gi[0] + gh[0]);
    out[1] = sigmoidf_(gi[1] + gh[1]);
    out[2] = tanhf_(gi[2] + out[0] * gh[2]);
    out[3] = gh[2];
    h = (1.0f - out[1]) * out[2] + out[1] * st;
    st = h * keep;
  } else {
    out[0] = sigmoidf_(gi[0] + gh[0]);
    out[1] = sigmoidf_(gi[1] + gh[1]);
    out[2] = tanhf_(gi[2] + gh[2]);
    out[3] = sigmoidf_(gi[G - 1] + gh[G - 1]);
    const float c = out[1] * st + out[0] * out[2];
    h = out[3] * tanhf_(c);
    st = c * keep;
  }
}

// With back = dg(t + 1) W_hh^T and keep = 1 - done, both 0 on the last step:
//   GRU:  dh = dh_ext + keep (back + carry);  d = [dr, dz, dn r], dn (pre-activation gradients; dgi has dn in place of dn r),
//         carry = dh z
//   LSTM: dh = dh_ext + keep back, dc = keep carry;  d = d loss / d pre-activations,  carry = (dc + dh o (1 - tanh^2 c')) f
template <int CELL, int G>
__device__ __forceinline__ void gates_backward(const float (&gate)[4], float st, float dh_ext, float back, float keep, float& carry,
                                               float (&d)[G], float& dn) {
  if constexpr (CELL == CELL_GRU) {
    const float dh = dh_ext + (back + carry) * keep;
    const float rr = gate[0], zz = gate[1], nn = gate[2];
    const float dz = dh * (st - nn);
    dn = dh * (1.0f - zz) * (1.0f - nn * nn);
    d[0] = dn * gate[3] * rr * (1.0f - rr);
    d[1] = dz * zz * (1.0f - zz);
    d[2] = dn * rr;
    carry = dh * zz;
  } else {
    const float dh = dh_ext + back * keep;
    const float ii = gate[0], ff = gate[1], gg = gate[2], oo = gate[3];
    const float tc = tanhf_(ff * st + ii * gg);
    const float dct = carry * keep + dh * oo * (1.0f - tc * tc);
    carry = dct * ff;
    d[0] = dct * gg * ii * (1.0f - ii);
    d[1] = dct * st * ff * (1.0f - ff);
    d[2] = dct * ii * (1.0f - gg * gg);
    d[G - 1] = dh * tc * oo * (1.0f - oo);
    dn = 0.f;
  }
}

// ---- a whole roll-out in one launch each way ---------------------------------------------------------------
// The update path's recurrence, for the width whose weights fit one CU: the states, and in the backward pass the gradients
// and the carried term, stay in the workgroup from step to step.
//
// A workgroup of 8 wavefronts owns 16 batch rows of one memory and all its hidden units: no step waits for another
// workgroup.  Wavefront w owns the hidden units w H / 8 .. (w + 1) H / 8 and all their gates, so the gate stage works on
// the lane's own accumulators.  The products run on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16) on operands split in
// three (gemm.hip has the arithmetic): operand A holds 16 weight columns (forward: one gate of 16 hidden units; backward:
// 16 hidden units), operand B the 16 rows, D[4 * (lane / 16) + r][lane % 16] the four consecutive units of a row.
//
// The split weights stay in registers and LDS for all steps (295 KB for a GRU of 128; what a width of 256 has, 1.2 MB, does
// not fit and would be streamed from the L2 on every step: 12 to 17 us a step, where a launch per step takes 10 to 19).
// What is left of a step is the contraction (1 us of matrix instructions), the gate stage and two barriers, one after the
// other; its own operands are requested a whole step ahead.  Measured at 16 to 1024 rows and two memories of 128, us a step,
// one launch per step in brackets: GRU forward 3.6 to 3.9 (6.7 to 7.8), backward 3.7 to 4.3 (6.2 to 8.3); LSTM forward 4.7 to
// 5.0 (7.0 to 8.9), backward 4.0 to 4.3 (7.3 to 8.5).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int SQ_ROWS = 16;
constexpr int SQ_WAVES = 8;
constexpr int SQ_THREADS = 64 * SQ_WAVES;
constexpr int SQ_BLOCK = 1024;         // bytes of one part of a 16-column, 32-index operand block

// Operand B in LDS: 16 bytes are one part of eight consecutive contraction indices of a row, [part][index / 8][row].
template <int K> __device__ __forceinline__ int sq_unit(int part, int k8, int row) { return part * (K * 32) + (k8 * SQ_ROWS + row) * 16; }

// Splits the values of contraction indices k .. k + 3 (k % 4 == 0) of a row and writes them to LDS.
template <int K>
__device__ __forceinline__ void sq_put(char* x, int k, int row, f4 v, float scale) {
  uint2 p[3];
  split_pair(scale * v[0], scale * v[1], p[0].x, p[1].x, p[2].x);
  split_pair(scale * v[2], scale * v[3], p[0].y, p[1].y, p[2].y);
#pragma unroll
  for (int s = 0; s < 3; ++s) *reinterpret_cast<uint2*>(x + sq_unit<K>(s, k >> 3, row) + (k & 4) * 2) = p[s];
}

// The contraction of one step: acc[tile] += W(tile)^T X over K indices, TILES tiles of 16 weight columns per wavefront.  Blocks
// (16 columns, 32 indices, one part) are numbered in the order of their use; the first NREG live in registers, the others in LDS.
template <int K, int TILES, int NREG>
struct SeqContract {
  static constexpr int KS = K / 32, GB = 3 * TILES, NB = KS * GB, NLDS = NB - NREG;
  static constexpr int LDS_BYTES = NLDS * SQ_WAVES * SQ_BLOCK;

  u32x4 reg[NREG];
  char* lw;                                // the lane's place in the wavefront's blocks in LDS

  __device__ __forceinline__ void setup(const uint16_t* packed, int wave, int lane, char* lds) {
    const char* w = reinterpret_cast<const char*>(packed) + wave * SQ_BLOCK + lane * 16;
    lw = lds + (wave * NLDS) * SQ_BLOCK + lane * 16;
#pragma unroll
    for (int n = 0; n < NREG; ++n) reg[n] = *reinterpret_cast<const u32x4*>(w + n * (SQ_WAVES * SQ_BLOCK));
#pragma unroll
    for (int n = NREG; n < NB; ++n)
      *reinterpret_cast<u32x4*>(lw + (n - NREG) * SQ_BLOCK) = *reinterpret_cast<const u32x4*>(w + n * (SQ_WAVES * SQ_BLOCK));
#pragma unroll
    for (int n = 0; n < NREG; ++n) asm volatile("" : "+v"(reg[n]));     // held, not loaded again
  }
  // NACC: TILES, or 2 TILES with alternate steps of 32 in sums of their own (shorter chains where there are few tiles)
  template <int NACC>
  __device__ __forceinline__ void run(const char* x, int lane, f4 (&acc)[NACC]) {
    const int kq = lane >> 4, m = lane & 15;
    const char* xb = x + sq_unit<K>(0, kq, m);
    bf16x8 b[2][3];
    auto read_x = [&](int ks) {
#pragma unroll
      for (int s = 0; s < 3; ++s) b[ks & 1][s] = *reinterpret_cast<const bf16x8*>(xb + s * (K * 32) + ks * (4 * SQ_ROWS * 16));
    };
    read_x(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) read_x(ks + 1);
      bf16x8 a[GB];
#pragma unroll
      for (int n = 0; n < GB; ++n) {
        const int id = ks * GB + n;
        a[n] = __builtin_bit_cast(bf16x8, id < NREG ? reg[id < NREG ? id : 0] : *reinterpret_cast<const u32x4*>(lw + (id - NREG) * SQ_BLOCK));
      }
      constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
          const int at = i + (NACC == 2 * TILES ? (ks & 1) * TILES : 0);
          acc[at] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[3 * i + PA[p]], b[ks & 1][PB[p]], acc[at], 0, 0, 0);
        }
    }
  }
};

// Sums of fp32 products in place of the non-finite ones of a tile (such inputs have no split, see gemm.hip).  w: element
// (k, column) at w[k * wk + column * wc], `col` the tile's first column; x: the lane's row, contiguous along k.  RAGGED: K need
// not be a multiple of 16.
template <bool RAGGED = false>
__device__ __forceinline__ void sq_repeat_fp32(const float* w, long wk, long wc, const float* x, int K, int lane, f4& acc) {
  const int kq = lane >> 4, m = lane & 15;
  f4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int k0 = 0; k0 < K; k0 += 16) {
    float a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = k0 + 4 * i + kq, kr = RAGGED ? min(k, K - 1) : k;
      a[i] = w[(long)kr * wk + m * wc];
      b[i] = x[kr];
      if (RAGGED && k >= K) a[i] = b[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (!__builtin_isfinite(acc[r])) acc[r] = c[r];
}

// Blocks in registers, as many as it takes for the rest to fit LDS, forward and backward.
template <int CELL, int H> struct SeqShape;
template <> struct SeqShape<CELL_GRU, 128> { static constexpr int G = 3, REGF = 18, REGB = 21; };
template <> struct SeqShape<CELL_LSTM, 128> { static constexpr int G = 4, REGF = 30, REGB = 34; };

template <int CELL, int H> struct SeqFwd {
  using S = SeqShape<CELL, H>;
  static constexpr int UT = H / (16 * SQ_WAVES), W = CELL == CELL_LSTM ? 2 * H : H;      // unit tiles per wavefront, state width
  using C = SeqContract<H, S::G * UT, S::REGF>;
  static constexpr int X_BYTES = H * 96, BIAS = X_BYTES, WEIGHTS = BIAS + S::G * H * 4;
  static constexpr int LDS = WEIGHTS + C::LDS_BYTES;
};

template <int CELL, int H>
__global__ __launch_bounds__(SQ_THREADS, 2) void seq_fwd_kernel(const SeqArgs a) {
  using F = SeqFwd<CELL, H>;
  constexpr int G = F::S::G, UT = F::UT, W = F::W, GH = G * H;
  extern __shared__ __align__(16) char lds[];
  const SeqNet& n = a.net[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, kq = lane >> 4, j0 = wave * (H / SQ_WAVES);
  const int nb = a.nb, row = min((int)blockIdx.x * SQ_ROWS + b, nb - 1);
  const bool ok = (int)blockIdx.x * SQ_ROWS + b < nb;       // rows past the end repeat the last one and store nothing
  float* bias = reinterpret_cast<float*>(lds + F::BIAS);
  for (int i = tid; i < GH; i += SQ_THREADS) bias[i] = n.b_hh[i];
  const int ju = j0 + 4 * kq;                               // the lane's units: ju + 16 u + 0 .. 3
  const float scale = split_scale(b), unscale = split_unscale(b);

  f4 gi[UT][G], gi_next[UT][G], st[UT], h[UT];           // st: what the gates blend with (GRU: h, LSTM: c)
#pragma unroll
  for (int u = 0; u < UT; ++u) {
    const float* s0 = n.hin + (long)row * W + ju + 16 * u;
    const f4 h0 = ld4(s0);
    st[u] = CELL == CELL_LSTM ? ld4(s0 + H) : h0;
    sq_put<H>(lds, ju + 16 * u, b, h0, scale);
#pragma unroll
    for (int g = 0; g < G; ++g) gi[u][g] = ld4(n.gi + (long)row * GH + g * H + ju + 16 * u);
  }
  // episode ends: the flag of a step is requested one step ahead, its place two steps ahead
  auto place = [&](int t) { return a.ridx ? a.ridx[(long)min(t, a.T - 1) * nb + row] : row; };
  int flag = a.done ? a.done[place(0)] : 0, flag_next = 0, at = place(1), at_next = 0;
  typename F::C c;
  c.setup(n.packed, wave, lane, lds + F::WEIGHTS);
  __syncthreads();

#pragma unroll 1
  for (int t = 0; t < a.T; ++t) {
    const long r0 = (long)t * nb + row, r1 = (long)min(t + 1, a.T - 1) * nb + row;
#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
      for (int g = 0; g < G; ++g) gi_next[u][g] = ld4(n.gi + r1 * GH + g * H + ju + 16 * u);
    if (a.done) flag_next = a.done[at];
    at_next = place(t + 2);
    f4 acc[UT * G];
#pragma unroll
    for (int i = 0; i < UT * G; ++i) acc[i] = f4{0.f, 0.f, 0.f, 0.f};
    c.run(lds, lane, acc);
    float z = 0.f;                                          // becomes NaN with any non-finite sum
#pragma unroll
    for (int i = 0; i < UT * G; ++i) {
      acc[i] *= unscale;
#pragma unroll
      for (int r = 0; r < 4; ++r) z = fmaf(acc[i][r], 0.f, z);
    }
    if (__any(!(z == 0.f))) {
#pragma unroll
      for (int i = 0; i < UT * G; ++i) sq_repeat_fp32(n.w_hh + i % G * H + j0 + 16 * (i / G), GH, 1, n.hin + r0 * W, H, lane, acc[i]);
    }
    const float keep = flag ? 0.f : 1.f;
    f4 out[UT][4];
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      f4 bv[G];
#pragma unroll
      for (int g = 0; g < G; ++g) bv[g] = ld4(bias + g * H + ju + 16 * u);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float x[G], y[G], o[4], hv, sv = st[u][r];
#pragma unroll
        for (int g = 0; g < G; ++g) { x[g] = gi[u][g][r]; y[g] = acc[u * G + g][r] + bv[g][r]; }
        gates_forward<CELL>(x, y, keep, sv, hv, o);
        h[u][r] = hv; st[u][r] = sv;
#pragma unroll
        for (int g = 0; g < 4; ++g) out[u][g][r] = o[g];
      }
    }
    __syncthreads();                                        // every wavefront has read the old states
    const bool more = t + 1 < a.T;
#pragma unroll
    for (int u = 0; u < UT; ++u) sq_put<H>(lds, ju + 16 * u, b, h[u] * keep, scale);
#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
      for (int g = 0; g < G; ++g) gi[u][g] = gi_next[u][g];
    flag = flag_next;
    at = at_next;
    if (ok) {
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        const int j = ju + 16 * u;
        st4(n.hs + r0 * H + j, h[u]);
        if (more) {
          float* nx = n.hin + (r0 + nb) * W + j;
          st4(nx, h[u] * keep);
          if (CELL == CELL_LSTM) st4(nx + H, st[u]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) st4(n.gi + r0 * GH + g * H + j, out[u][g]);
        if (CELL == CELL_GRU) st4(n.ghn + r0 * H + j, out[u][3]);
      }
    }
    __syncthreads();
  }
}

template <int CELL, int H> struct SeqBwd {
  using S = SeqShape<CELL, H>;
  static constexpr int UT = H / (16 * SQ_WAVES), W = CELL == CELL_LSTM ? 2 * H : H, GH = S::G * H;
  using C = SeqContract<GH, UT, S::REGB>;
  static constexpr int X_BYTES = GH * 96, WEIGHTS = X_BYTES;
  static constexpr int LDS = WEIGHTS + C::LDS_BYTES;
};

template <int CELL, int H>
__global__ __launch_bounds__(SQ_THREADS, 2) void seq_bwd_kernel(const SeqArgs a) {
  using F = SeqBwd<CELL, H>;
  constexpr int G = F::S::G, UT = F::UT, W = F::W, GH = F::GH;
  extern __shared__ __align__(16) char lds[];
  const SeqNet& n = a.net[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, kq = lane >> 4, j0 = wave * (H / SQ_WAVES);
  const int nb = a.nb, row = min((int)blockIdx.x * SQ_ROWS + b, nb - 1);
  const bool ok = (int)blockIdx.x * SQ_ROWS + b < nb;
  const int ju = j0 + 4 * kq;
  const float scale = split_scale(b), unscale = split_unscale(b);

  struct Operands { f4 gate[UT][4], st[UT], dh[UT]; };   // gate: GRU r, z, n, ghn; LSTM i, f, g, o.  st: h or c before the step
  auto operands = [&](int t, Operands& o) {
    const long r0 = (long)t * nb + row;
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      const int j = ju + 16 * u;
#pragma unroll
      for (int g = 0; g < G; ++g) o.gate[u][g] = ld4(n.gi + r0 * GH + g * H + j);
      if (CELL == CELL_GRU) o.gate[u][3] = ld4(n.ghn + r0 * H + j);
      o.st[u] = ld4(n.hin + r0 * W + (CELL == CELL_LSTM ? H : 0) + j);
      o.dh[u] = ld4(n.dh + r0 * H + j);
    }
  };
  Operands now, next;
  operands(a.T - 1, now);
  f4 carry[UT];
#pragma unroll
  for (int u = 0; u < UT; ++u) carry[u] = f4{0.f, 0.f, 0.f, 0.f};
  // the flag of step t gates what step t + 1 sends back: requested one step ahead, its place two steps ahead
  auto place = [&](int t) { return a.ridx ? a.ridx[(long)max(t, 0) * nb + row] : row; };
  int flag = 0, flag_next = 0, at = place(a.T - 2), at_next = 0;
  typename F::C c;
  c.setup(n.packed_t, wave, lane, lds + F::WEIGHTS);

#pragma unroll 1
  for (int t = a.T - 1; t >= 0; --t) {
    const long r0 = (long)t * nb + row;
    operands(max(t - 1, 0), next);
    if (a.done) flag_next = a.done[at];
    at_next = place(t - 2);
    f4 back[UT];
#pragma unroll
    for (int u = 0; u < UT; ++u) back[u] = f4{0.f, 0.f, 0.f, 0.f};
    if (t + 1 < a.T) {
      f4 acc[2 * UT];
#pragma unroll
      for (int i = 0; i < 2 * UT; ++i) acc[i] = f4{0.f, 0.f, 0.f, 0.f};
      c.run(lds, lane, acc);
      float z = 0.f;
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        back[u] = (acc[u] + acc[UT + u]) * unscale;
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(back[u][r], 0.f, z);
      }
      if (__any(!(z == 0.f))) {
#pragma unroll
        for (int u = 0; u < UT; ++u)
          sq_repeat_fp32(n.w_hh + (long)(j0 + 16 * u) * GH, 1, GH, n.dg + (r0 + nb) * GH, GH, lane, back[u]);
      }
    }
    const float keep = t + 1 == a.T || flag ? 0.f : 1.f;
    f4 d[UT][G], dn[UT];
#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float gt[4], dv[G], dnv, cv = carry[u][r];
#pragma unroll
        for (int g = 0; g < 4; ++g) gt[g] = now.gate[u][g][r];
        gates_backward<CELL>(gt, now.st[u][r], now.dh[u][r], back[u][r], keep, cv, dv, dnv);
        carry[u][r] = cv; dn[u][r] = dnv;
#pragma unroll
        for (int g = 0; g < G; ++g) d[u][g][r] = dv[g];
      }
    __syncthreads();                                        // every wavefront has read the gradients of the step after
    if (t > 0) {
#pragma unroll
      for (int u = 0; u < UT; ++u)
#pragma unroll
        for (int g = 0; g < G; ++g) sq_put<GH>(lds, g * H + ju + 16 * u, b, d[u][g], scale);
    }
    now = next;
    flag = flag_next;
    at = at_next;
    if (ok) {
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        const long o = r0 * GH + ju + 16 * u;
#pragma unroll
        for (int g = 0; g < G; ++g) st4(n.dg + o + g * H, d[u][g]);
        if (CELL == CELL_GRU) { st4(n.dgi + o, d[u][0]); st4(n.dgi + o + H, d[u][1]); st4(n.dgi + o + 2 * H, dn[u]); }
      }
    }
    __syncthreads();
  }
}

// ---- act(): one time step on split operands ----------------------------------------------------------------
// For many rows and widths that are multiples of 64.  A workgroup of 4 wavefronts takes 64 rows and 32 hidden units; wavefront w
// its rows 16 w .., operands and accumulators as in the roll-out kernels above (operand A 16 weight columns, operand B 16
// rows), so the gate stage works on the lane's own accumulators.  The weights come split, in the order in which LDS holds them, a
// chunk of 64 (LSTM: 32) contraction indices at a time through registers; the launch that copies the states splits them.  Each
// workgroup splitting them for itself, once per 64 rows, took two thirds of the loop's vector instructions: two GRUs of 256 at
// 4096 rows with 48 inputs in front of [512, 256, 128] 91.1 us a call that way, 84.4 this way; LSTMs with 235 in front of [256, 128]
// 102 and 90.  Rows are split in registers by the only wavefront that uses them.
// The input side's contraction follows the hidden side's in the same loop, into sums of its own (which GRU's candidate needs, and
// chains stay short): no product by itself, no [rows, G H] matrix written and read, 95.9 us a call with them.
constexpr int ST_ROWS = 64, ST_UNITS = 32, ST_THREADS = 256;

// Workgroup -> (network, row block, unit block).  Workgroup ids go round-robin to the 8 XCDs; each XCD takes one network, half
// of its units and half (of a single network: a quarter) of its rows, so that an L2 fetches half the weights.
struct StepGrid {
  int row_groups, unit_blocks, per_group, blocks;
  __host__ __device__ StepGrid(int n_nets, int nb, int H) {
    row_groups = n_nets == 2 ? 2 : 4;
    unit_blocks = H / ST_UNITS;
    per_group = (unit_blocks + 1) / 2;
    blocks = 8 * per_group * (((nb + ST_ROWS - 1) / ST_ROWS + row_groups - 1) / row_groups);
  }
};

typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));

// Contraction indices of a chunk: two workgroups are to fit a CU (72 KB of LDS for three gates, 48 for four).
template <int CELL> struct StepSplit {
  static constexpr int G = CellShape<CELL>::G, KC = CELL == CELL_LSTM ? 32 : 64, KS = KC / 32;
  static constexpr int NT = 2 * G, CHUNK = KS * NT * 3 * SQ_BLOCK;         // tiles of 16 weight columns, bytes of a chunk
  static constexpr int LOADS = CHUNK / (ST_THREADS * 16);
};

// Whether the weights of a step come split.  A GRU's whose inputs stay apart (step_takes_input) are split by every workgroup: without
// the input side's chunks the split ahead costs more than it saves.  rslx_memory_step, split ahead and in the workgroups, us: 128 units, 300
// inputs, 4301 rows 32.2 and 31.5; 64 units, 235 inputs, 8602 rows 35.0 and 34.2; 512 units, 1500 inputs, 1076 rows 86.2 and 83.5.  An
// LSTM's gains nothing from it (128 units, 300 inputs, 8602 rows 54.9 in the workgroups, 54.5 ahead).
__host__ __device__ constexpr bool step_comes_split(int cell, bool input) { return cell == CELL_LSTM || input; }

// Chunks of the hidden side, then those of the input side.
template <int CELL> __host__ __device__ __forceinline__ int step_chunks(int H, int D) {
  return H / StepSplit<CELL>::KC + (D + StepSplit<CELL>::KC - 1) / StepSplit<CELL>::KC;
}

// Unit e of a network's weights, split: [unit block][chunk][step of 32][unit tile][gate][part][lane], zeros past the input's width.
template <int CELL>
__device__ __forceinline__ void step_pack(const StepPackJob& J, long e) {
  using S = StepSplit<CELL>;
  const int total = step_chunks<CELL>(J.H, J.D), NC = J.H / S::KC, GH = S::G * J.H;
  const int lane = (int)e & 63;
  const long blk = e >> 6;
  const int t = (int)(blk % S::NT), ks = (int)(blk / S::NT % S::KS);
  const int uc = (int)(blk / (S::NT * S::KS)), c = uc % total, ub = uc / total;
  if (ub >= J.H / ST_UNITS) return;
  const bool in = c >= NC;
  const float* w = (in ? J.w_ih : J.w_hh) + t % S::G * J.H + ub * ST_UNITS + 16 * (t / S::G) + (lane & 15);
  const int k0 = (in ? c - NC : c) * S::KC + 32 * ks + 8 * (lane >> 4), K = in ? J.D : J.H;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = w[(long)min(k0 + i, K - 1) * GH];
  u32x4 part[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t p0, p1, p2;
    split_pair(k0 + 2 * i < K ? SPLIT_SCALE * v[2 * i] : 0.f, k0 + 2 * i + 1 < K ? SPLIT_SCALE * v[2 * i + 1] : 0.f, p0, p1, p2);
    part[0][i] = p0; part[1][i] = p1; part[2][i] = p2;
  }
  char* dst = reinterpret_cast<char*>(J.dst) + blk * (3 * SQ_BLOCK) + lane * 16;
#pragma unroll
  for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(dst + s * SQ_BLOCK) = part[s];
}

// Unit block ub, rows from row0 of a network; lds: 2 CHUNK bytes.  INPUT: with the input side's contraction, else gi holds its sums.
template <int CELL, bool INPUT>
__device__ __forceinline__ void step_split(const StepFwdNet& n, int nb, int ub, int row0, char* lds) {
  using S = StepSplit<CELL>;
  constexpr int G = S::G, NT = S::NT, KC = S::KC, CHUNK = S::CHUNK, LOADS = S::LOADS;
  const int H = n.H, GH = G * H, SW = CELL == CELL_LSTM ? 2 * H : H;
  if (ub >= H / ST_UNITS || row0 >= nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, kq = lane >> 4, j0 = ub * ST_UNITS, ju = j0 + 4 * kq;      // the lane's units: ju + 16 u + 0 .. 3
  const int row = min(row0 + 16 * wave + b, nb - 1);
  const bool ok = row0 + 16 * wave + b < nb;             // rows past the end repeat the last one and store nothing
  const float scale = split_scale(b), unscale = split_unscale(b);
  const int NC = H / KC, D = n.D, total = step_chunks<CELL>(H, INPUT ? D : 0);

  // weights: this lane's 16-byte units of a chunk, or its column of 32 and eight contraction indices for all gates, to be split
  constexpr bool PACKED = step_comes_split(CELL, INPUT);
  const char* wsrc = reinterpret_cast<const char*>(n.pack) + (long)ub * total * CHUNK + tid * 16;
  u32x4 wv[LOADS];
  const int wc = tid & 31, wk = tid >> 5;
  float wf[G][8];
  static_assert(PACKED || ST_THREADS == 4 * KC, "a lane's share of a chunk");
  auto load_w = [&](int c) {
    if constexpr (PACKED) {
      const char* p = wsrc + (long)min(c, total - 1) * CHUNK;
#pragma unroll
      for (int i = 0; i < LOADS; ++i) wv[i] = *reinterpret_cast<const u32x4*>(p + i * (ST_THREADS * 16));
    } else {
      const int k0 = min(c, NC - 1) * KC + 8 * wk;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) wf[g][i] = n.w_hh[(uint32_t)(k0 + i) * (uint32_t)GH + (uint32_t)(g * H + j0 + wc)];
    }
  };
  auto put_w = [&](int buf) {            // blocks: [step of 32][unit tile][gate][part]
    if constexpr (PACKED) {
      char* dst = lds + buf * CHUNK + tid * 16;
#pragma unroll
      for (int i = 0; i < LOADS; ++i) *reinterpret_cast<u32x4*>(dst + i * (ST_THREADS * 16)) = wv[i];
    } else {
      char* dst = lds + buf * CHUNK + (((wk >> 2) * NT + (wc >> 4) * G) * 3) * SQ_BLOCK + ((wk & 3) * 16 + (wc & 15)) * 16;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        u32x4 part[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t p0, p1, p2;
          split_pair(SPLIT_SCALE * wf[g][2 * i], SPLIT_SCALE * wf[g][2 * i + 1], p0, p1, p2);
          part[0][i] = p0; part[1][i] = p1; part[2][i] = p2;
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(dst + (3 * g + s) * SQ_BLOCK) = part[s];
      }
    }
  };
  // rows: operand B's eight contraction indices of every step of 32 of a chunk
  const float* xrow = n.sin + (long)row * SW;
  const float* irow = INPUT ? n.x + (long)row * D : nullptr;
  auto load_x = [&](int c, f4 (&x)[2 * S::KS]) {
    if (!INPUT || c < NC) {
      const float* p = xrow + (INPUT ? c : min(c, NC - 1)) * KC + 8 * kq;
#pragma unroll
      for (int i = 0; i < 2 * S::KS; ++i) x[i] = ld4(p + 32 * (i >> 1) + 4 * (i & 1));
    } else if (c < total) {
      const int k0 = (c - NC) * KC + 8 * kq;
      if ((D & 3) == 0 || (c + 1 - NC) * KC <= D) {       // whole groups of four; rows of an odd width are aligned to 4 bytes only
#pragma unroll
        for (int i = 0; i < 2 * S::KS; ++i) x[i] = *reinterpret_cast<const f4_any*>(irow + min(k0 + 32 * (i >> 1) + 4 * (i & 1), D - 4));
      } else {
#pragma unroll
        for (int i = 0; i < 2 * S::KS; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) x[i][r] = irow[min(k0 + 32 * (i >> 1) + 4 * (i & 1) + r, D - 1)];
      }
    }
  };

  f4 acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = f4{0.f, 0.f, 0.f, 0.f};
  f4 x0[2 * S::KS], x1[2 * S::KS];
  load_w(0);
  load_x(0, x0);
  // the gate stage's own operands: their latency passes under the contraction
  f4 gi[2][G], st[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int g = 0; g < G; ++g) gi[u][g] = INPUT ? f4{0.f, 0.f, 0.f, 0.f} : ld4(n.gi + (long)row * GH + g * H + ju + 16 * u);
    st[u] = ld4(n.sin + (long)row * SW + (CELL == CELL_LSTM ? H : 0) + ju + 16 * u);
  }
  put_w(0);
  load_w(1);
  __syncthreads();
  auto chunk = [&](int c, const f4 (&x)[2 * S::KS], f4 (&next)[2 * S::KS], auto sum) {
    load_x(c + 1, next);
    const char* wl = lds + (c & 1) * CHUNK + lane * 16;
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) {
      u32x4 xb[3];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4& v = x[2 * ks + (i >> 1)];
        uint32_t p0, p1, p2;
        split_pair(scale * v[2 * (i & 1)], scale * v[2 * (i & 1) + 1], p0, p1, p2);
        xb[0][i] = p0; xb[1][i] = p1; xb[2][i] = p2;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8 w[3 * G];
#pragma unroll
        for (int i = 0; i < 3 * G; ++i) w[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wl + ((ks * NT + u * G) * 3 + i) * SQ_BLOCK));
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
          for (int g = 0; g < G; ++g)
            sum(u, g) = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[3 * g + PA[p]], __builtin_bit_cast(bf16x8, xb[PB[p]]), sum(u, g), 0, 0, 0);
      }
    }
    if (c + 1 < total) {
      put_w((c + 1) & 1);
      load_w(c + 2);
    }
    __syncthreads();
  };
  const auto hidden = [&](int u, int g) -> f4& { return acc[u * G + g]; };
  const auto input = [&](int u, int g) -> f4& { return gi[u][g]; };
  for (int c = 0; c < NC; c += 2) {
    chunk(c, x0, x1, hidden);
    if (c + 1 < NC) chunk(c + 1, x1, x0, hidden);
    else if (INPUT)
#pragma unroll
      for (int i = 0; i < 2 * S::KS; ++i) x0[i] = x1[i];
  }
  if constexpr (INPUT) {
    for (int c = NC; c < total; c += 2) {
      chunk(c, x0, x1, input);
      if (c + 1 < total) chunk(c + 1, x1, x0, input);
    }
  }
  float nf = 0.f;                                         // becomes NaN with any non-finite sum
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    acc[i] *= unscale;
#pragma unroll
    for (int r = 0; r < 4; ++r) nf = fmaf(acc[i][r], 0.f, nf);
  }
  if (__any(!(nf == 0.f))) {
#pragma unroll
    for (int i = 0; i < NT; ++i) sq_repeat_fp32(n.w_hh + i % G * H + j0 + 16 * (i / G), GH, 1, xrow, H, lane, acc[i]);
  }
  if constexpr (INPUT) {
    nf = 0.f;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      f4& v = gi[i / G][i % G];
      v *= unscale;
#pragma unroll
      for (int r = 0; r < 4; ++r) nf = fmaf(v[r], 0.f, nf);
    }
    if (__any(!(nf == 0.f))) {
#pragma unroll
      for (int i = 0; i < NT; ++i) sq_repeat_fp32<true>(n.w_ih + i % G * H + j0 + 16 * (i / G), GH, 1, irow, D, lane, gi[i / G][i % G]);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) gi[i / G][i % G] += ld4(n.b_ih + i % G * H + ju + 16 * (i / G));
  }
  if (!ok) return;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int j = ju + 16 * u;
    f4 bv[G], h;
#pragma unroll
    for (int g = 0; g < G; ++g) bv[g] = ld4(n.b_hh + g * H + j);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x[G], y[G], out[4], hv, sv = st[u][r];
#pragma unroll
      for (int g = 0; g < G; ++g) { x[g] = gi[u][g][r]; y[g] = acc[u * G + g][r] + bv[g][r]; }
      gates_forward<CELL>(x, y, 1.f, sv, hv, out);
      h[r] = hv; st[u][r] = sv;
    }
    st4(n.h_out + (long)row * n.ld_out + j, h);
    if (CELL == CELL_LSTM) st4(n.c_out + (long)row * n.ld_out + j, st[u]);
  }
}

// Which networks of a launch contract their inputs in the step (StepFwdNet::x).
enum StepInput : int { STEP_IN_NONE = 0, STEP_IN_ALL = 1, STEP_IN_SOME = 2 };

template <int CELL, int IN>
__device__ __forceinline__ void step_split_in(const StepFwdNet& n, int nb, int ub, int row0, char* lds) {
  if (IN == STEP_IN_ALL || (IN == STEP_IN_SOME && n.x != nullptr)) step_split<CELL, true>(n, nb, ub, row0, lds);
  else step_split<CELL, false>(n, nb, ub, row0, lds);
}

// One network, or two of one width.  Without inputs the LSTM's step fits three workgroups on a CU (164 registers, 48 KB of LDS); in one
// kernel with the other form it had two: rslx_memory_step of 64 units with 160 inputs at 33 424 rows 62.3 and 59.1 us, of 128 with 300 at
// 8602 rows 56.5 and 54.5.
template <int CELL, int IN>
__global__ __launch_bounds__(ST_THREADS, CELL == CELL_LSTM && IN == STEP_IN_NONE ? 3 : 2) void step_split_kernel(const StepFwdArgs a) {
  extern __shared__ __align__(16) char lds[];
  const StepGrid grid(a.n_nets, a.nb, a.net[0].H);
  const int xcd = blockIdx.x & 7, id = blockIdx.x >> 3;
  const int z = a.n_nets == 2 ? xcd >> 2 : 0, rg = a.n_nets == 2 ? xcd & 1 : xcd & 3, ug = a.n_nets == 2 ? (xcd >> 1) & 1 : xcd >> 2;
  step_split_in<CELL, IN>(a.net[z], a.nb, ug * grid.per_group + id % grid.per_group, ((id / grid.per_group) * grid.row_groups + rg) * ST_ROWS, lds);
}

// Two networks of different widths, the wider one first (blockIdx.y): each over the whole chip and through the kernel that its own
// sizes call for (bit z of split), in one launch.
template <int CELL>
__global__ __launch_bounds__(ST_THREADS, 2) void step_uneven_kernel(const StepFwdArgs a, int split) {
  extern __shared__ __align__(16) char lds[];
  const StepFwdNet& n = a.net[blockIdx.y];
  if ((split >> blockIdx.y) & 1) {
    const StepGrid grid(1, a.nb, n.H);
    const int xcd = blockIdx.x & 7, id = blockIdx.x >> 3;
    step_split_in<CELL, STEP_IN_SOME>(n, a.nb, (xcd >> 2) * grid.per_group + id % grid.per_group, ((id / grid.per_group) * grid.row_groups + (xcd & 3)) * ST_ROWS, lds);
  } else {
    step_fwd<CELL>(a, n, blockIdx.x, reinterpret_cast<float*>(lds));
  }
}

template <int CELL, int IN>
hipError_t step_split_launch(const StepFwdArgs& a, hipStream_t stream) {
  constexpr int bytes = 2 * StepSplit<CELL>::CHUNK;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(step_split_kernel<CELL, IN>), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((step_split_kernel<CELL, IN>), dim3(StepGrid(a.n_nets, a.nb, a.net[0].H).blocks), dim3(ST_THREADS), bytes, stream, a);
  return hipGetLastError();
}

template <int CELL>
hipError_t step_split_launch(const StepFwdArgs& a, hipStream_t stream) {
  int in = 0;
  for (int k = 0; k < a.n_nets; ++k) in += a.net[k].x != nullptr;
  if (in == 0) return step_split_launch<CELL, STEP_IN_NONE>(a, stream);
  return in == a.n_nets ? step_split_launch<CELL, STEP_IN_ALL>(a, stream) : step_split_launch<CELL, STEP_IN_SOME>(a, stream);
}

template <int CELL>
hipError_t step_uneven_launch(const StepFwdArgs& a, int split, int rest_blocks, hipStream_t stream) {
  static_assert(GS_THREADS == ST_THREADS, "one launch");
  constexpr int bytes_split = 2 * StepSplit<CELL>::CHUNK, bytes_rest = StepFwdTile<CELL>::LDS_FLOATS * 4;
  const int bytes = split == 3 || bytes_split > bytes_rest ? bytes_split : bytes_rest;
  int blocks = rest_blocks;
  for (int z = 0; z < 2; ++z)
    if (split >> z & 1) blocks = std::max(blocks, StepGrid(1, a.nb, a.net[z].H).blocks);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(step_uneven_kernel<CELL>), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((step_uneven_kernel<CELL>), dim3(blocks, 2), dim3(ST_THREADS), bytes, stream, a, split);
  return hipGetLastError();
}

template <int CELL, int H>
hipError_t seq_launch(const SeqArgs& a, bool backward, hipStream_t stream) {
  const dim3 grid((a.nb + SQ_ROWS - 1) / SQ_ROWS, a.n_nets);
  const void* kernel = backward ? reinterpret_cast<const void*>(seq_bwd_kernel<CELL, H>) : reinterpret_cast<const void*>(seq_fwd_kernel<CELL, H>);
  const int bytes = backward ? SeqBwd<CELL, H>::LDS : SeqFwd<CELL, H>::LDS;
  static_assert(SeqBwd<CELL, H>::LDS <= 160 * 1024 && SeqFwd<CELL, H>::LDS <= 160 * 1024, "LDS");
  hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  if (backward) hipLaunchKernelGGL((seq_bwd_kernel<CELL, H>), grid, dim3(SQ_THREADS), bytes, stream, a);
  else hipLaunchKernelGGL((seq_fwd_kernel<CELL, H>), grid, dim3(SQ_THREADS), bytes, stream, a);
  return hipGetLastError();
}

hipError_t seq_dispatch(const SeqArgs& a, bool backward, hipStream_t stream) {
  if (a.nb <= 0 || a.n_nets <= 0 || a.T <= 0) return hipSuccess;
  return a.cell == CELL_LSTM ? seq_launch<CELL_LSTM, 128>(a, backward, stream) : seq_launch<CELL_GRU, 128>(a, backward, stream);
}

__device__ __forceinline__ void row_gather(const RowGatherArgs& a, const RowGatherJob& J, long e) {
  const int q = J.H >> 2;
  if (e >= (long)a.nb * q) return;
  const int i = (int)(e / q), j = (int)(e - (long)i * q) * 4;
  const int src = a.idx ? a.idx[i] : i;
  f4 v = ld4(J.src + (long)src * J.H + j);
  if (a.reset != nullptr && a.reset[i]) v = f4{0.f, 0.f, 0.f, 0.f};
  st4(J.dst + (long)i * J.H + j, v);
  if (J.dst2 != nullptr) st4(J.dst2 + (long)i * J.H + j, v);
}

__global__ __launch_bounds__(256) void row_gather_kernel(const RowGatherArgs a) {
  row_gather(a, a.job[blockIdx.y], (long)blockIdx.x * 256 + threadIdx.x);
}

__global__ __launch_bounds__(256) void row_split_kernel(const RowSplitArgs a) {
  int part = 0;
  while ((int)blockIdx.x >= a.end[part]) ++part;                  // the last end is the grid's
  const long e = ((long)blockIdx.x - (part ? a.end[part - 1] : 0)) * 256 + threadIdx.x;
  if (part < a.layers.count) {
    fused_pack_unit(a.layers.job[part], (int)e);
    return;
  }
  part -= a.layers.count;
  if (part < a.n_packs) {
    if (a.pack[part].cell == CELL_LSTM) step_pack<CELL_LSTM>(a.pack[part], e);
    else step_pack<CELL_GRU>(a.pack[part], e);
    return;
  }
  row_gather(a.rows, a.rows.job[part - a.n_packs], e);
}

__global__ __launch_bounds__(256) void copy_matrix_kernel(const float* __restrict__ src, int ld_src, int rows, int cols,
                                                          float* __restrict__ dst) {
  const int q = cols >> 2;
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long)rows * q) return;
  const int r = (int)(e / q), c = (int)(e - (long)r * q) * 4;
  st4(dst + (long)r * cols + c, ld4(src + (long)r * ld_src + c));
}

__global__ __launch_bounds__(256) void copy_input_kernel(const float* __restrict__ src, long n, float* __restrict__ dst) {
  const long e = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e + 4 <= n) {
    st4(dst + e, *reinterpret_cast<const f4_any*>(src + e));
  } else {
    for (long i = e; i < n; ++i) dst[i] = src[i];
  }
}

__global__ __launch_bounds__(256) void column_rows_kernel(const int32_t* __restrict__ perm, int E, int M, int T, int N,
                                                          int32_t* __restrict__ rows_out) {
  const long total = (long)E * T * N;
  const long o = (long)blockIdx.x * 256 + threadIdx.x;
  if (o >= total) return;
  const int nb = N / M;
  const int i = (int)(o % nb);
  long r = o / nb;
  const int t = (int)(r % T); r /= T;
  const int m = (int)(r % M);
  const int e = (int)(r / M);
  rows_out[o] = t * N + perm[(long)e * N + (long)m * nb + i];
}

}  // namespace

static dim3 step_grid(int nb, const int* H, int n_nets) {
  int blocks = 0;
  for (int k = 0; k < n_nets; ++k) {
    const int rblocks = ((nb + GS_ROWS - 1) / GS_ROWS + GS_XCDS - 1) / GS_XCDS * GS_XCDS;   // see step_block
    const int b = rblocks * ((H[k] + GS_JB - 1) / GS_JB);
    blocks = b > blocks ? b : blocks;
  }
  return dim3(blocks, n_nets);
}

static hipError_t launch_step_rest(const StepFwdArgs& a, hipStream_t stream) {
  if (a.n_nets <= 0) return hipSuccess;
  const int G = a.cell == CELL_LSTM ? 4 : 3;
  int H[2] = {a.net[0].H, a.net[1].H};
  double flops = 0.0;
  for (int k = 0; k < a.n_nets; ++k) flops += 2.0 * a.nb * H[k] * (double)G * H[k];
  TraceScope ts(stream, a.cell == CELL_LSTM ? "lstm_step_fwd" : "gru_step_fwd", flops, 0.0);
  const dim3 grid = step_grid(a.nb, H, a.n_nets);
  if (a.cell == CELL_LSTM) hipLaunchKernelGGL(step_fwd_kernel<CELL_LSTM>, grid, dim3(GS_THREADS), 0, stream, a);
  else hipLaunchKernelGGL(step_fwd_kernel<CELL_GRU>, grid, dim3(GS_THREADS), 0, stream, a);
  return hipGetLastError();
}

// Which steps take that kernel: those of act() and rslx_memory_step (nothing kept for a backward pass, no flags), from the sizes on where
// an earlier form, which split the weights in every workgroup and left the input side out, was the faster one for a memory by itself.
// The present form leads on both sides of these lines, so they lie too high, not too low; they stay where their tests have them.
// The fp32 step's time over this one's, every size run through both, rslx_memory_step / act() with two such memories in front of
// [256, 128], 48 inputs:
//   GRU of 256   below the line 1.12 / 1.04 at 512 rows, 1.14 / 1.18 at 1024;  above 1.42 at 1100, 1.45 / 1.31 at 2048
//   GRU of 128                  1.28 / 1.11 at 1024, 1.28 / 1.21 at 2048;  1.53 at 2887, 1.52 / 1.33 at 4096
//   GRU of 512                  0.95 / 1.16 at 512;  1.20 / 1.31 at 1024, 1.61 at 1443
//   LSTM of 256                 0.99 / 1.01 at 512, 1.04 / 1.12 at 1024, 1.32 at 1443;  1.31 / 1.35 at 2048
//   LSTM of 128                 1.12 / 1.06 at 1024, 1.42 / 1.24 at 4096;  1.49 / 1.26 at 8192
//   LSTM of 64                  1.24 / 1.18 at 4096, 1.47 / 1.12 at 16 384;  1.38 / 1.15 at 32 768
// With more inputs than step_takes_input allows, where the product stays apart, the lines are the present form's as well: 600 inputs, GRU
// of 64 0.98 at 4096 rows and 1.04 at 8192, LSTM of 64 0.96 at 8192 and 1.0 from 16 384 on.  A memory's own sizes decide, so that a
// call for the values alone returns the bits of a full one; only rslx_memory_step, which has no such counterpart, may draw its line later.
bool step_split_sizes(int32_t cell, int32_t H, int32_t nb, bool alone) {
  if (H % 64 != 0 || H > 8192 || nb < 1024) return false;
  const int64_t size = (int64_t)nb * H;
  return cell == CELL_LSTM ? size >= (H < 128 ? 1 << 21 : alone && H < 256 ? 3 << 18 : 1 << 19) : size > 1 << 18;
}

// Its line: act() with the input side in a product of its own and weights split by every workgroup, and here, memories in front of
// [256, 128], us: GRU of 256 at 4096 rows 73.2 and 65.5 with 48 inputs, 91.8 and 79.1 with 235, 108 and 95.6 with 512, at 1200 rows
// 54.7 and 47.9, 62.6 and 55.2, 67.9 and 62.7; GRU of 512 at 1024 rows with 1000 116 and 102; LSTM of 256 at 4096 rows 85.0 and
// 74.5, 109 and 89.9, 130 and 112; of 128 at 8192 rows with 48 88.2 and 78.1, with 256 109 and 93.1.
bool step_takes_input(int32_t H, int32_t D) { return D <= 2 * H; }

size_t step_pack_bytes(int32_t cell, int32_t H, int32_t D) {
  if (!step_comes_split(cell, D > 0)) return 0;
  const size_t units = H / ST_UNITS;
  return cell == CELL_LSTM ? units * step_chunks<CELL_LSTM>(H, D) * StepSplit<CELL_LSTM>::CHUNK : units * step_chunks<CELL_GRU>(H, D) * StepSplit<CELL_GRU>::CHUNK;
}

hipError_t launch_step_fwd(const StepFwdArgs& a, hipStream_t stream) {
  if (a.nb <= 0 || a.n_nets <= 0) return hipSuccess;
  const bool lstm = a.cell == CELL_LSTM;
  StepFwdArgs b = a;
  if (b.n_nets == 2 && b.net[1].H > b.net[0].H) std::swap(b.net[0], b.net[1]);
  int split = 0;
  double flops = 0.0;
  for (int k = 0; k < b.n_nets; ++k) {
    split |= (b.net[k].split != 0) << k;
    flops += 2.0 * b.nb * (b.net[k].H + (b.net[k].x ? b.net[k].D : 0)) * (lstm ? 4.0 : 3.0) * b.net[k].H;
  }
  if (split == 0) return launch_step_rest(a, stream);
  if (b.n_nets == 2 && (split != 3 || b.net[0].H != b.net[1].H)) {
    int rest_blocks = 0;
    for (int k = 0; k < 2; ++k)
      if (!(split >> k & 1)) rest_blocks = step_grid(b.nb, &b.net[k].H, 1).x;
    TraceScope ts(stream, lstm ? "lstm_uneven" : "gru_uneven", flops, 0.0);
    return lstm ? step_uneven_launch<CELL_LSTM>(b, split, rest_blocks, stream) : step_uneven_launch<CELL_GRU>(b, split, rest_blocks, stream);
  }
  TraceScope ts(stream, lstm ? "lstm_split" : "gru_split", flops, 0.0);
  return lstm ? step_split_launch<CELL_LSTM>(b, stream) : step_split_launch<CELL_GRU>(b, stream);
}

hipError_t launch_step_bwd(const StepBwdArgs& a, hipStream_t stream) {
  if (a.nb <= 0 || a.n_nets <= 0) return hipSuccess;
  const int G = a.cell == CELL_LSTM ? 4 : 3;
  int H[2] = {a.net[0].H, a.net[1].H};
  double flops = 0.0;
  for (int k = 0; k < a.n_nets; ++k) flops += a.net[k].dg_next ? 2.0 * a.nb * H[k] * (double)G * H[k] : 0.0;
  TraceScope ts(stream, a.cell == CELL_LSTM ? "lstm_step_bwd" : "gru_step_bwd", flops, 0.0);
  const dim3 grid = step_grid(a.nb, H, a.n_nets);
  if (a.cell == CELL_LSTM) hipLaunchKernelGGL(step_bwd_kernel<CELL_LSTM>, grid, dim3(GS_THREADS), 0, stream, a);
  else hipLaunchKernelGGL(step_bwd_kernel<CELL_GRU>, grid, dim3(GS_THREADS), 0, stream, a);
  return hipGetLastError();
}

// One step has no recurrence to keep the weights for: an update of T = 1 (two memories of 128 and [64, 12], us a call) takes
// 97 with these kernels and 85 with a launch per step at one minibatch of 16 rows (LSTM; GRU 92 and 84), 428 and 378 at two of 8192 (GRU 382
// and 353).
// T = 2: GRU 103 and 102, 568 and 660; LSTM 108 and 104, 623 and 675.
bool seq_supported(int32_t cell, int32_t H, int32_t T) { return (cell == CELL_GRU || cell == CELL_LSTM) && H == 128 && T >= 2; }

hipError_t launch_seq_fwd(const SeqArgs& a, hipStream_t stream) {
  const double G = a.cell == CELL_LSTM ? 4 : 3;
  TraceScope ts(stream, a.cell == CELL_LSTM ? "lstm_seq_fwd" : "gru_seq_fwd", 2.0 * a.n_nets * a.T * (double)a.nb * G * a.H * a.H, 0.0);
  return seq_dispatch(a, false, stream);
}

hipError_t launch_seq_bwd(const SeqArgs& a, hipStream_t stream) {
  const double G = a.cell == CELL_LSTM ? 4 : 3;
  TraceScope ts(stream, a.cell == CELL_LSTM ? "lstm_seq_bwd" : "gru_seq_bwd", 2.0 * a.n_nets * (a.T - 1) * (double)a.nb * G * a.H * a.H, 0.0);
  return seq_dispatch(a, true, stream);
}

hipError_t launch_row_gather(const RowGatherArgs& a, hipStream_t stream) {
  long work = 0;
  for (int k = 0; k < a.n_jobs; ++k) { const long w = (long)a.nb * (a.job[k].H >> 2); work = w > work ? w : work; }
  if (work == 0) return hipSuccess;
  hipLaunchKernelGGL(row_gather_kernel, dim3((unsigned)((work + 255) / 256), a.n_jobs), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// The parts' blocks follow each other in one dimension, first the splits, whose threads' loads and stores are the longer chain.  Two
// GRUs of 256 in front of [512, 256, 128] at 4096 rows, us a call, in turn on one card: copies first 85.6, splits first 84.5 (runs of one
// side differ by 0.1).
hipError_t launch_row_split(const RowSplitArgs& args, hipStream_t stream) {
  if (args.n_packs == 0 && args.layers.count == 0) return launch_row_gather(args.rows, stream);
  RowSplitArgs a = args;
  int64_t blocks = 0;
  int n = 0;
  auto part = [&](int64_t threads) {
    blocks += (threads + 255) / 256;
    a.end[n++] = (int32_t)std::min<int64_t>(blocks, INT32_MAX);
  };
  for (int k = 0; k < a.layers.count; ++k) part((int64_t)4 * fused_pack_steps(a.layers.job[k].K) * fused_pack_columns(a.layers.job[k].N));
  for (int k = 0; k < a.n_packs; ++k) part((int64_t)step_pack_bytes(a.pack[k].cell, a.pack[k].H, a.pack[k].D) / (3 * 16));
  for (int k = 0; k < a.rows.n_jobs; ++k) part((int64_t)a.rows.nb * (a.rows.job[k].H >> 2));
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(row_split_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_copy_matrix(const float* src, int32_t ld_src, int32_t rows, int32_t cols, float* dst, hipStream_t stream) {
  const long total = (long)rows * (cols >> 2);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(copy_matrix_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, src, ld_src, rows, cols, dst);
  return hipGetLastError();
}

hipError_t launch_copy_input(const float* src, int64_t n, float* dst, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 1023) / 1024;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  TraceScope ts(stream, "copy_input", 0.0, 8.0 * n);
  hipLaunchKernelGGL(copy_input_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, src, (long)n, dst);
  return hipGetLastError();
}

hipError_t launch_column_rows(const int32_t* perm, int32_t E, int32_t M, int32_t T, int32_t N, int32_t* rows_out,
                              hipStream_t stream) {
  const long total = (long)E * T * N;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(column_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, perm, E, M, T, N, rows_out);
  return hipGetLastError();
}

}  // namespace rslx
