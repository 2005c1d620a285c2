// Contraction kernel for gfx950, used by every dense layer of the actor, critic, student, teacher and RND networks:
// forward, input gradient and weight gradient.  Operands, sums and results are fp32; the products run on the bf16
// matrix cores (v_mfma_f32_32x32x16_bf16), sixteen times the rate of the fp32 ones, on operands split in three:
//
//   a = a0 + a1 + a2,   a0 = bf16(a), a1 = bf16(a - a0), a2 = bf16(a - a0 - a1)      (exact: 3 x 8 significant bits)
//   a b ~ a0 b0 + (a0 b1 + a1 b0) + (a1 b1 + a0 b2 + a2 b0)
//
// What is left out (a1 b2, a2 b1, a2 b2) is below 2^-24 of the product, as the rounding of an fp32 product is (largest seen
// over four million random pairs 0.9 of that bound, root mean square 0.09 of it).  Operands are scaled by 2^16, so that
// the split is exact down to the smallest fp32 value (SPLIT_SCALE).  Six products at sixteen times the rate are 2.7 times
// the fp32 peak.  Operands that have no such split (infinite, or 2^111 and above) make their outputs non-finite; a
// wavefront that finds non-finite sums forms those on the fp32 matrix cores (fp32_repeat), so the results of such inputs
// are those of fp32 arithmetic and all others what they are without them.
//
// Tiling: one workgroup = 4 wavefronts (256 lanes) computes a BM x BN block of C in steps of 16 contraction indices.
// The operand tile of step k + 1 is split in registers and written to LDS, and the fp32 values of step k + 2 are
// requested, while step k feeds the matrix cores (LDS double buffer).  An LDS plane holds one of the three parts of
// eight consecutive contraction indices of all tile rows, 16 bytes a row: a lane's matrix operand is one 16-byte
// read, and 32 lanes read 512 contiguous bytes.
//
// MFMA 32x32x16 bf16 register layout (wave64, lane l, g = l / 32, j = l % 32):
//   A operand: A[row = j][k = 8 g .. 8 g + 7]      B operand: B[k = 8 g .. 8 g + 7][col = j]
//   D/C, 16 accumulators r = 0..15:   D[row = 8 * (r / 4) + 4 * g + r % 4][col = j]
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "kernels.h"
#include "split_bf16.h"

namespace rslx {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NT = 256;   // lanes per workgroup
constexpr int BK = 16;    // contraction indices per step

__device__ __forceinline__ int wrap_row(const GemmProblem& P, int r) { return r >= P.idx_mod ? r - P.idx_mod : r; }

__device__ __forceinline__ int src_row(const GemmProblem& P, int r) {
  int rr = wrap_row(P, r);
  const int v = P.row_idx ? P.row_idx[rr] : rr;
  return r >= P.idx_mod ? v + P.wrap_add : v;
}

// LDS image of one operand tile of R rows: plane (part s, k-group kg) at (2 s + kg) * pitch, 16 bytes per row.  The 64
// bytes between planes put the two k-groups of a row in different banks when they are written together.
template <int R> constexpr int plane_pitch() { return R * 16 + 64; }
template <int R> constexpr int tile_bytes() { return 6 * plane_pitch<R>(); }

// The parts of four values of consecutive contraction indices 4 q .. 4 q + 3 of one tile row, and their LDS writes.
struct Quad {
  uint2 part[3];
  __device__ __forceinline__ void split_lo(const float* v) { split_pair(v[0], v[1], part[0].x, part[1].x, part[2].x); }
  __device__ __forceinline__ void split_hi(const float* v) { split_pair(v[2], v[3], part[0].y, part[1].y, part[2].y); }
  template <int R>
  __device__ __forceinline__ void put(char* tile, int row, int q) const {
    char* d = tile + (q >> 1) * plane_pitch<R>() + row * 16 + (q & 1) * 8;
#pragma unroll
    for (int s = 0; s < 3; ++s) *reinterpret_cast<uint2*>(d + 2 * s * plane_pitch<R>()) = part[s];
  }
};

// How an operand is read.  FORM_FAST: 16-byte loads of rows that are contiguous along the contraction, by 32-bit offsets
// (from the tile's first row; gathered rows from the matrix, which must be smaller than 4 GiB); plain rows where the
// M / N index is contiguous.  FORM_GATHER (weight gradient): its contraction rows are gathered.  FORM_FAR (forward): as
// FORM_FAST with gathered rows of a larger matrix.  FORM_GENERAL: any alignment, gather and column map.
enum Form { FORM_FAST, FORM_GATHER, FORM_FAR, FORM_GENERAL };

// ---- operand with the contraction index contiguous in memory (rows of X or dZ) ------------------------------
// Lane -> row tid / 4 (+ 64 per pass), contraction indices 4 (tid % 4) .. + 3: four lanes read the 64 bytes of a row's
// step.  Everything that does not change along the contraction (row offsets with the gather applied) is set up once
// per tile.  Rows past the end repeat the last one; the outputs they feed are dropped.
template <int R, bool IS_X, int FORM>
struct KContig {
  static constexpr int NP = R >= 64 ? R / 64 : 1;
  static constexpr int NREG = 4 * NP;
  static constexpr bool VEC = FORM == FORM_FAST;
  const float* base;
  const float* ptr[VEC ? 1 : NP];
  uint32_t off[VEC ? NP : 1];   // bytes from `base`
  uint32_t mapped;              // bit p: the row of pass p reads through col_map / col_sign (FORM_GENERAL)
  int q;

  __device__ __forceinline__ void setup(const GemmProblem& P, const float* b, int ld, int row0, int row_end) {
    const int first = IS_X && P.row_idx != nullptr ? 0 : row0;
    base = b + (long)first * ld;
    q = threadIdx.x & 3;
    mapped = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int row = min(row0 + p * 64 + (int)(threadIdx.x >> 2), row_end - 1);
      const int sr = IS_X ? src_row(P, row) : row;
      if constexpr (VEC) {
        off[p] = 4u * ((uint32_t)(sr - first) * (uint32_t)ld);
      } else {
        ptr[p] = b + (long)sr * ld;
        if (IS_X && P.col_map != nullptr && row >= P.map_from) mapped |= 1u << p;
      }
    }
  }
  // One pass of the fetch of step k0.  Past k_end the last values are read again: in bounds, and nullified by a zero in
  // one of the two operands.
  __device__ __forceinline__ void fetch(const GemmProblem& P, int k0, int k_end, float (&reg)[NREG], int p) {
    if constexpr (VEC) {
      const uint32_t kb = 4u * (uint32_t)min(k0 + 4 * q, k_end - 4);
      const float4 v = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base) + (off[p] + kb));
      reg[4 * p + 0] = v.x; reg[4 * p + 1] = v.y; reg[4 * p + 2] = v.z; reg[4 * p + 3] = v.w;
    } else if constexpr (FORM == FORM_FAR) {
      const float4 v = *reinterpret_cast<const float4*>(ptr[p] + min(k0 + 4 * q, k_end - 4));
      reg[4 * p + 0] = v.x; reg[4 * p + 1] = v.y; reg[4 * p + 2] = v.z; reg[4 * p + 3] = v.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int col = min(k0 + 4 * q + c, k_end - 1);
        float v;
        if (IS_X && ((mapped >> p) & 1u)) v = (P.col_sign != nullptr ? P.col_sign[col] : 1.0f) * ptr[p][P.col_map[col]];
        else v = ptr[p][col];
        reg[4 * p + c] = v;
      }
    }
  }
  __device__ __forceinline__ bool valid(int k0, int k_end, int c) const { return k0 + 4 * q + c < k_end; }
  __device__ __forceinline__ void put(char* tile, const Quad& quad, int p) const {
    const int row = p * 64 + (int)(threadIdx.x >> 2);
    if (R >= 64 || row < R) quad.template put<R>(tile, row, q);
  }
};

// ---- operand with the M / N index contiguous in memory (contraction index = memory row) ---------------------
// Wavefront w takes the contraction indices 4 w .. 4 w + 3 of a step, its lanes 64 consecutive columns (+ 64 per pass):
// the memory rows are uniform, every load is a scalar row address plus the lane's column, of any alignment, and a
// lane ends up with consecutive contraction indices of one column, which is what the split parts are packed along.
template <int Cw, int FORM>
struct Direct {
  static constexpr int NP = Cw >= 64 ? Cw / 64 : 1;
  static constexpr int NREG = 4 * NP;
  static constexpr bool MAPPED = FORM == FORM_GENERAL;
  const float* base;
  int ld, w;
  uint32_t col[NP], cm[MAPPED ? NP : 1];        // byte offsets of the lane's columns in a row
  float sg[MAPPED ? NP : 1];
  const int32_t* row_idx;
  int idx_mod, wrap_add, map_from;
  int next_row;                                 // lane c % 4: source row c of the next fetch, looked up one step ahead of it

  __device__ __forceinline__ void setup(const GemmProblem& P, const float* b, int ld_, int col0, int col_end) {
    base = b; ld = ld_;
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    row_idx = P.row_idx; idx_mod = P.idx_mod; wrap_add = P.wrap_add; map_from = P.map_from;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int c = min(col0 + p * 64 + (int)(threadIdx.x & 63), col_end - 1);   // columns past the end repeat the last one
      col[p] = 4u * (uint32_t)c;
      if constexpr (MAPPED) {
        cm[p] = col[p]; sg[p] = 1.0f;
        if (P.col_map != nullptr) {
          cm[p] = 4u * (uint32_t)P.col_map[c];
          if (P.col_sign != nullptr) sg[p] = P.col_sign[c];
        }
      }
    }
  }
  __device__ __forceinline__ void look_up(int k0, int k_end) {
    if constexpr (FORM != FORM_FAST) {
      const int r = min(k0 + 4 * w + (int)(threadIdx.x & 3), k_end - 1);
      const bool wrap = r >= idx_mod;
      const int rr = wrap ? r - idx_mod : r;
      next_row = (row_idx != nullptr ? row_idx[rr] : rr) + (wrap ? wrap_add : 0);
    }
  }
  __device__ __forceinline__ void fetch(const GemmProblem&, int k0, int k_end, float (&reg)[NREG], int p) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int kk = min(k0 + 4 * w + c, k_end - 1);   // uniform
      const int row = FORM == FORM_FAST ? kk : __builtin_amdgcn_readlane(next_row, c);
      const char* rowp = reinterpret_cast<const char*>(base + (long)row * ld);
      if (MAPPED && kk >= map_from) reg[4 * p + c] = sg[MAPPED ? p : 0] * *reinterpret_cast<const float*>(rowp + cm[MAPPED ? p : 0]);
      else reg[4 * p + c] = *reinterpret_cast<const float*>(rowp + col[p]);
    }
  }
  __device__ __forceinline__ bool valid(int k0, int k_end, int c) const { return k0 + 4 * w + c < k_end; }
  __device__ __forceinline__ void put(char* tile, const Quad& quad, int p) const {
    const int lane = threadIdx.x & 63;
    if (Cw >= 64 || lane < Cw) quad.template put<Cw>(tile, p * 64 + lane, w);
  }
};

// ---- weights that were split once for the optimiser step (launch_pack_weights) -------------------------------
// Memory holds the LDS image already, step by step: 16 bytes are one part of eight consecutive contraction indices of one
// column, the contraction padded with zeros to whole steps.  Loads and LDS writes only.  A step's six planes lie together,
// so that a lane's place in them fits 32 bits (96 bytes per column) whatever the length of the contraction.
template <int Cw>
struct Packed {
  static constexpr int UNITS = 6 * Cw;                      // 16-byte units of a step
  static constexpr int NP = (UNITS + NT - 1) / NT;
  static constexpr int NREG = 4 * NP;
  const char* base;
  uint32_t off[NP], step;                                   // bytes: the lane's units within a step, a whole step
  __device__ __forceinline__ void setup(const GemmProblem& P, int col0, int col_end) {
    base = reinterpret_cast<const char*>(P.Bp);
    step = 96u * (uint32_t)P.N;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int u = min(p * NT + (int)threadIdx.x, UNITS - 1);
      off[p] = 16u * (uint32_t)(u / Cw * P.N + min(col0 + u % Cw, col_end - 1));   // plane u / Cw: 2 * part + k-group
    }
  }
  __device__ __forceinline__ void fetch(const GemmProblem&, int k0, int, float (&reg)[NREG], int p) {
    const char* b = base + (long)(k0 / BK) * step;          // uniform
    uint32_t o = off[p];
    asm volatile("" : "+v"(o));                             // a 32-bit offset beside the uniform base, not a 64-bit sum kept over the loop
    const float4 v = *reinterpret_cast<const float4*>(b + o);
    reg[4 * p + 0] = v.x; reg[4 * p + 1] = v.y; reg[4 * p + 2] = v.z; reg[4 * p + 3] = v.w;
  }
  __device__ __forceinline__ void put_raw(char* tile, const float* v, int p) const {
    const int u = p * NT + (int)threadIdx.x;
    if (NP * NT == UNITS || u < UNITS)
      *reinterpret_cast<float4*>(tile + (u / Cw) * plane_pitch<Cw>() + (u % Cw) * 16) = make_float4(v[0], v[1], v[2], v[3]);
  }
};

// LDS bytes of one tile configuration: two buffers of split operand tiles.
template <int BM, int BN>
constexpr int gemm_lds_bytes() { return 2 * (tile_bytes<BM>() + tile_bytes<BN>()); }

// Puts the sums of fp32 products (v_mfma_f32_32x32x2_f32, operands element by element from memory) in place of the
// non-finite ones among a wavefront's accumulators; `blocks` holds a bit per 32 x 32 block that has any.  The other sums
// stay, so that a row's result does not depend on what else is in its tile.
template <int MODE, int WN, int TM, int TN>
__device__ __forceinline__ void fp32_repeat(const GemmProblem& P, int tid, int m0, int n0, int k_begin, int k_end, uint32_t blocks,
                                            f32x16 (&acc)[TM][TN]) {
  constexpr int AHEAD = 4;             // products whose operands are requested together
  const int g = (tid >> 5) & 1, j = tid & 31, wave = tid >> 6;
  const int row0 = m0 + wave / WN * (TM * 32), col0 = n0 + wave % WN * (TN * 32);
  const int a_cols = (MODE == GEMM_DW && P.a_cols > P.M) ? P.a_cols : P.M;
#pragma unroll
  for (int b = 0; b < TM * TN; ++b) {
    if (!((blocks >> b) & 1u)) continue;
    const int m = row0 + b / TN * 32 + j, n = col0 + b % TN * 32 + j;
    const bool m_ok = m < (MODE == GEMM_DW ? a_cols : P.M), n_ok = n < P.N;
    const float* arow = P.A;                                    // operand A's row, where it is one along the contraction
    if (m_ok && MODE != GEMM_DW) arow += (long)(MODE == GEMM_FWD ? src_row(P, m) : m) * P.lda;
    f32x16 c;
#pragma unroll
    for (int r = 0; r < 16; ++r) c[r] = 0.f;
#pragma unroll 1
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * AHEAD) {
      float a[AHEAD], w[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        const int k = k0 + 2 * i + g;
        a[i] = w[i] = 0.f;
        if (k >= k_end) continue;
        if (n_ok) w[i] = P.B[MODE == GEMM_DX ? (long)n * P.ldb + k : (long)k * P.ldb + n];
        if (!m_ok) continue;
        const float* rp = MODE == GEMM_DW ? P.A + (long)src_row(P, k) * P.lda : arow;
        const int col = MODE == GEMM_DW ? m : k;
        const bool mapped = MODE != GEMM_DX && P.col_map != nullptr && (MODE == GEMM_DW ? k : m) >= P.map_from;
        a[i] = mapped ? (P.col_sign != nullptr ? P.col_sign[col] : 1.0f) * rp[P.col_map[col]] : rp[col];
      }
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], w[i], c, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!__builtin_isfinite(acc[b / TN][b % TN][r])) acc[b / TN][b % TN][r] = c[r];
  }
}

// One output tile (one split of it for the weight gradient) of problem P.  `lin` numbers the workgroups of the
// problem's grid of gx tiles x (total / gx) splits; `smem` holds gemm_lds_bytes<BM, BN>() bytes.
template <int MODE, int BM, int BN, int WM, int WN, int FORM, bool PACK>
__device__ __forceinline__ void gemm_tile(const GemmProblem& P, int lin, const int total, const int gx, char* smem) {
  static_assert(WM * WN == 4, "four wavefronts per workgroup");
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  static_assert(TM >= 1 && TN >= 1, "wave tile must hold at least one 32x32 block");
  constexpr int ABYTES = tile_bytes<BM>(), BBYTES = tile_bytes<BN>();
  char* As = smem;                          // [2][ABYTES]
  char* Bs = smem + 2 * ABYTES;             // [2][BBYTES]

  const int tiles_n = (P.N + BN - 1) / BN;
  const int tiles_m = (P.M + BM - 1) / BM;
  // Workgroups are handed to the 8 XCDs round-robin by linear id; remap so that neighbours in (tile, split)
  // order - which share operand rows - run on the same XCD and meet in its L2.
  if ((total & 7) == 0) lin = (lin & 7) * (total >> 3) + (lin >> 3);
  const int tile = lin % gx;
  if (tile >= tiles_m * tiles_n) return;
  const int split = lin / gx;
  if (MODE == GEMM_DW && split >= P.n_split) return;
  const int tn = tile % tiles_n, tm = tile / tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int k_begin = (MODE == GEMM_DW) ? split * P.k_chunk : 0;
  const int k_end = (MODE == GEMM_DW) ? min(P.K, k_begin + P.k_chunk) : P.K;
  const int nk = (k_end - k_begin + BK - 1) / BK;

  int tid = threadIdx.x;
  int lane = tid & 63, wave = tid >> 6;
  int g = lane >> 5, j = lane & 31;
  int wm = wave / WN, wn = wave % WN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  // operand A: DW reads X rows as contraction rows (M index contiguous); FWD / DX read rows with k contiguous.
  // operand B: split weights (FWD, DX), else rows with the N index contiguous (FWD: W, DW: dZ).
  const int a_cols = (MODE == GEMM_DW && P.a_cols > P.M) ? P.a_cols : P.M;   // DW: readable (zero-padded) width of X
  typename std::conditional<MODE == GEMM_DW, Direct<BM, FORM>, KContig<BM, MODE == GEMM_FWD, FORM>>::type la;
  static_assert(PACK || MODE != GEMM_DX, "input gradients have split weights");
  typename std::conditional<PACK, Packed<BN>, Direct<BN, FORM_FAST>>::type lb;
  la.setup(P, P.A, P.lda, m0, a_cols);
  if constexpr (PACK) lb.setup(P, n0, P.N);
  else lb.setup(P, P.B, P.ldb, n0, P.N);
  // values on their way to LDS: one step ahead; activation rows that meet weights two steps ahead, since they come from
  // memory, where the loads' own addresses leave registers for them (general rows, packed weights, 128 x 128: 22 registers
  // spilled at two steps; update with [301, 150, 75] at 24 576 rows 9.30 ms at two, 8.61 at one, 8.99 without the packed weights)
  constexpr int DA = MODE != GEMM_DW && FORM == FORM_FAST ? 2 : 1;
  float ra[DA][decltype(la)::NREG], rb[decltype(lb)::NREG];

  // DW: column sums of dZ for the bias gradient, over the contraction rows of this lane
  constexpr int NBS = MODE == GEMM_DW ? decltype(lb)::NP : 1;
  float bsum[NBS];
#pragma unroll
  for (int p = 0; p < NBS; ++p) bsum[p] = 0.f;
  // Odd result rows are computed negated (see split_scale), the weight gradient's by turns from split to split.  A lane
  // splits rows of one parity: tile rows tid / 4 + 64 p, the weight gradient's tid % 64 + 64 p.
  const int turn = MODE == GEMM_DW ? split & 1 : 0;
  const float a_scale = split_scale(MODE == GEMM_DW ? tid + turn : tid >> 2);
  const bool with_bias = MODE == GEMM_DW && tm == 0 && P.bias_off >= 0;

  const bool full_mn = m0 + BM <= P.M && n0 + BN <= P.N;

  // The loop is a fixed sequence of slots, one matrix instruction each, with the other work dealt out between them: a
  // wave that converts, loads or stores in one burst leaves its matrix cores idle meanwhile, and the other waves of the
  // SIMD tend to be in the same phase.  Body t runs the last three products of step t - 1 and the first three of step
  // t, so the operands of step t replace those of step t - 1 in their registers as these are used up, and the parts
  // of step t + 1 have the whole body to be formed and written; one barrier per body.
  // Two bodies to a round of the loop, so that the two places of the values on their way, and of the LDS buffers, are known at
  // compile time: with one body the compiler moved the later values over at its end and waited there for loads of the same
  // body, and 22 more vector instructions a step were moves and addresses.  Whole updates, us, in turn on one card: 4096
  // environments, [512, 256, 128] 8641 -> 8499, [256, 256, 128] by regression 1561 -> 1523 (on another card no gain: 1626 and 1630);
  // 16 384 environments with the curiosity networks 46 212 -> 45 221.
  // Steps past the end: the last body forms the parts of one step too many (nobody reads them), and where the range is
  // no whole number of steps, the indices past its end meet a zero in one operand: the zero padding of packed weights, else
  // zeros put in place of operand B's (weight gradient) or A's values.
  constexpr int NA = decltype(la)::NP, NB = decltype(lb)::NP, NQ = NA + NB, TT = TM * TN;
  {
    using EVEN = std::integral_constant<int, 0>;
    using ODD = std::integral_constant<int, 1>;
    bf16x8 a[3][TM], b[3][TN];
    Quad quad;
    // piece p of step kt: a pass of operand A (p < NA) or B; `par` = kt mod 2, known at compile time
    auto fetch_piece = [&](int p, int kt, int slot) {
      const int k0 = k_begin + min(kt, nk - 1) * BK;
      if (p < NA) {
        la.fetch(P, k0, k_end, ra[slot], p < NA ? p : 0);
        if constexpr (MODE == GEMM_DW) {
          if (p == NA - 1) la.look_up(k_begin + min(kt + 1, nk - 1) * BK, k_end);
        }
      } else {
        lb.fetch(P, k0, k_end, rb, p < NA ? 0 : p - NA);
      }
    };
    auto split_piece = [&](int p, int kt, int half, int slot) {
      if (PACK && p >= NA) return;
      float* v = p < NA ? ra[slot] + 4 * (p < NA ? p : 0) : rb + 4 * (p < NA ? 0 : p - NA);
      if constexpr (!PACK) {
        if ((MODE == GEMM_DW) == (p >= NA)) {
          const int k0 = k_begin + kt * BK;
#pragma unroll
          for (int c = 2 * half; c < 2 * half + 2; ++c) v[c] = (MODE == GEMM_DW ? lb.valid(k0, k_end, c) : la.valid(k0, k_end, c)) ? v[c] : 0.f;
        }
      }
      const float s = p < NA ? a_scale : SPLIT_SCALE;
      const float w[4] = {s * v[0], s * v[1], s * v[2], s * v[3]};
      if (half == 0) quad.split_lo(w);
      else quad.split_hi(w);
    };
    auto put_piece = [&](int p, int par) {
      if (p < NA) {
        la.put(As + par * ABYTES, quad, p);
      } else {
        const float* v = rb + 4 * (p < NA ? 0 : p - NA);
        if constexpr (PACK) lb.put_raw(Bs + par * BBYTES, v, p - NA);
        else lb.put(Bs + par * BBYTES, quad, p - NA);
        if constexpr (MODE == GEMM_DW) bsum[p < NA ? 0 : p - NA] += (v[0] + v[1]) + (v[2] + v[3]);
      }
    };
    auto body = [&](int t, auto par_tag, auto g2_tag) {
      constexpr bool G2 = decltype(g2_tag)::value;
      constexpr int par = decltype(par_tag)::value, next = DA == 2 ? par ^ 1 : 0;
      constexpr int S = (G2 ? 6 : 3) * TT;
      constexpr int PA[6] = {0, 1, 0, 1, 0, 2}, PB[6] = {1, 0, 0, 1, 2, 0};   // the parts that meet: step t - 1, then step t
      const char* ab = As + par * ABYTES + g * plane_pitch<BM>() + (wm * (TM * 32) + j) * 16;
      const char* bb = Bs + par * BBYTES + g * plane_pitch<BN>() + (wn * (TN * 32) + j) * 16;
      auto read_a = [&](int s) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[s][i] = *reinterpret_cast<const bf16x8*>(ab + 2 * s * plane_pitch<BM>() + i * 512);
      };
      auto read_b = [&](int s) {
#pragma unroll
        for (int i = 0; i < TN; ++i) b[s][i] = *reinterpret_cast<const bf16x8*>(bb + 2 * s * plane_pitch<BN>() + i * 512);
      };
      if (!G2) { read_a(1); read_b(1); read_b(0); read_a(0); }
      read_a(2); read_b(2);
#pragma unroll
      for (int i = 0; i < S; ++i) {
        const int q = i / TT + (G2 ? 0 : 3), x = i % TT / TN, y = i % TN;
        if (G2 && i == 2 * TT) { read_a(1); read_b(1); }
        if (G2 && i == 3 * TT) { read_b(0); read_a(0); }
        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[q]][x], b[PB[q]][y], acc[x][y], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
          if (i == 3 * p * S / (3 * NQ)) split_piece(p, t + 1, 0, next);
          if (i == (3 * p + 1) * S / (3 * NQ)) split_piece(p, t + 1, 1, next);
          if (i == (3 * p + 2) * S / (3 * NQ)) {
            put_piece(p, par ^ 1);
            fetch_piece(p, t + 1 + (p < NA ? DA : 1), next);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    };
    if constexpr (MODE == GEMM_DW) la.look_up(k_begin, k_end);
#pragma unroll
    for (int p = 0; p < NQ; ++p) fetch_piece(p, 0, 0);
    if (DA == 2) {
#pragma unroll
      for (int p = 0; p < NA; ++p) fetch_piece(p, 1, DA - 1);
    }
#pragma unroll
    for (int p = 0; p < NQ; ++p) {
      split_piece(p, 0, 0, 0); split_piece(p, 0, 1, 0);
      put_piece(p, 0);
      fetch_piece(p, p < NA ? DA : 1, 0);
    }
    __syncthreads();
    body(0, EVEN{}, std::false_type{});
    int t = 1;
    for (; t + 1 < nk; t += 2) {
      body(t, ODD{}, std::true_type{});
      body(t + 1, EVEN{}, std::true_type{});
    }
    if (t < nk) body(t, ODD{}, std::true_type{});
#pragma unroll
    for (int i = 0; i < 3 * TT; ++i) {
      constexpr int PA[3] = {0, 1, 0}, PB[3] = {1, 0, 0};
      const int q = i / TT, x = i % TT / TN, y = i % TN;
      acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[q]][x], b[PB[q]][y], acc[x][y], 0, 0, 0);
    }
  }
  // What follows is formed anew from an opaque lane number: addresses for it would otherwise be computed before the loop
  // and take registers from it.
  asm volatile("" : "+v"(tid));
  lane = tid & 63; wave = tid >> 6;
  g = lane >> 5; j = lane & 31;
  wm = wave / WN; wn = wave % WN;
  {
    uint32_t blocks = 0;           // those with non-finite sums
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int y = 0; y < TN; ++y) {
        float z = 0.f;             // becomes NaN with any
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[x][y][r] *= split_unscale(r + turn);           // register r holds a row of r's parity
          z = fmaf(acc[x][y][r], 0.f, z);
        }
        if (__any(!(z == 0.f))) blocks |= 1u << (x * TN + y);
      }
    if (blocks) fp32_repeat<MODE, WN>(P, tid, m0, n0, k_begin, k_end, blocks, acc);
  }
  float bias_grad = 0.f;
  if (with_bias) {                 // the four wavefronts hold different contraction rows of the same columns
    float* red = reinterpret_cast<float*>(smem);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NBS; ++p)
      if (BN >= 64 || lane < BN) red[wave * BN + p * 64 + lane] = bsum[p];
    __syncthreads();
    if (tid < BN) bias_grad = (red[tid] + red[BN + tid]) + (red[2 * BN + tid] + red[3 * BN + tid]);
  }

  // ---- epilogue -------------------------------------------------------------------------------
  // Problem fields are copied to registers first: read through the reference they would be fetched again after
  // every store, since a store may alias them as far as the compiler can tell.
  const int Mr = P.M, Nc = P.N, ldc = P.ldc;
  const bool elu = P.elu != 0;
  const float alpha = P.alpha;
  const float* aux = P.aux;
  const int bias_off = P.bias_off;
  float* Cb = P.C;
  if (MODE == GEMM_DW) Cb += (long)split * P.split_stride;
  // Tiles inside the matrix.  Loads issued after a block's stores would have to wait for those stores as well (one
  // counter covers both), so everything a block reads is requested before the previous block's stores: the biases
  // of all blocks up front, the activation values that gate the input gradient one block ahead.
  if (full_mn) {
    float bias[TN];
#pragma unroll
    for (int y = 0; y < TN; ++y) bias[y] = (MODE == GEMM_FWD && aux != nullptr) ? aux[n0 + wn * (TN * 32) + y * 32 + j] : 0.f;
    constexpr bool GATE_PIPE = MODE == GEMM_DX;
    float hx[2][16];
    auto block_offset = [&](int b) {
      const int x = b / TN, y = b % TN;
      // register r of a 32x32 block sits 8 * (r / 4) + r % 4 rows below its first row: a uniform offset
      return (long)(m0 + wm * (TM * 32) + x * 32 + 4 * g) * ldc + (n0 + wn * (TN * 32) + y * 32 + j);
    };
    auto load_gate = [&](int b, float (&h)[16]) {
      const float* hp = aux + block_offset(b);
#pragma unroll
      for (int r = 0; r < 16; ++r) h[r] = hp[(8 * (r / 4) + (r % 4)) * ldc];
    };
    if (GATE_PIPE && aux != nullptr) load_gate(0, hx[0]);
#pragma unroll
    for (int b = 0; b < TM * TN; ++b) {
      const int x = b / TN, y = b % TN;
      float* cp = Cb + block_offset(b);
      if (GATE_PIPE && aux != nullptr && b + 1 < TM * TN) load_gate(b + 1, hx[(b + 1) & 1]);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v = acc[x][y][r];
        if (MODE == GEMM_FWD) {
          v += bias[y];
          if (elu) {
            const float e = alpha * (__expf(v) - 1.0f);
            v = v > 0.f ? v : e;
          }
        } else if (MODE == GEMM_DX) {
          if (aux != nullptr) v *= (hx[b & 1][r] > 0.f) ? 1.0f : (hx[b & 1][r] + alpha);
        }
        cp[(8 * (r / 4) + (r % 4)) * ldc] = v;
      }
    }
    if (with_bias && tid < BN && n0 + tid < Nc) Cb[bias_off + n0 + tid] = bias_grad;
    return;
  }
#pragma unroll
  for (int x = 0; x < TM; ++x) {
#pragma unroll
    for (int y = 0; y < TN; ++y) {
      const int col = n0 + wn * (TN * 32) + y * 32 + j;
      const int row_base = m0 + wm * (TM * 32) + x * 32 + 4 * g;
      // Edge tiles: what a block reads is read through clamped indices and turned into the block's 16 results before
      // the first conditional store, so that no store has to wait behind a load (or behind the store before it).
      const int colc = min(col, Nc - 1);
      float bias = 0.f;
      if (MODE == GEMM_FWD && aux != nullptr) bias = aux[colc];
      float out[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v = acc[x][y][r];
        if (MODE == GEMM_FWD) {
          v += bias;
          if (elu) {
            const float e = alpha * (__expf(v) - 1.0f);
            v = v > 0.f ? v : e;
          }
        } else if (MODE == GEMM_DX) {
          if (aux != nullptr) {
            const int rowc = min(row_base + 8 * (r / 4) + (r % 4), Mr - 1);
            const float h = aux[(long)rowc * ldc + colc];
            v *= (h > 0.f) ? 1.0f : (h + alpha);
          }
        }
        out[r] = v;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(out[r]));   // the results exist before the branches below
      if (col >= Nc) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = row_base + 8 * (r / 4) + (r % 4);
        if (row < Mr) Cb[(long)row * ldc + col] = out[r];
      }
    }
  }
  if (with_bias && tid < BN && n0 + tid < Nc) Cb[bias_off + n0 + tid] = bias_grad;
}

// Workgroups resident per CU: three of 128 x 128 (50 KB of LDS, up to 168 registers), four of the smaller tiles.
template <int BM, int BN> constexpr int waves_per_simd() { return BM * BN >= 128 * 128 ? 3 : 4; }

template <int MODE, int BM, int BN, int WM, int WN, int FORM, bool PACK>
__global__ __launch_bounds__(NT, (waves_per_simd<BM, BN>())) void gemm_kernel(const GemmBatch batch) {
  __shared__ __align__(16) char smem[gemm_lds_bytes<BM, BN>()];
  gemm_tile<MODE, BM, BN, WM, WN, FORM, PACK>(batch.p[blockIdx.z], blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y,
                                       gridDim.x, smem);
}

// Weight gradient and input gradient of one layer in one launch (both read the same dZ and neither reads the
// other's result): the workgroups of the second fill the CUs as those of the first drain, so one launch tail and
// one output phase disappear.  Workgroups [0, nw) belong to the weight gradient (gw tiles x sw splits per
// problem), the next ne to an optional second weight gradient of narrow output (the network's output layer, whose
// operands are ready at the same time: 128 x 32 tiles, ge tiles x se splits per problem), the rest to the input
// gradient (gx tiles per problem, 16-byte operand paths only).
template <int WBM, int WBN, int WWM, int WWN, int XBM, int XBN, int XWM, int XWN>
__global__ __launch_bounds__(NT, (waves_per_simd<(WBM > XBM ? WBM : XBM), WBN>())) void gemm_pair_kernel(
    const GemmBatch bw, const GemmBatch bx, const GemmBatch be, const int gw, const int sw, const int gx, const int ge,
    const int se) {
  constexpr int LW = gemm_lds_bytes<WBM, WBN>(), LX = gemm_lds_bytes<XBM, XBN>();
  constexpr int LE = gemm_lds_bytes<128, 32>();
  constexpr int LWX = LW > LX ? LW : LX;
  __shared__ __align__(16) char smem[LWX > LE ? LWX : LE];
  const int per_w = gw * sw, per_e = ge * se;
  const int nw = bw.count * per_w, ne = be.count * per_e;
  const int b = blockIdx.x;
  if (b < nw) {
    const int z = b / per_w;
    gemm_tile<GEMM_DW, WBM, WBN, WWM, WWN, FORM_FAST, false>(bw.p[z], b - z * per_w, per_w, gw, smem);
  } else if (b < nw + ne) {
    const int c = b - nw;
    const int z = c / per_e;
    gemm_tile<GEMM_DW, 128, 32, 4, 1, FORM_FAST, false>(be.p[z], c - z * per_e, per_e, ge, smem);
  } else {
    const int c = b - nw - ne;
    const int z = c / gx;
    gemm_tile<GEMM_DX, XBM, XBN, XWM, XWN, FORM_FAST, true>(bx.p[z], c - z * gx, gx, gx, smem);
  }
}

// ---- splitting weights --------------------------------------------------------------------------------------
// One lane forms the three parts of eight consecutive contraction indices of one column.
__global__ __launch_bounds__(256) void pack_weights_kernel(const PackBatch b) {
  const PackJob& J = b.job[blockIdx.y];
  const int u = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (u >= 2 * J.steps * J.cols) return;
  const int kg = u / J.cols, c = u - kg * J.cols;
  const float* src = J.src + (long)c * J.stride_c;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = src[(long)min(8 * kg + i, J.K - 1) * J.stride_k];   // all requested before the first is used
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = 8 * kg + i < J.K ? SPLIT_SCALE * v[i] : 0.f;
  uint4 part[3];
  split_pair(v[0], v[1], part[0].x, part[1].x, part[2].x);
  split_pair(v[2], v[3], part[0].y, part[1].y, part[2].y);
  split_pair(v[4], v[5], part[0].z, part[1].z, part[2].z);
  split_pair(v[6], v[7], part[0].w, part[1].w, part[2].w);
  const PackPlace to = pack_place(kg, c, J.cols, J.units);
#pragma unroll
  for (int s = 0; s < 3; ++s) reinterpret_cast<uint4*>(J.dst)[to.at + (long)s * to.step] = part[s];
}

hipError_t launch_pack_weights(const PackBatch& b, hipStream_t stream) {
  int units = 0;
  for (int i = 0; i < b.count; ++i) units = 2 * b.job[i].steps * b.job[i].cols > units ? 2 * b.job[i].steps * b.job[i].cols : units;
  if (units == 0) return hipSuccess;
  TraceScope ts(stream, "pack_weights", 0.0, 0.0);
  hipLaunchKernelGGL(pack_weights_kernel, dim3((units + 255) / 256, b.count), dim3(256), 0, stream, b);
  return hipGetLastError();
}

// Grid geometry of a batch for a tile shape, and the operand form that all its problems allow.
struct BatchGeom {
  int tiles = 0, splits = 1, form = FORM_FAST;
  bool pack = true;                  // every problem has split weights
  double flops = 0.0;
};

static BatchGeom batch_geom(GemmMode mode, const GemmBatch& batch, int BM, int BN) {
  BatchGeom g;
  for (int i = 0; i < batch.count; ++i) {
    const GemmProblem& P = batch.p[i];
    const int t = ((P.M + BM - 1) / BM) * ((P.N + BN - 1) / BN);
    g.tiles = t > g.tiles ? t : g.tiles;
    int form = FORM_FAST;
    if (mode == GEMM_DW) {
      g.splits = P.n_split > g.splits ? P.n_split : g.splits;
      if (P.col_map != nullptr) form = FORM_GENERAL;
      else if (P.row_idx != nullptr || P.idx_mod < P.K) form = FORM_GATHER;
    } else {
      if (!P.a_vec) form = FORM_GENERAL;
      else if (P.row_idx != nullptr && (P.a_src_rows <= 0 || P.a_src_rows * (int64_t)P.lda >= (int64_t)1 << 30)) form = FORM_FAR;
      g.pack = g.pack && P.Bp != nullptr;
    }
    g.form = form > g.form ? form : g.form;
    g.flops += 2.0 * P.M * (double)P.N * P.K;
  }
  return g;
}

template <int MODE, int BM, int BN, int WM, int WN, int FORM, bool PACK>
static void launch_form(const GemmBatch& batch, const dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL((gemm_kernel<MODE, BM, BN, WM, WN, FORM, PACK>), grid, dim3(NT), 0, stream, batch);
}

template <int MODE, int BM, int BN, int WM, int WN>
static hipError_t launch_cfg(const GemmBatch& batch, hipStream_t stream) {
  const BatchGeom g = batch_geom((GemmMode)MODE, batch, BM, BN);
  if (g.tiles == 0) return hipSuccess;
  if (MODE == GEMM_DX && !g.pack) return hipErrorInvalidValue;
  static const char* const mode_name[3] = {"fwd", "dx", "dw"};
  char name[48];
  snprintf(name, sizeof name, "gemm_%s_%dx%d", mode_name[MODE], BM, BN);
  TraceScope ts(stream, name, g.flops, 0.0);
  const dim3 grid(g.tiles, g.splits, batch.count);
  if constexpr (MODE == GEMM_DW) {
    if (g.form == FORM_FAST) launch_form<MODE, BM, BN, WM, WN, FORM_FAST, false>(batch, grid, stream);
    else if (g.form == FORM_GATHER) launch_form<MODE, BM, BN, WM, WN, FORM_GATHER, false>(batch, grid, stream);
    else launch_form<MODE, BM, BN, WM, WN, FORM_GENERAL, false>(batch, grid, stream);
  } else {
    auto launch = [&](auto form) {
      constexpr int F = decltype(form)::value;
      if (g.pack) launch_form<MODE, BM, BN, WM, WN, F, true>(batch, grid, stream);
      else launch_form<MODE, BM, BN, WM, WN, F, MODE == GEMM_DX>(batch, grid, stream);
    };
    if (g.form == FORM_FAST) launch(std::integral_constant<int, FORM_FAST>{});
    else if (MODE == GEMM_FWD && g.form == FORM_FAR) launch(std::integral_constant<int, MODE == GEMM_FWD ? FORM_FAR : FORM_GENERAL>{});
    else launch(std::integral_constant<int, FORM_GENERAL>{});
  }
  return hipGetLastError();
}

// Tile selection.  Three 128x128 workgroups are resident per CU; where there are fewer than about that many (700 tiles
// over 256 CUs), 64x128 tiles fill the chip better (whole updates with a limit of 350 tiles: 0.6 % slower at 4096
// environments and [512, 256, 128], 2.2 % at 1501 and [400, 200, 100]; with 1400: 1.2 % slower and the same), and short
// contractions (K <= 64, bound by their output) also use them.
enum TileCfg { TILE_128x128, TILE_64x128, TILE_128x64, TILE_128x32 };

static TileCfg pick_tile(GemmMode mode, const GemmBatch& batch) {
  int maxM = 0, maxN = 0, minK = 1 << 30, dw_big = 1;
  long tiles128 = 0;
  for (int i = 0; i < batch.count; ++i) {
    const GemmProblem& P = batch.p[i];
    maxM = P.M > maxM ? P.M : maxM;
    maxN = P.N > maxN ? P.N : maxN;
    minK = P.K < minK ? P.K : minK;
    tiles128 += (long)((P.M + 127) / 128) * ((P.N + 127) / 128);
    dw_big &= P.dw_big;
  }
  if (maxN <= 32) return TILE_128x32;
  if (maxM <= 64) return TILE_64x128;
  if (maxN <= 64) return TILE_128x64;
  if (mode == GEMM_DW) return dw_big ? TILE_128x128 : TILE_64x128;
  if (minK <= 64 || tiles128 < 700) return TILE_64x128;
  return TILE_128x128;
}

int gemm_dw_tiles(int32_t M, int32_t N, bool big) {
  if (N <= 32) return (M + 127) / 128;
  if (M <= 64 || !big) return ((M + 63) / 64) * ((N + 127) / 128);
  if (N <= 64) return ((M + 127) / 128) * ((N + 63) / 64);
  return ((M + 127) / 128) * ((N + 127) / 128);
}

template <int MODE>
static hipError_t launch_mode(const GemmBatch& batch, hipStream_t stream) {
  switch (pick_tile((GemmMode)MODE, batch)) {
    case TILE_128x32: return launch_cfg<MODE, 128, 32, 4, 1>(batch, stream);
    case TILE_64x128: return launch_cfg<MODE, 64, 128, 1, 4>(batch, stream);
    case TILE_128x64: return launch_cfg<MODE, 128, 64, 2, 2>(batch, stream);
    default: return launch_cfg<MODE, 128, 128, 2, 2>(batch, stream);
  }
}

template <int WBM, int WBN, int WWM, int WWN, int XBM, int XBN, int XWM, int XWN>
static hipError_t launch_pair_cfg(const GemmBatch& bw, const GemmBatch& bx, const GemmBatch& be, const BatchGeom& gw,
                                  const BatchGeom& gx, const BatchGeom& ge, hipStream_t stream) {
  char name[48];
  snprintf(name, sizeof name, "gemm_dwdx_%dx%d_%dx%d", WBM, WBN, XBM, XBN);
  TraceScope ts(stream, name, gw.flops + gx.flops + ge.flops, 0.0);
  const int blocks = bw.count * gw.tiles * gw.splits + bx.count * gx.tiles + be.count * ge.tiles * ge.splits;
  hipLaunchKernelGGL((gemm_pair_kernel<WBM, WBN, WWM, WWN, XBM, XBN, XWM, XWN>), dim3(blocks), dim3(NT), 0, stream,
                     bw, bx, be, gw.tiles, gw.splits, gx.tiles, ge.tiles, ge.splits);
  return hipGetLastError();
}

// The narrow weight gradient can ride in the paired launch when it takes 128 x 32 tiles.
static bool narrow_dw_fits(const GemmBatch& be) {
  return be.count > 0 && pick_tile(GEMM_DW, be) == TILE_128x32 && batch_geom(GEMM_DW, be, 128, 32).form == FORM_FAST;
}

hipError_t launch_gemm_dw_dx(const GemmBatch& bw, const GemmBatch& bx, hipStream_t stream, const GemmBatch* narrow_dw) {
  const TileCfg tw = pick_tile(GEMM_DW, bw), tx = pick_tile(GEMM_DX, bx);
  const bool w_ok = tw == TILE_128x128 || tw == TILE_64x128, x_ok = tx == TILE_128x128 || tx == TILE_64x128;
  if (w_ok && x_ok && bw.count > 0 && bx.count > 0) {
    const BatchGeom gw = batch_geom(GEMM_DW, bw, tw == TILE_128x128 ? 128 : 64, 128);
    const BatchGeom gx = batch_geom(GEMM_DX, bx, tx == TILE_128x128 ? 128 : 64, 128);
    if (gw.form == FORM_FAST && gx.form == FORM_FAST && gx.pack && gw.tiles > 0 && gx.tiles > 0) {
      GemmBatch be;
      memset(&be, 0, sizeof be);
      BatchGeom ge;
      ge.tiles = 0; ge.splits = 0;
      if (narrow_dw != nullptr && narrow_dw_fits(*narrow_dw)) {
        be = *narrow_dw;
        ge = batch_geom(GEMM_DW, be, 128, 32);
      } else if (narrow_dw != nullptr) {
        hipError_t e = launch_gemm(GEMM_DW, *narrow_dw, stream);
        if (e != hipSuccess) return e;
      }
      if (tw == TILE_128x128 && tx == TILE_128x128) return launch_pair_cfg<128, 128, 2, 2, 128, 128, 2, 2>(bw, bx, be, gw, gx, ge, stream);
      if (tw == TILE_128x128) return launch_pair_cfg<128, 128, 2, 2, 64, 128, 1, 4>(bw, bx, be, gw, gx, ge, stream);
      if (tx == TILE_128x128) return launch_pair_cfg<64, 128, 1, 4, 128, 128, 2, 2>(bw, bx, be, gw, gx, ge, stream);
      return launch_pair_cfg<64, 128, 1, 4, 64, 128, 1, 4>(bw, bx, be, gw, gx, ge, stream);
    }
  }
  if (narrow_dw != nullptr) {
    hipError_t e = launch_gemm(GEMM_DW, *narrow_dw, stream);
    if (e != hipSuccess) return e;
  }
  hipError_t e = launch_gemm(GEMM_DW, bw, stream);
  if (e != hipSuccess) return e;
  return launch_gemm(GEMM_DX, bx, stream);
}

hipError_t launch_gemm(GemmMode mode, const GemmBatch& batch, hipStream_t stream) {
  switch (mode) {
    case GEMM_FWD: return launch_mode<GEMM_FWD>(batch, stream);
    case GEMM_DX: return launch_mode<GEMM_DX>(batch, stream);
    default: return launch_mode<GEMM_DW>(batch, stream);
  }
}

}  // namespace rslx
