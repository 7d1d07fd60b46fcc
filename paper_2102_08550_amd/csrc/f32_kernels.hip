// Local steps of fp32 MLPs for gfx950: forward, backward-data, backward-weight
// with the SGD update of Eq. 4, and the classifier head.
//
// fp32 MFMA (16x16x4: 2048 flops in 32 cycles per SIMD, 157 TFLOP/s over the
// chip) is slow next to the vector caches: a 64 x 64 wave tile takes 2048
// cycles of products per 16 K and needs only 8 KB of operands for them.  So
// the waves read their MFMA operands straight from memory (L1 / L2) into
// registers, one or more K groups ahead of the products: no LDS staging and
// no barrier in any K loop, and waves drift freely.  LDS is used once, to add
// the K slices of an output tile.
//
// K order of forward and backward-data: slice j = 0..3 takes the 32-wide K
// tiles j, j + 4, j + 8, ... in order (one wave per slice), the output is
// ((s0 + s1) + s2) + s3 (the classifier head: eight slices).  A slice sums each
// 1024 of its K from zero and adds those sums in order, so no accumulator
// runs over more than 1024 products however wide the layer is.  The order
// depends only on K, not on the tile shape or on how many replicas share a
// launch, so every tiling gives the same bits.  Backward-weight sums the batch
// in row order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "mfma_f32.h"

namespace oscars {
namespace {

constexpr int SLICES = 4;  // K slices of forward / backward-data = waves per workgroup
constexpr int HEAD_SLICES = 8;  // of the classifier head
constexpr int KTILE = 32;  // K tile dealt to the slices in turn
constexpr int KFOLD = 1024;  // of a slice's K in one running sum

// K groups (16 deep) a wave loads at once: enough bytes in flight for small
// tiles, few registers for large ones.  A slice is summed in whole pairs of
// such loads (zeros past K): with a test between the products the compiler
// sinks the loads of the next groups behind it, next to their use.
template <int MI, int NJ> struct Depth {
  static constexpr int G = MI + NJ >= 8 ? 1 : (MI + NJ >= 4 ? 2 : 4);
};
// Floats of a wave's LDS for the K-contiguous operands of slice_products.
template <bool TRANS, int MI, int NJ> constexpr int slice_lds() {
  return Depth<MI, NJ>::G * ((TRANS ? 0 : MI) + NJ) * BLOCK_FLOATS;
}

// A K-contiguous operand of a tile: rows row0 .. of a matrix with row stride
// ld, N blocks of 16 (rows past the last repeat it; their outputs are not
// stored), or, gathered, rows anywhere.
template <int N>
struct Rows {
  Buf buf;
  uint32_t at[N];
  const float* row[N];  // gathered
  bool gathered;
  __device__ __forceinline__ void init(const float* base, int64_t ld, int row0, int rows, int lane) {
    const int last = min(rows - 1 - row0, 16 * N - 1);
    buf = buffer(base + static_cast<int64_t>(row0) * ld, (last + 1) * ld * 4);
#pragma unroll
    for (int i = 0; i < N; ++i)
      at[i] = 4u * (static_cast<uint32_t>(min(16 * i + load_row(lane), last)) *
                        static_cast<uint32_t>(ld) + load_k(lane));
    gathered = false;
  }
  __device__ __forceinline__ void init_gathered(const float* base, int64_t ld,
                                                const int32_t* gather, int row0, int rows,
                                                int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      row[i] = base + static_cast<int64_t>(gather[min(row0 + 16 * i + load_row(lane), rows - 1)]) * ld +
               load_k(lane);
    gathered = true;
  }
};

// K slice `slice` of S of a 16 MI x 16 NJ tile of A B^T.  A: rows (K-contiguous)
// or, TRANS, a_cols: row 0, column m0 (the tile's first) of a K x M matrix with
// row stride a_ld = M.  Zeros from K (A) and from b_ext (B) on.  The loads of groups
// q + 2, the turn through LDS of q + 1 and the products of q are in flight
// together.  FOLD: slices longer than KFOLD; kernels of their own, since the
// second accumulator set cost the others registers they never used.
template <bool TRANS, bool GATHER, bool FOLD, int S, int MI, int NJ>
__device__ __forceinline__ void slice_products(f32x4 (&acc)[MI][NJ], const Rows<TRANS ? 1 : MI>& ra,
                                               const Rows<NJ>& rb, const float* a_cols,
                                               int m0, int64_t a_ld, int K, int b_ext, int slice,
                                               int lane, float* lds) {
  constexpr int G = Depth<MI, NJ>::G;
  constexpr int AB = TRANS ? 0 : MI, NB = G * (AB + NJ);  // blocks through LDS
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int tiles = (K + KTILE - 1) / KTILE;
  const int nq = tiles > slice ? 2 * ((tiles - slice + S - 1) / S) : 0;
  if (nq == 0) return;
  const float* zero = GATHER ? zero_words() : nullptr;
  auto k_of = [&](int q) { return KTILE * (slice + S * (q >> 1)) + 16 * (q & 1); };
  f32x4 raw[NB];
  auto load_rows = [&](int q0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int k = k_of(q0 + g);
      const uint32_t k4 = 4u * min(k, K);  // within every row's buffer
      const bool a_ok = load_k(lane) < K - k;  // K is a multiple of 4: whole chunks
      const bool b_ok = load_k(lane) < b_ext - k;
#pragma unroll
      for (int i = 0; i < AB; ++i)
        raw[g * (AB + NJ) + i] = load_buffer<4>(ra.buf, a_ok ? ra.at[i] : NOWHERE, k4);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f32x4& v = raw[g * (AB + NJ) + AB + j];
        if constexpr (GATHER) v = load_global<4>(b_ok ? rb.row[j] + k : zero);
        else v = load_buffer<4>(rb.buf, b_ok ? rb.at[j] : NOWHERE, k4);
      }
    }
  };
  uint32_t col_at[4];
  if constexpr (TRANS) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      col_at[t] = 4u * ((4 * (lane >> 4) + t) * static_cast<uint32_t>(a_ld) + MI * (lane & 15));
  }
  struct Set {
    f32x4 rows[NB];
    float cols[TRANS ? G : 1][TRANS ? MI : 1][4];
  } f0, f1;
  auto load_cols = [&](Set& f, int q0) {
    if constexpr (TRANS) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // 16 rows of the matrix from K row k; zeros past K.  (Columns past M are
        // other rows' values or zeros; their outputs are not stored.)
        const int k = min(k_of(q0 + g), K);
        const Buf b = buffer(a_cols + static_cast<int64_t>(k) * a_ld,
                             k < K ? (min(K - k, 16) * a_ld - m0) * 4 : 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float v[MI];
          load_buffer_vec<MI>(v, b, col_at[t], 0);
#pragma unroll
          for (int i = 0; i < MI; ++i) f.cols[g][i][t] = v[i];
        }
      }
    }
  };
  auto mma = [&](const Set& f) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            float a;
            if constexpr (TRANS) a = f.cols[g][i][t];
            else a = f.rows[g * (AB + NJ) + i][t];
            acc[i][j] = mfma16(a, f.rows[g * (AB + NJ) + AB + j][t], acc[i][j]);
          }
  };
  constexpr int NM = 4 * G * MI * NJ, NV = NB + (TRANS ? 4 * G : 0);
  load_rows(0);
  load_cols(f0, 0);
  blocks_write(lds, raw, lane);
  load_rows(G);
  blocks_read(lds, f0.rows, lane);
  auto two_sets = [&](int q0) {
    blocks_write(lds, raw, lane);
    load_rows(q0 + 2 * G);
    load_cols(f1, q0 + G);
    blocks_read(lds, f1.rows, lane);
    mma(f0);
    spread<NM, NB, NB, NV>();
    blocks_write(lds, raw, lane);
    load_rows(q0 + 3 * G);
    load_cols(f0, q0 + 2 * G);
    blocks_read(lds, f0.rows, lane);
    mma(f1);
    spread<NM, NB, NB, NV>();
  };
  if constexpr (!FOLD) {
    for (int q0 = 0; q0 < nq; q0 += 2 * G) two_sets(q0);
  } else {
    constexpr int PER = KFOLD / 16;  // groups per sum
    static_assert(PER % (2 * G) == 0, "whole loop steps per sum");
    f32x4 tot[MI][NJ];
    for (int q0 = 0; q0 < nq;) {
      const bool first = q0 == 0;
      for (const int end = min(nq, q0 + PER); q0 < end; q0 += 2 * G) two_sets(q0);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          tot[i][j] = first ? acc[i][j] : tot[i][j] + acc[i][j];
          acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = tot[i][j];
  }
}

// Forward and backward-data (GemmArgs as for the other GEMM kernels, without
// rows_out and the split): one 16 MI x 16 NJ output tile per workgroup, one
// K slice per wave.
template <int MODE, int MI, int NJ, bool GATHER, bool FOLD>
__global__ __launch_bounds__(64 * SLICES, 2) void f32_gemm_kernel(GemmArgs g) {
  constexpr bool TRANS = MODE == GEMM_DGRAD;
  // The slices meet in LDS, at most 32 columns at a time (64 x 64 tiles: two
  // phases of 70 KB).
  constexpr int TM = 16 * MI, TN = 16 * NJ, LD = TM + 4;
  constexpr int NP = NJ > 2 ? 2 : 1, PN = TN / NP;  // phases, columns per phase
  constexpr int STAGE = slice_lds<TRANS, MI, NJ>();
  __shared__ __attribute__((aligned(16))) union {
    float stage[SLICES][STAGE];  // each wave's own
    float red[SLICES][PN][LD];
  } sm;
  auto& red = sm.red;
  const int lane = threadIdx.x & 63;
  const int slice = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int work = xcd_item(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int z = work / gridDim.x, tile = work % gridDim.x;
  const int rep = g.order[z];
  const int gn = (g.N + TN - 1) / TN;
  const int m0 = tile / gn * TM, n0 = tile % gn * TN;
  const float* A = static_cast<const float*>(g.a) + (g.a_by_order ? rep : z) * g.a_slot;
  const float* B = static_cast<const float*>(g.b) + z * g.b_slot;

  Rows<TRANS ? 1 : MI> ra;
  Rows<NJ> rb;
  if constexpr (!TRANS) ra.init(A, g.a_ld, m0, g.M, lane);
  if constexpr (GATHER) rb.init_gathered(B, g.b_ld, g.gather + z * g.gather_slot, n0, g.N, lane);
  else rb.init(B, g.b_ld, n0, g.N, lane);
  f32x4 acc[MI][NJ];
  slice_products<TRANS, GATHER, FOLD, SLICES>(acc, ra, rb, A + m0, m0, g.a_ld, g.K, g.b_ext, slice,
                                              lane, sm.stage[slice]);

  // A thread takes four consecutive rows m of column n.
  constexpr int PER = (MI * 4 * PN + 64 * SLICES - 1) / (64 * SLICES);  // per thread and phase
  f32x4 aux[NP][PER];  // bias, or the activations that mask the delta
  const float* bias = g.master_in + static_cast<int64_t>(rep) * g.master_in_slot + g.b_off;
#pragma unroll
  for (int ph = 0; ph < NP; ++ph)
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = threadIdx.x + 64 * SLICES * p;
      const int n = min(n0 + ph * PN + c / (4 * MI), g.N - 1);
      const int m = min(m0 + 4 * (c % (4 * MI)), (g.M - 1) & ~3);
      // bias segments and activation rows are padded to 64 elements
      aux[ph][p] = *reinterpret_cast<const f32x4*>(
          MODE == GEMM_FWD ? bias + m
                           : static_cast<const float*>(g.mask) + z * g.mask_slot +
                                 static_cast<int64_t>(n) * g.mask_ld + m);
    }
#pragma unroll
  for (int ph = 0; ph < NP; ++ph) {
    __syncthreads();  // every wave is done with its stage, or the last phase is read
#pragma unroll
    for (int j = 0; j < NJ / NP; ++j)
#pragma unroll
      for (int qd = 0; qd < MI; ++qd)
        *reinterpret_cast<f32x4*>(
            &red[slice][16 * j + (lane & 15)][quad_row<TRANS, MI>(qd, lane)]) =
            acc_quad<TRANS>(acc, ph * (NJ / NP) + j, qd);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = threadIdx.x + 64 * SLICES * p;
      const int nl = c / (4 * MI), n = n0 + ph * PN + nl, m = 4 * (c % (4 * MI));
      if (nl >= PN || n >= g.N || m0 + m >= g.M) continue;
      f32x4 v = *reinterpret_cast<const f32x4*>(&red[0][nl][m]);
#pragma unroll
      for (int s = 1; s < SLICES; ++s) v = v + *reinterpret_cast<const f32x4*>(&red[s][nl][m]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (MODE == GEMM_FWD) {
          v[e] += aux[ph][p][e];
          if (g.relu) v[e] = fmaxf(v[e], 0.0f);
        } else {
          v[e] = aux[ph][p][e] > 0.0f ? v[e] : 0.0f;
        }
      }
      float* o = static_cast<float*>(g.out) + z * g.out_slot + static_cast<int64_t>(n) * g.out_ld +
                 m0 + m;
      if (m0 + m + 4 <= g.M) {
        *reinterpret_cast<f32x4*>(o) = v;
      } else {
        for (int e = 0; m0 + m + e < g.M; ++e) o[e] = v[e];
      }
    }
  }
}

// The classifier head of 16 batch rows per workgroup, up to 64 classes:
// logits (the forward pass of the last layer, as f32_gemm_kernel), softmax
// cross-entropy (as softmax_ce_kernel), and, with DGRAD, the delta of the
// layer below (as f32_gemm_kernel's backward-data).  One launch instead of
// three whose own latency was all they cost.
template <int MI, bool DGRAD, bool GATHER, bool FOLD>
__global__ __launch_bounds__(64 * HEAD_SLICES) void f32_head_kernel(F32HeadArgs h) {
  constexpr int TM = 16 * MI, LD = TM + 4, ROWS = 16;
  constexpr int STAGE = slice_lds<false, MI, 1>();
  __shared__ __attribute__((aligned(16))) union {
    float stage[HEAD_SLICES][STAGE];  // each wave's own
    float red[HEAD_SLICES][ROWS][LD];
  } sm;
  auto& red = sm.red;
  __shared__ __attribute__((aligned(16))) float dl[ROWS][LD];
  const int lane = threadIdx.x & 63, c16 = lane & 15, gq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int z = blockIdx.y, rep = h.order[z], n0 = blockIdx.x * ROWS;
  const float* master = h.master_in + static_cast<int64_t>(rep) * h.master_in_slot;
  const float* W = master + h.w_off;
  const float* act = h.act + z * h.act_slot;
  Rows<MI> ra;
  Rows<1> rb;
  ra.init(W, h.K, 0, h.C, lane);
  if constexpr (GATHER) rb.init_gathered(act, h.act_ld, h.gather + z * h.gather_slot, n0, h.B, lane);
  else rb.init(act, h.act_ld, n0, h.B, lane);
  // labels and bias before the products: their latency is hidden
  int label[ROWS / HEAD_SLICES];
#pragma unroll
  for (int r = 0; r < ROWS / HEAD_SLICES; ++r) {
    const int b = min(n0 + wave * (ROWS / HEAD_SLICES) + r, h.B - 1);
    label[r] = h.y[h.gather ? h.gather[z * h.gather_slot + b] : b];
  }
  const float bias = master[h.b_off + min(lane, h.C - 1)];
  f32x4 acc[MI][1];
  slice_products<false, GATHER, FOLD, HEAD_SLICES>(acc, ra, rb, nullptr, 0, h.K, h.K, h.K, wave, lane,
                                                   sm.stage[wave]);
  __syncthreads();  // every wave is done with its stage
#pragma unroll
  for (int i = 0; i < MI; ++i)
    *reinterpret_cast<f32x4*>(&red[wave][c16][16 * i + 4 * gq]) = acc[i][0];
  __syncthreads();
  // A wave takes two rows, lane c the class c (the sums as softmax_ce_kernel).
  const float invB = 1.0f / static_cast<float>(h.B);
#pragma unroll
  for (int r = 0; r < ROWS / HEAD_SLICES; ++r) {
    const int row = wave * (ROWS / HEAD_SLICES) + r, b = n0 + row;
    const int cl = min(lane, TM - 1);
    float v = red[0][row][cl];
#pragma unroll
    for (int s = 1; s < HEAD_SLICES; ++s) v += red[s][row][cl];
    v += bias;
    const bool in = lane < h.C;
    if (!in) v = -INFINITY;
    const bool label_ok = label[r] >= 0 && label[r] < h.C;
    const float zl = __shfl(v, label[r] & 63);
    float mx = v;
    for (int d = 32; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
    const float ex = in ? expf(v - mx) : 0.0f;
    float s = ex;
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    const float dv = in && b < h.B ? (ex / s - (lane == label[r] ? 1.0f : 0.0f)) * invB : 0.0f;
    if (DGRAD && lane < TM) dl[row][lane] = dv;
    if (b < h.B) {
      if (h.delta)
        for (int c = lane; c < h.delta_ld; c += 64)
          h.delta[z * h.delta_slot + static_cast<int64_t>(b) * h.delta_ld + c] = c < 64 ? dv : 0.0f;
      if (lane == 0) {
        h.loss[z * h.loss_slot + b] = label_ok ? logf(s) - (zl - mx) : __builtin_nanf("");
        if (h.correct) h.correct[z * h.loss_slot + b] = label_ok && zl >= mx ? 1 : 0;
      }
    }
  }
  if constexpr (DGRAD) {
    __syncthreads();
    // delta of the layer below for these rows, 64 inputs per wave and turn:
    // K = classes, slices 0 (classes 0..31) and 1 (32..63) summed apart.
    float bd[MI][4];
#pragma unroll
    for (int s = 0; s < MI; ++s) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&dl[c16][16 * s + 4 * gq]);
#pragma unroll
      for (int t = 0; t < 4; ++t) bd[s][t] = v[t];
    }
    const int b = n0 + c16;
    const float* zero = zero_words();
    for (int m0 = 64 * wave; m0 < h.K; m0 += 64 * HEAD_SLICES) {
      const int m = m0 + 4 * c16;
      const float* col = W + (m < h.K ? m : 0);
      f32x4 w[MI][4];
#pragma unroll
      for (int s = 0; s < MI; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int k = 16 * s + 4 * gq + t;
          w[s][t] = load_global<4>(k < h.C ? col + static_cast<int64_t>(k) * h.K : zero);
        }
      const int mo = m0 + 16 * gq;  // this lane's 16 outputs
      const int64_t at = static_cast<int64_t>(min(b, h.B - 1)) * h.act_ld;
      f32x4 mask[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        mask[r] = load_global<4>(mo + 4 * r < h.K ? h.act + z * h.act_slot + at + mo + 4 * r : zero);
      f32x4 d[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) d[u][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < MI; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            d[s >> 1][i] = mfma16(w[s][t][i], bd[s][t], d[s >> 1][i]);
      if (b < h.B) {
        float* o = h.below + z * h.below_slot + static_cast<int64_t>(b) * h.below_ld + mo;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          f32x4 v;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x = d[0][i][r] + d[1][i][r];
            v[i] = mask[r][i] > 0.0f ? x : 0.0f;
          }
          if (mo + 4 * r < h.K) *reinterpret_cast<f32x4*>(o + 4 * r) = v;
        }
      }
    }
  }
}

// One wave's 16 T inputs x 16 T outputs of a layer: dW over the batch, then
// the update.  `rows`: the addresses of the batch's dataset rows (GATHER).  BIAS:
// the bias gradient too, from the deltas that the products have in registers:
// each lane adds the rows of its own (4 q .. 4 q + 3 of 16, q its group of
// 16 lanes), the four groups are added at the end, (0 + 1) + (2 + 3).
template <int T, bool GATHER, bool BIAS>
__device__ __forceinline__ void update_tile(const F32UpdateArgs& u, const F32UpdateLayer& y, int z,
                                            int rep, int m0, int n0, int lane,
                                            const uint64_t* rows, float* lds) {
  const int c16 = lane & 15, gq = lane >> 4;
  // Four batch rows of 16 T columns per load.  Columns past M are other rows'
  // values (never stored); delta rows are padded to 64.
  const float* A = y.a + z * y.a_slot + m0;
  const float* D = y.d + z * y.d_slot + n0;
  // (Gathered rows: column 0 of the tile instead, inside the row.)
  const uint32_t ma = m0 + T * c16 < y.M ? 4u * ((m0 & 16 * T) + T * c16) : 0;
  uint32_t a_at[4], d_at[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a_at[t] = 4u * ((4 * gq + t) * static_cast<uint32_t>(y.a_ld) + T * c16);
    d_at[t] = 4u * ((4 * gq + t) * static_cast<uint32_t>(y.d_ld) + T * c16);
  }
  float a[2][T][4], b[2][T][4];
  uint64_t row[2][4];  // of the group loaded next into each set
  auto load_index = [&](int set, int s) {
    if constexpr (GATHER) {
#pragma unroll
      for (int t = 0; t < 4; ++t) row[set][t] = rows[16 * s + 4 * gq + t];
    }
  };
  auto load = [&](int set, int s) {
    // 16 batch rows from row 16 s; zeros past the batch
    const int k = min(16 * s, u.B), n = min(u.B - k, 16);
    const Buf db = buffer(D + static_cast<int64_t>(k) * y.d_ld, n > 0 ? (n * y.d_ld - n0) * 4 : 0);
    const Buf ab = buffer(A + static_cast<int64_t>(k) * y.a_ld, n > 0 ? (n * y.a_ld - m0) * 4 : 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float va[T], vb[T];
      if constexpr (GATHER) {
        load_vec<T>(va, reinterpret_cast<const float*>(row[set][t] + ma));
      } else {
        load_buffer_vec<T>(va, ab, a_at[t], 0);
      }
      load_buffer_vec<T>(vb, db, d_at[t], 0);
#pragma unroll
      for (int i = 0; i < T; ++i) {
        a[set][i][t] = va[i];
        b[set][i][t] = vb[i];
      }
    }
  };
  f32x4 acc[T][T];
#pragma unroll
  for (int j = 0; j < T; ++j)
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto mma = [&](int set) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = mfma16(a[set][i][t], b[set][j][t], acc[i][j]);
  };
  float db[T];
#pragma unroll
  for (int j = 0; j < T; ++j) db[j] = 0.0f;
  auto add_bias = [&](int set) {
    if constexpr (BIAS) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < T; ++j) db[j] += b[set][j][t];
    }
  };
  const int ns = (u.B + 15) / 16;
  load_index(0, 0);
  load_index(1, 1);
  load(0, 0);
  // The weights, needed after the products only: whole rows of the tile (4 T
  // lanes of 16 bytes), the sums come to this layout through LDS.
  const float* win = u.master_in + static_cast<int64_t>(rep) * u.master_in_slot;
  float* wout = u.master + static_cast<int64_t>(rep) * u.master_slot;
  constexpr int CH = 4 * T, RPI = 64 / CH;  // 16-byte chunks per row, rows per load
  const int wr = lane / CH, wc = lane % CH;
  const bool col_in = m0 + 4 * wc < y.M;
  f32x4 w[T * T];
#pragma unroll
  for (int i = 0; i < T * T; ++i) {
    const int n = n0 + RPI * i + wr;
    w[i] = *reinterpret_cast<const f32x4*>(win + y.w_off + static_cast<int64_t>(n < y.N ? n : 0) * y.M +
                                           (col_in ? m0 + 4 * wc : 0));
  }
  float bias[T];  // and the biases: loaded where they are used, their latency was the wave's end
  if constexpr (BIAS) {
#pragma unroll
    for (int j = 0; j < T; ++j) bias[j] = win[y.b_off + min(n0 + T * c16 + j, y.N - 1)];
  }
  for (int s = 0; s < ns; s += 2) {
    load(1, s + 1);
    load_index(0, s + 2);
    loads_first();
    mma(0);
    add_bias(0);
    loads_first();
    load(0, s + 2);
    load_index(1, s + 3);
    loads_first();
    mma(1);  // zeros past the batch
    add_bias(1);
    loads_first();
  }
  if constexpr (BIAS) {
#pragma unroll
    for (int j = 0; j < T; ++j) {
      db[j] += __shfl_xor(db[j], 16);
      db[j] += __shfl_xor(db[j], 32);
      const int n = n0 + T * c16 + j;
      if (gq == 0 && n < y.N) wout[y.b_off + n] = fmaf(-u.lr, db[j], bias[j]);
    }
  }
  // Chunk c of row r at c ^ (r / T) (no bank conflicts either way); LDS
  // operations of one wave execute in order, no barrier.
#pragma unroll
  for (int j = 0; j < T; ++j)
#pragma unroll
    for (int qd = 0; qd < T; ++qd)
      *reinterpret_cast<f32x4*>(lds + (T * c16 + j) * 4 * CH + 4 * ((T * gq + qd) ^ (c16 & (CH - 1)))) =
          acc_quad<true>(acc, j, qd);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < T * T; ++i) {
    const int r = RPI * i + wr, n = n0 + r;
    const f32x4 d = *reinterpret_cast<const f32x4*>(lds + r * 4 * CH + 4 * (wc ^ (r / T & (CH - 1))));
#pragma unroll
    for (int e = 0; e < 4; ++e) w[i][e] = fmaf(-u.lr, d[e], w[i][e]);
    if (n < y.N && col_in)
      *reinterpret_cast<f32x4*>(wout + y.w_off + static_cast<int64_t>(n) * y.M + m0 + 4 * wc) = w[i];
  }
}

// Backward-weight and the SGD update of every layer in one launch (nothing
// reads the weights after the last backward-data launch).  A workgroup of 2 x
// 2 waves covers 32 T inputs x 32 T outputs of one layer, a wave 16 T x 16 T:
// dW[o][i] over the batch, then W <- W - lr dW; the waves of input 0 update the
// biases too.  ALONE: registers for one wave per SIMD only.  What bounds it is
// the fp32 products where a wave's tile is 64 x 64 (1024-2048-2048-10, batch 512: 79
// us, 82 TFLOP/s in two uneven passes over the CUs), and the weights, read and
// written once, at short batches (4096-4096-4096-4096-1000, two replicas, batch 256:
// 543 us).  Biases in workgroups of their own read every delta once more
// and held a CU each: 784-4000 at one replica, batch 1012 134 against 75 us,
// 256-4000 at 35, batch 128 179 against 137; 16-byte pieces of the weights, as the
// products leave them, instead of whole rows: 2048-2048-10 at 8, batch 128 119
// against 115, 4096-wide 576 against 543.
constexpr int UPDATE_ROWS = 1024 + 48;  // largest batch and the groups read ahead
template <int T, bool ALONE>
__global__ __launch_bounds__(256, ALONE ? 1 : 2) void f32_update_kernel(F32UpdateArgs u) {
  // Addresses of the gathered activations' rows at the workgroup's first column
  // (zeros past the batch): one addition per load.
  __shared__ __attribute__((aligned(16))) uint64_t rows[UPDATE_ROWS];
  __shared__ __attribute__((aligned(16))) float sums[4][256 * T * T];  // each wave's own
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int work = xcd_item(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int z = work / gridDim.x, wg = work % gridDim.x;
  // one load of the whole table instead of one per layer, each waiting for
  // the last (entries past the last layer are INT_MAX)
  int l = 0;
#pragma unroll
  for (int i = 1; i < F32_UPDATE_LAYERS; ++i) l += wg >= u.first_wg[i] ? 1 : 0;
  const F32UpdateLayer& y = u.layer[l];
  const int rep = u.order[z];
  const int gm = (y.M + 32 * T - 1) / (32 * T), tile = wg - u.first_wg[l];
  const int m0 = (tile % gm * 2 + (wave & 1)) * 16 * T;
  const int n0 = (tile / gm * 2 + (wave >> 1)) * 16 * T;
  const bool gathered = l == 0 && u.gather != nullptr;
  if (gathered) {
    const uint64_t base = reinterpret_cast<uint64_t>(y.a + z * y.a_slot + (m0 & ~(32 * T - 1)));
    const uint64_t zero = reinterpret_cast<uint64_t>(f32_zero_words);
    const int end = (u.B + 15) / 16 * 16 + 48;  // and the groups read ahead
    for (int b = threadIdx.x; b < end; b += 256)
      rows[b] = b < u.B ? base + 4 * offset_of(u.gather[z * u.gather_slot + b], y.a_ld) : zero;
    __syncthreads();
  }
  if (m0 >= y.M || n0 >= y.N) return;
  if constexpr (ALONE) asm volatile("" ::: "a255");
  if (gathered) {
    if (m0 == 0) update_tile<T, true, true>(u, y, z, rep, m0, n0, lane, rows, sums[wave]);
    else update_tile<T, true, false>(u, y, z, rep, m0, n0, lane, rows, sums[wave]);
  } else {
    if (m0 == 0) update_tile<T, false, true>(u, y, z, rep, m0, n0, lane, rows, sums[wave]);
    else update_tile<T, false, false>(u, y, z, rep, m0, n0, lane, rows, sums[wave]);
  }
}

template <int MODE, int MI, int NJ, bool FOLD>
hipError_t f32_gemm_grid(const GemmArgs& g, int n_slots, hipStream_t s) {
  const int64_t gx = static_cast<int64_t>((g.M + 16 * MI - 1) / (16 * MI)) *
                     ((g.N + 16 * NJ - 1) / (16 * NJ));
  if (gx * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(gx), n_slots), block(64 * SLICES);
  if constexpr (MODE == GEMM_FWD) {
    if (g.gather) {
      hipLaunchKernelGGL((f32_gemm_kernel<MODE, MI, NJ, true, FOLD>), grid, block, 0, s, g);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((f32_gemm_kernel<MODE, MI, NJ, false, FOLD>), grid, block, 0, s, g);
  return hipGetLastError();
}
template <int MODE, int MI, int NJ>
hipError_t f32_gemm_launch(const GemmArgs& g, int n_slots, hipStream_t s) {
  return g.K > SLICES * KFOLD ? f32_gemm_grid<MODE, MI, NJ, true>(g, n_slots, s)
                              : f32_gemm_grid<MODE, MI, NJ, false>(g, n_slots, s);
}

template <int MODE>
hipError_t f32_gemm_mode(const GemmArgs& g, int n_slots, hipStream_t s, int tiling) {
  switch (tiling) {
    case GEMM_TILING_L: return f32_gemm_launch<MODE, 4, 4>(g, n_slots, s);
    case GEMM_TILING_M: return f32_gemm_launch<MODE, 2, 2>(g, n_slots, s);
    default: return f32_gemm_launch<MODE, 1, 1>(g, n_slots, s);
  }
}

}  // namespace

hipError_t launch_f32_gemm(const GemmArgs& g, GemmMode mode, int n_slots, hipStream_t s,
                           int tiling) {
  if (mode == GEMM_FWD) return f32_gemm_mode<GEMM_FWD>(g, n_slots, s, tiling);
  if (mode == GEMM_DGRAD) return f32_gemm_mode<GEMM_DGRAD>(g, n_slots, s, tiling);
  return hipErrorInvalidValue;
}

hipError_t launch_f32_head(const F32HeadArgs& h, int n_slots, hipStream_t s) {
  if (h.B < 1 || n_slots < 1) return hipSuccess;
  if (h.C < 1 || h.C > F32_HEAD_CLASSES || (h.below && h.act_gather)) return hipErrorInvalidValue;
  const dim3 grid((h.B + 15) / 16, n_slots), block(64 * HEAD_SLICES);
#define HEAD(mi, fold)                                                                               \
  if (h.below) hipLaunchKernelGGL((f32_head_kernel<mi, true, false, fold>), grid, block, 0, s, h);   \
  else if (h.act_gather)                                                                             \
    hipLaunchKernelGGL((f32_head_kernel<mi, false, true, fold>), grid, block, 0, s, h);              \
  else hipLaunchKernelGGL((f32_head_kernel<mi, false, false, fold>), grid, block, 0, s, h)
  if (h.K > HEAD_SLICES * KFOLD) {
    if (h.C <= 16) { HEAD(1, true); }
    else if (h.C <= 32) { HEAD(2, true); }
    else { HEAD(4, true); }
  } else if (h.C <= 16) { HEAD(1, false); }
  else if (h.C <= 32) { HEAD(2, false); }
  else { HEAD(4, false); }
#undef HEAD
  return hipGetLastError();
}

hipError_t launch_f32_update(const F32UpdateArgs& u_in, int n_slots, hipStream_t s) {
  if (n_slots < 1) return hipSuccess;
  F32UpdateArgs u = u_in;
  if (u.n_layers < 1 || u.n_layers > F32_UPDATE_LAYERS || u.B < 1 || u.B > 1024)
    return hipErrorInvalidValue;
  auto groups = [&](int t) {
    int64_t n = 0;
    for (int l = 0; l < u.n_layers; ++l) {
      const F32UpdateLayer& y = u.layer[l];
      u.first_wg[l] = static_cast<int>(n);
      n += static_cast<int64_t>((y.M + 32 * t - 1) / (32 * t)) * ((y.N + 32 * t - 1) / (32 * t));
    }
    return n;
  };
  for (int l = u.n_layers; l < F32_UPDATE_LAYERS; ++l) u.first_wg[l] = 0x7FFFFFFF;
  // Waves of 64 x 64 outputs, or of 32 x 32, whose 8-byte loads take twice the
  // L1 accesses per byte but whose waves are four times as many, start up sooner
  // and waste less of narrow layers.  Their times (us) fitted over 76 models of
  // 10 to 4096 wide layers, 1 to 44 replicas and batches 8 to 1024 (rms 13 and 9%;
  // the faster one is missed by 1% on average): a start, the weights per
  // workgroup, and per batch row one wave's products or all workgroups'.  Both
  // sides, 32 x 32 and 64 x 64: 784-512-256-10 at 8 replicas, batch 64 19 and 22,
  // batch 512 77 and 76; 456-100 at 10, batch 855 25 and 62; 1024-2048-2048-10 at
  // one, batch 512 121 and 79; 784-4000 at one, batch 1012 132 and 75.
  const int64_t g4 = groups(4) * n_slots, g2 = groups(2) * n_slots;
  const float t2 = 8.0f + 4e-3f * g2 + u.B * std::max(0.02f, 1.15e-4f * g2);
  const float t4 = 9.0f + 0.024f * g4 + u.B * std::max(0.06f, 2.65e-4f * g4);
  const int64_t gx = groups(t2 < t4 ? 2 : 4);
  // Two waves of the larger tile on one SIMD slow each other's products (dense
  // activations: 100 us for a pair of tiles, 39 for one) but hide each other's
  // start and weights, which is more with short batches and several tiles per
  // CU.  Alone and in pairs: 2048-2048-10 at 8 replicas (2176 workgroups), batch
  // 128 127 and 115, 200 176 and 172, 320 230 and 235, 512 331 and 359;
  // 256-4000, batch 128, at 35 (2240) 146 and 137, at 8 (512) 38 and 41.
  const bool alone = u.B >= 176 || g4 < 1024;
  if (g2 > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(gx), n_slots), block(256);
  if (t2 < t4) hipLaunchKernelGGL((f32_update_kernel<2, false>), grid, block, 0, s, u);
  else if (alone) hipLaunchKernelGGL((f32_update_kernel<4, true>), grid, block, 0, s, u);
  else hipLaunchKernelGGL((f32_update_kernel<4, false>), grid, block, 0, s, u);
  return hipGetLastError();
}

}  // namespace oscars
