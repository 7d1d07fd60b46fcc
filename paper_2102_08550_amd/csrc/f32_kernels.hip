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
// the update.  `rows`: the addresses of the batch's dataset rows (GATHER).
template <int T, bool GATHER>
__device__ __forceinline__ void update_tile(const F32UpdateArgs& u, const F32UpdateLayer& y, int z,
                                            int rep, int m0, int n0, int lane,
                                            const uint64_t* rows) {
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
  const int ns = (u.B + 15) / 16;
  load_index(0, 0);
  load_index(1, 1);
  load(0, 0);
  // The weights, needed after the products only.  Lane (gq, c16) holds inputs
  // m0 + 4 T gq .. + 4 T - 1 of outputs n0 + T c16 + j.
  const float* win = u.master_in + static_cast<int64_t>(rep) * u.master_in_slot;
  float* wout = u.master + static_cast<int64_t>(rep) * u.master_slot;
  const int mo = m0 + 4 * T * gq;
  f32x4 w[T][T];
#pragma unroll
  for (int j = 0; j < T; ++j) {
    const int n = n0 + T * c16 + j < y.N ? n0 + T * c16 + j : 0;
    const float* wrow = win + y.w_off + static_cast<int64_t>(n) * y.M;
#pragma unroll
    for (int qd = 0; qd < T; ++qd) {
      const int m = mo + 4 * qd < y.M ? mo + 4 * qd : 0;
      w[j][qd] = *reinterpret_cast<const f32x4*>(wrow + m);
    }
  }
  for (int s = 0; s < ns; s += 2) {
    load(1, s + 1);
    load_index(0, s + 2);
    loads_first();
    mma(0);
    loads_first();
    load(0, s + 2);
    load_index(1, s + 3);
    loads_first();
    mma(1);  // zeros past the batch
    loads_first();
  }
#pragma unroll
  for (int j = 0; j < T; ++j) {
    const int n = n0 + T * c16 + j;
    const int64_t at = y.w_off + static_cast<int64_t>(n < y.N ? n : 0) * y.M;
#pragma unroll
    for (int qd = 0; qd < T; ++qd) {
      const f32x4 d = acc_quad<true>(acc, j, qd);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[j][qd][e] = fmaf(-u.lr, d[e], w[j][qd][e]);
      if (n < y.N && mo + 4 * qd < y.M)
        *reinterpret_cast<f32x4*>(wout + at + mo + 4 * qd) = w[j][qd];
    }
  }
}

// Backward-weight and the SGD update of every layer in one launch (nothing
// reads the weights after the last backward-data launch).  A workgroup of 2 x
// 2 waves covers 32 T inputs x 32 T outputs of one layer, a wave 16 T x 16 T:
// dW[o][i] over the batch, then W <- W - lr dW.  The biases have workgroups of
// their own (64 outputs each): blocks of 64 batch rows row by row, the block
// sums left to right.
constexpr int UPDATE_ROWS = 1024 + 80;  // largest batch and the groups read ahead
template <int T>
__global__ __launch_bounds__(256, T == 4 ? 1 : 2) void f32_update_kernel(F32UpdateArgs u) {
  // Addresses of the gathered activations' rows at the workgroup's first column
  // (zeros past the batch): one addition per load.
  __shared__ __attribute__((aligned(16))) uint64_t rows[UPDATE_ROWS];
  __shared__ float bias_sum[16][64];  // of the blocks of 64 batch rows
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
  if (tile >= y.tiles) {  // the biases of 64 outputs
    const int n = (tile - y.tiles) * 64 + lane, blocks = (u.B + 63) / 64;
    const float* D = y.d + z * y.d_slot;
    for (int b = wave; b < blocks; b += 4) {
      float sum = 0.0f;
      for (int k = 64 * b; k < 64 * b + 64; k += 16) {
        float v[16];
        const int in = max(min(u.B - k, 16), 0);  // rows padded to 64; zeros past the batch
        const Buf rows16 = buffer(D + static_cast<int64_t>(min(k, u.B)) * y.d_ld, in * y.d_ld * 4);
#pragma unroll
        for (int e = 0; e < 16; ++e)
          v[e] = load_buffer<1>(rows16, 4u * n, 4u * min(e, in) * static_cast<uint32_t>(y.d_ld));
#pragma unroll
        for (int e = 0; e < 16; ++e) sum += v[e];
      }
      bias_sum[b][lane] = sum;
    }
    __syncthreads();
    if (wave == 0 && n < y.N) {
      float db = bias_sum[0][lane];
      for (int b = 1; b < blocks; ++b) db += bias_sum[b][lane];
      const int64_t at = static_cast<int64_t>(rep) * u.master_slot + y.b_off + n;
      u.master[at] = fmaf(-u.lr, db, u.master_in[static_cast<int64_t>(rep) * u.master_in_slot +
                                                 y.b_off + n]);
    }
    return;
  }
  if (gathered) {
    const uint64_t base = reinterpret_cast<uint64_t>(y.a + z * y.a_slot + (m0 & ~(32 * T - 1)));
    const uint64_t zero = reinterpret_cast<uint64_t>(f32_zero_words);
    for (int b = threadIdx.x; b < UPDATE_ROWS; b += 256)
      rows[b] = b < u.B ? base + 4 * offset_of(u.gather[z * u.gather_slot + b], y.a_ld) : zero;
    __syncthreads();
  }
  if (m0 >= y.M || n0 >= y.N) return;
  // The larger tile keeps a SIMD's products busy alone, and two such waves on
  // one SIMD slowed each other (dense activations: 100 us for a pair of tiles, 39
  // for one): these registers leave room for one.
  if constexpr (T == 4) asm volatile("" ::: "a255");
  if (gathered) update_tile<T, true>(u, y, z, rep, m0, n0, lane, rows);
  else update_tile<T, false>(u, y, z, rep, m0, n0, lane, rows);
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
      F32UpdateLayer& y = u.layer[l];
      const int64_t tiles =
          static_cast<int64_t>((y.M + 32 * t - 1) / (32 * t)) * ((y.N + 32 * t - 1) / (32 * t));
      u.first_wg[l] = static_cast<int>(n);
      y.tiles = static_cast<int>(tiles);
      n += tiles + (y.N + 63) / 64;
    }
    return n;
  };
  // 64 x 64 per wave, or 32 x 32, whose 8-byte loads take twice the L1 accesses
  // per byte but whose waves are four times as many and start up sooner.
  // Measured: 784-512-256-10, batch 64, 8 replicas (304 workgroups of the
  // larger tile) 22.8 against 17.9 us; 1024-2048-2048-10, batch 512, 1 replica
  // (465 workgroups) 82 against 102 us.
  for (int l = u.n_layers; l < F32_UPDATE_LAYERS; ++l) u.first_wg[l] = 0x7FFFFFFF;
  int t = 4;
  int64_t gx = groups(4);
  if (u.B < 128 || gx * n_slots < 256) {
    t = 2;
    gx = groups(2);
  }
  if (gx * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(gx), n_slots), block(256);
  if (t == 4) hipLaunchKernelGGL(f32_update_kernel<4>, grid, block, 0, s, u);
  else hipLaunchKernelGGL(f32_update_kernel<2>, grid, block, 0, s, u);
  return hipGetLastError();
}

}  // namespace oscars
