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
// K order of forward and backward-data: slice j = 0..3 sums the 32-wide K
// tiles j, j + 4, j + 8, ... from zero in K order (one wave per slice), the
// output is ((s0 + s1) + s2) + s3 (the classifier head: eight slices).  It
// depends only on K, not on the tile
// shape or on how many replicas share a launch, so every tiling gives the
// same bits.  Backward-weight sums the batch in row order.
//
// An MFMA contracts k = 16 s + 4 q + t over the lane groups q = 0..3
// (lane >> 4) for its t; a lane's four K-contiguous elements feed t = 0..3.
// An operand stored M/N-contiguous is read as vectors of one K row: element i
// of the vector at column MI * (lane & 15) feeds block i, so block i holds
// the columns MI * c + i.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace oscars {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

constexpr int SLICES = 4;  // K slices of forward / backward-data = waves per workgroup
constexpr int HEAD_SLICES = 8;  // of the classifier head
constexpr int KTILE = 32;  // K tile dealt to the slices in turn

template <int W> struct Vec;
template <> struct Vec<1> { typedef float T; };
template <> struct Vec<2> { typedef f32x2 T; };
template <> struct Vec<4> { typedef f32x4 T; };

// Lanes with nothing to load read these zeros (no branch around a load).
__device__ __attribute__((aligned(16))) float f32_zero[4];

// a * b elements in one instruction (rows and strides are below 2^31).
__device__ __forceinline__ int64_t offset_of(int a, int64_t b) {
  return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(a)) *
                              static_cast<uint32_t>(b));
}

// Keeps the loads issued before it above the products that follow: the
// scheduler otherwise moves them down to their first use, which then waits
// out the whole latency.
__device__ __forceinline__ void loads_first() { __builtin_amdgcn_sched_barrier(0); }

// Flattened workgroup id -> work item: the workgroups that the hardware puts
// on one XCD (id mod 8) take one contiguous range of the T work items.
__device__ __forceinline__ int xcd_item(int id, int T) {
  const int x = id & 7, i = id >> 3, q = T >> 3, r = T & 7;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// K groups (16 deep) a wave loads at once: enough bytes in flight for small
// tiles, few registers for large ones.  A slice is summed in whole pairs of
// such loads (zeros past K): with a test between the products the compiler
// sinks the loads of the next groups behind it, next to their use.
template <int MI, int NJ> struct Depth {
  static constexpr int G = MI + NJ >= 8 ? 1 : (MI + NJ >= 4 ? 2 : 4);
};

// The operands of G consecutive K groups of one slice.
template <bool TRANS, int MI, int NJ, int G, int S>
struct Frags {
  float a[G][MI][4], b[G][NJ][4];

  // a_row[i]: row of block i (K-contiguous), or, TRANS, a_row[0]: column
  // MI * (lane & 15) of K row 0; b_row[j]: row of block j (K-contiguous).
  // Slice `slice`, its K groups q0 .. q0 + G - 1; zeros from K (A) and from
  // b_ext (B) on.
  __device__ __forceinline__ void load(const float* const (&a_row)[MI],
                                       const float* const (&b_row)[NJ], int64_t a_ld, int K,
                                       int b_ext, int slice, int q0, int lane) {
    const int kq = 4 * (lane >> 4);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int q = q0 + g;
      const int k = KTILE * (slice + S * (q >> 1)) + 16 * (q & 1) + kq;
      if constexpr (!TRANS) {
        const bool ok = k < K;  // K is a multiple of 4: whole chunks
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(ok ? a_row[i] + k : f32_zero);
#pragma unroll
          for (int t = 0; t < 4; ++t) a[g][i][t] = v[t];
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float* row = a_row[0] + offset_of(k + t, a_ld);
          const float* p = k + t < K ? row : f32_zero;
          const typename Vec<MI>::T v = *reinterpret_cast<const typename Vec<MI>::T*>(p);
          if constexpr (MI == 1) a[g][0][t] = v;
          else {
#pragma unroll
            for (int i = 0; i < MI; ++i) a[g][i][t] = v[i];
          }
        }
      }
      const bool ok = k < b_ext;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(ok ? b_row[j] + k : f32_zero);
#pragma unroll
        for (int t = 0; t < 4; ++t) b[g][j][t] = v[t];
      }
    }
  }

  __device__ __forceinline__ void mma(f32x4 (&acc)[MI][NJ]) const {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[g][i][t], b[g][j][t], acc[i][j], 0,
                                                             0, 0);
    }
  }
};

// One K slice of a 16 MI x 16 NJ tile.
template <bool TRANS, int S, int MI, int NJ>
__device__ __forceinline__ void slice_products(f32x4 (&acc)[MI][NJ],
                                               const float* const (&a_row)[MI],
                                               const float* const (&b_row)[NJ], int64_t a_ld, int K,
                                               int b_ext, int slice, int lane) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int tiles = (K + KTILE - 1) / KTILE;
  const int nq = tiles > slice ? 2 * ((tiles - slice + S - 1) / S) : 0;
  constexpr int G = Depth<MI, NJ>::G;
  Frags<TRANS, MI, NJ, G, S> f0, f1;
  f0.load(a_row, b_row, a_ld, K, b_ext, slice, 0, lane);
  for (int q0 = 0; q0 < nq; q0 += 2 * G) {
    f1.load(a_row, b_row, a_ld, K, b_ext, slice, q0 + G, lane);
    loads_first();
    f0.mma(acc);
    f0.load(a_row, b_row, a_ld, K, b_ext, slice, q0 + 2 * G, lane);
    loads_first();
    f1.mma(acc);
  }
}

// Four consecutive rows m of quad `qd` (0 .. MI - 1) of a lane, and their
// first row within the tile: TRANS blocks interleave the columns.
template <bool TRANS, int MI, int NJ>
__device__ __forceinline__ f32x4 acc_quad(const f32x4 (&acc)[MI][NJ], int j, int qd) {
  if constexpr (!TRANS) return acc[qd][j];
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = acc[(4 * qd + e) % MI][j][(4 * qd + e) / MI];
  return v;
}
template <bool TRANS, int MI>
__device__ __forceinline__ int quad_row(int qd, int lane) {
  return TRANS ? 4 * MI * (lane >> 4) + 4 * qd : 16 * qd + 4 * (lane >> 4);
}

// Forward and backward-data (GemmArgs as for the other GEMM kernels, without
// rows_out and the split): one 16 MI x 16 NJ output tile per workgroup, one
// K slice per wave.
template <int MODE, int MI, int NJ>
__global__ __launch_bounds__(64 * SLICES) void f32_gemm_kernel(GemmArgs g) {
  constexpr bool TRANS = MODE == GEMM_DGRAD;
  // The slices meet in LDS, at most 32 columns at a time (64 x 64 tiles: two
  // phases of 70 KB).
  constexpr int TM = 16 * MI, TN = 16 * NJ, LD = TM + 4;
  constexpr int NP = NJ > 2 ? 2 : 1, PN = TN / NP;  // phases, columns per phase
  __shared__ __attribute__((aligned(16))) float red[SLICES][PN][LD];
  const int lane = threadIdx.x & 63;
  const int slice = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int work = xcd_item(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int z = work / gridDim.x, tile = work % gridDim.x;
  const int rep = g.order[z];
  const int gn = (g.N + TN - 1) / TN;
  const int m0 = tile / gn * TM, n0 = tile % gn * TN;
  const float* A = static_cast<const float*>(g.a) + (g.a_by_order ? rep : z) * g.a_slot;
  const float* B = static_cast<const float*>(g.b) + z * g.b_slot;

  // Rows past M or N repeat the last one: their outputs are never stored.
  const float *a_row[MI], *b_row[NJ];
  if constexpr (TRANS) {
    const int m = m0 + MI * (lane & 15);  // M is a multiple of 8
#pragma unroll
    for (int i = 0; i < MI; ++i) a_row[i] = A + (m < g.M ? m : 0);
  } else {
#pragma unroll
    for (int i = 0; i < MI; ++i)
      a_row[i] = A + static_cast<int64_t>(min(m0 + 16 * i + (lane & 15), g.M - 1)) * g.a_ld;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = min(n0 + 16 * j + (lane & 15), g.N - 1);
    const int64_t row = g.gather ? g.gather[z * g.gather_slot + n] : n;
    b_row[j] = B + row * g.b_ld;
  }
  f32x4 acc[MI][NJ];
  slice_products<TRANS, SLICES>(acc, a_row, b_row, g.a_ld, g.K, g.b_ext, slice, lane);

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
    if (ph > 0) __syncthreads();
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
template <int MI, bool DGRAD>
__global__ __launch_bounds__(64 * HEAD_SLICES) void f32_head_kernel(F32HeadArgs h) {
  constexpr int TM = 16 * MI, LD = TM + 4, ROWS = 16;
  __shared__ __attribute__((aligned(16))) float red[HEAD_SLICES][ROWS][LD];
  __shared__ __attribute__((aligned(16))) float dl[ROWS][LD];
  const int lane = threadIdx.x & 63, c16 = lane & 15, gq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int z = blockIdx.y, rep = h.order[z], n0 = blockIdx.x * ROWS;
  const float* master = h.master_in + static_cast<int64_t>(rep) * h.master_in_slot;
  const float* W = master + h.w_off;
  const float *a_row[MI], *b_row[1];
#pragma unroll
  for (int i = 0; i < MI; ++i)
    a_row[i] = W + static_cast<int64_t>(min(16 * i + c16, h.C - 1)) * h.K;
  const int nb = min(n0 + c16, h.B - 1);
  b_row[0] = h.act + z * h.act_slot +
             (h.act_gather ? static_cast<int64_t>(h.gather[z * h.gather_slot + nb])
                           : static_cast<int64_t>(nb)) * h.act_ld;
  // labels and bias before the products: their latency is hidden
  int label[ROWS / HEAD_SLICES];
#pragma unroll
  for (int r = 0; r < ROWS / HEAD_SLICES; ++r) {
    const int b = min(n0 + wave * (ROWS / HEAD_SLICES) + r, h.B - 1);
    label[r] = h.y[h.gather ? h.gather[z * h.gather_slot + b] : b];
  }
  const float bias = master[h.b_off + min(lane, h.C - 1)];
  f32x4 acc[MI][1];
  slice_products<false, HEAD_SLICES>(acc, a_row, b_row, h.K, h.K, h.K, wave, lane);
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
    for (int m0 = 64 * wave; m0 < h.K; m0 += 64 * HEAD_SLICES) {
      const int m = m0 + 4 * c16;
      const float* col = W + (m < h.K ? m : 0);
      f32x4 w[MI][4];
#pragma unroll
      for (int s = 0; s < MI; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int k = 16 * s + 4 * gq + t;
          w[s][t] = *reinterpret_cast<const f32x4*>(
              k < h.C ? col + static_cast<int64_t>(k) * h.K : f32_zero);
        }
      const int mo = m0 + 16 * gq;  // this lane's 16 outputs
      const int64_t at = static_cast<int64_t>(min(b, h.B - 1)) * h.act_ld;
      f32x4 mask[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        mask[r] = *reinterpret_cast<const f32x4*>(
            mo + 4 * r < h.K ? h.act + z * h.act_slot + at + mo + 4 * r : f32_zero);
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
            d[s >> 1][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][t][i], bd[s][t], d[s >> 1][i],
                                                                0, 0, 0);
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

// Backward-weight and the SGD update of every layer in one launch (nothing
// reads the weights after the last backward-data launch).  A workgroup of 2 x
// 2 waves covers 32 T inputs x 32 T outputs of one layer, a wave 16 T x 16 T:
// dW[o][i] over the batch, then W <- W - lr dW.  The biases have workgroups of
// their own (64 outputs each): blocks of 64 batch rows row by row, the block
// sums left to right.
constexpr int UPDATE_ROWS = 1024 + 80;  // largest batch and the groups read ahead
template <int T>
__global__ __launch_bounds__(256) void f32_update_kernel(F32UpdateArgs u) {
  __shared__ __attribute__((aligned(16))) int32_t rows[UPDATE_ROWS];  // of the activations
  __shared__ float bias_sum[16][64];  // of the blocks of 64 batch rows
  typedef typename Vec<T>::T V;
  const int lane = threadIdx.x & 63, c16 = lane & 15, gq = lane >> 4;
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
  for (int b = threadIdx.x; b < UPDATE_ROWS; b += 256)
    rows[b] = b >= u.B ? 0 : (gathered ? u.gather[z * u.gather_slot + b] : b);
  __syncthreads();
  if (tile >= y.tiles) {  // the biases of 64 outputs
    const int n = (tile - y.tiles) * 64 + lane, blocks = (u.B + 63) / 64;
    const float* D = y.d + z * y.d_slot + n;  // rows padded to 64
    for (int b = wave; b < blocks; b += 4) {
      float sum = 0.0f;
      for (int k = 64 * b; k < 64 * b + 64; k += 16) {
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = *(k + e < u.B ? D + offset_of(k + e, y.d_ld) : f32_zero);
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
  if (m0 >= y.M || n0 >= y.N) return;
  // Columns past M repeat column 0 (never stored); delta rows are padded to 64.
  const int ma = m0 + T * c16;
  const float* A = y.a + z * y.a_slot + (ma < y.M ? ma : 0);
  const float* D = y.d + z * y.d_slot + n0 + T * c16;
  float a[2][T][4], b[2][T][4];
  i32x4 row[2];  // of the group loaded next into each set
  auto load_rows = [&](int set, int s) {
    row[set] = *reinterpret_cast<const i32x4*>(&rows[16 * s + 4 * gq]);
  };
  auto load = [&](int set, int s) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 16 * s + 4 * gq + t;
      const float* pa = A + offset_of(row[set][t], y.a_ld);
      const float* pd = D + offset_of(k, y.d_ld);
      const V va = *reinterpret_cast<const V*>(k < u.B ? pa : f32_zero);
      const V vb = *reinterpret_cast<const V*>(k < u.B ? pd : f32_zero);
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
        for (int j = 0; j < T; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[set][i][t], b[set][j][t], acc[i][j], 0,
                                                           0, 0);
  };
  const int ns = (u.B + 15) / 16;
  load_rows(0, 0);
  load_rows(1, 1);
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
    const float* row = win + y.w_off + static_cast<int64_t>(n) * y.M;
#pragma unroll
    for (int qd = 0; qd < T; ++qd)
      w[j][qd] = *reinterpret_cast<const f32x4*>(mo + 4 * qd < y.M ? row + mo + 4 * qd : f32_zero);
  }
  for (int s = 0; s < ns; s += 2) {
    load_rows(0, s + 2);
    load(1, s + 1);
    loads_first();
    mma(0);
    load_rows(1, s + 3);
    load(0, s + 2);
    loads_first();
    mma(1);  // zeros past the batch
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

template <int MODE, int MI, int NJ>
hipError_t f32_gemm_launch(const GemmArgs& g, int n_slots, hipStream_t s) {
  const int64_t gx = static_cast<int64_t>((g.M + 16 * MI - 1) / (16 * MI)) *
                     ((g.N + 16 * NJ - 1) / (16 * NJ));
  if (gx * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((f32_gemm_kernel<MODE, MI, NJ>), dim3(static_cast<unsigned>(gx), n_slots),
                     dim3(64 * SLICES), 0, s, g);
  return hipGetLastError();
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
  if (h.C < 1 || h.C > F32_HEAD_CLASSES) return hipErrorInvalidValue;
  const dim3 grid((h.B + 15) / 16, n_slots), block(64 * HEAD_SLICES);
#define HEAD(mi)                                                                          \
  if (h.below) hipLaunchKernelGGL((f32_head_kernel<mi, true>), grid, block, 0, s, h);     \
  else hipLaunchKernelGGL((f32_head_kernel<mi, false>), grid, block, 0, s, h)
  if (h.C <= 16) { HEAD(1); }
  else if (h.C <= 32) { HEAD(2); }
  else { HEAD(4); }
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
  // (465 workgroups) 83 against 102 us.
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
