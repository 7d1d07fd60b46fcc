// Device helpers shared by the fp32 MFMA kernels whose waves fetch their own
// operands, without barriers in the K loop (f32_kernels.hip,
// conv_direct.hip).
//
// MFMA 16x16x4 (2048 flops in 32 cycles per SIMD): lane (c = lane & 15,
// q = lane >> 4) holds row c of A and column c of B at k = q, and rows 4 q ..
// 4 q + 3 of column c of the accumulator.  A K group is 16 deep: its MFMA t
// contracts k = 4 q + t over the lane groups q, so a lane's four K-contiguous
// elements feed t = 0..3.  An operand stored M/N-contiguous is read as
// vectors of one K row: element i of the vector at column I c feeds block i of
// I blocks, so block i holds the columns I c + i.
//
// The vector L1 takes a 16-byte load of a wave as quads of lanes: 16 accesses
// where four consecutive lanes read 64 contiguous bytes, 64 where they do
// not.  In MFMA layout a K-contiguous operand is the latter (consecutive
// lanes are consecutive rows), which bound these kernels by the L1 (93% of its
// cycles busy).  So such operands are loaded with four lanes per row and turned
// through LDS private to the wave: LDS operations of one wave execute in
// order, so there is no barrier and one buffer suffices.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace oscars {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

template <int W> struct Vec;
template <> struct Vec<1> { typedef float T; };
template <> struct Vec<2> { typedef f32x2 T; };
template <> struct Vec<4> { typedef f32x4 T; };

// W consecutive floats of global memory at p (aligned to their size).  The
// cast keeps the load a global one where p was chosen between an operand and
// zero_words(), whose address space the compiler cannot see.
template <int W>
__device__ __forceinline__ typename Vec<W>::T load_global(const float* p) {
  typedef const __attribute__((address_space(1))) typename Vec<W>::T* P;
  return *(P)p;
}
template <int W>
__device__ __forceinline__ void load_vec(float (&v)[W], const float* p) {
  const typename Vec<W>::T x = load_global<W>(p);
  if constexpr (W == 1) v[0] = x;
  else {
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = x[i];
  }
}

// Lanes with nothing to load read zeros from here (no branch around a load).
// The compiler must not see where the pointer leads: knowing both sides of the
// choice it loads the zeros apart, behind a branch that splits the K loop.
__device__ __attribute__((aligned(16))) float f32_zero_words[128];
__device__ __forceinline__ const float* zero_words() {
  const float* p = f32_zero_words;
  asm("" : "+v"(p));
  return p;
}

// a * b elements in one instruction (rows and strides are below 2^31).
__device__ __forceinline__ int64_t offset_of(int a, int64_t b) {
  return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(a)) *
                              static_cast<uint32_t>(b));
}

// Buffer loads: address = uniform base + per-lane byte offset + uniform byte
// offset, all but the per-lane part on the scalar unit; from `bytes` on they
// read zeros.  fp32 MFMA and vector arithmetic share the SIMD's multipliers:
// an MFMA with one vector instruction behind it took 40 cycles instead of 34,
// with four 60 (bf16 MFMA: 34 and 37), so the K loops keep their addresses
// scalar where they can.  NOWHERE is past every buffer (they are all smaller);
// the uniform offset stays within the buffer.
constexpr uint32_t NOWHERE = 0x80000000u;
typedef __amdgpu_buffer_rsrc_t Buf;
__device__ __forceinline__ Buf buffer(const float* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, static_cast<int>(bytes),
                                           0x00020000);
}
template <int W>
__device__ __forceinline__ typename Vec<W>::T load_buffer(Buf b, uint32_t at, uint32_t uniform) {
  typedef typename Vec<W>::T T;
  if constexpr (W == 1)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, at, uniform, 0));
  else if constexpr (W == 2)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, at, uniform, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(b, at, uniform, 0));
}
template <int W>
__device__ __forceinline__ void load_buffer_vec(float (&v)[W], Buf b, uint32_t at,
                                                uint32_t uniform) {
  const typename Vec<W>::T x = load_buffer<W>(b, at, uniform);
  if constexpr (W == 1) v[0] = x;
  else {
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = x[i];
  }
}

// Schedule of one part of a K loop: M products, the LDS writes (W), LDS reads
// (R) and loads (V) shared out behind them in that order.  Left alone the
// compiler moves the loads down to their first use, where the whole latency
// is waited out.
template <int M, int W, int R, int V>
__device__ __forceinline__ void spread() {
  constexpr int PER = (W + R + V + M - 1) / M;
#pragma unroll
  for (int u = 0; u < M; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
    for (int k = PER * u; k < PER * u + PER; ++k) {
      if (k < W) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      else if (k < W + R) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      else if (k < W + R + V) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Schedule of kernels with many products per load: all loads, then the
// products undisturbed.
__device__ __forceinline__ void loads_first() { __builtin_amdgcn_sched_barrier(0); }

// Flattened workgroup id -> work item: the workgroups that the hardware puts
// on one XCD (id mod 8) take one contiguous range of the T work items.
__device__ __forceinline__ int xcd_item(int id, int T) {
  const int x = id & 7, i = id >> 3, q = T >> 3, r = T & 7;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// A 16 x 16 block (rows x K) of a K-contiguous operand: loaded by lane l as
// elements 4 (l & 3) .. + 3 of row l >> 2, put into LDS with the 16-byte
// chunks of row r at c ^ (r >> 1 & 3) (neither side has bank conflicts), read
// back in MFMA layout.
constexpr int BLOCK_FLOATS = 256;
__device__ __forceinline__ int load_row(int lane) { return lane >> 2; }
__device__ __forceinline__ int load_k(int lane) { return 4 * (lane & 3); }
template <int NB>
__device__ __forceinline__ void blocks_write(float* lds, const f32x4 (&v)[NB], int lane) {
  float* at = lds + 16 * (lane >> 2) + (((lane & 3) ^ ((lane >> 3) & 3)) << 2);
#pragma unroll
  for (int b = 0; b < NB; ++b) *reinterpret_cast<f32x4*>(at + b * BLOCK_FLOATS) = v[b];
  __builtin_amdgcn_wave_barrier();  // the reads below stay below (other lanes' data)
}
template <int NB>
__device__ __forceinline__ void blocks_read(const float* lds, f32x4 (&v)[NB], int lane) {
  const int r = lane & 15;
  const float* at = lds + 16 * r + (((lane >> 4) ^ ((r >> 1) & 3)) << 2);
#pragma unroll
  for (int b = 0; b < NB; ++b) v[b] = *reinterpret_cast<const f32x4*>(at + b * BLOCK_FLOATS);
  __builtin_amdgcn_wave_barrier();  // the next writes stay below
}

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four consecutive rows m of quad `qd` (0 .. MI - 1) of a lane, and their
// first row within the tile; TRANS: A was stored M-contiguous, so its blocks
// interleave the rows.
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

}  // namespace
}  // namespace oscars
