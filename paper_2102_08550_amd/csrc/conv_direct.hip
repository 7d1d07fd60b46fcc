// 3 x 3 convolutions on fp32 MFMA for gfx950, channel counts multiples of 4:
// forward, backward-data and backward-weight as implicit GEMMs whose waves
// gather their own MFMA operands, a K group or two ahead of the products.
// fp32 MFMA is slow next to the vector caches (a 64 x 64 wave tile: 2048
// cycles of products per 16 K for 8 KB of operands), so sharing operands
// between waves through LDS gains nothing, and its barrier per K step left the
// matrix cores idle more than half of the time with one or two workgroups per
// CU.  The K loops have no barriers.
//
//   pass        M (A rows)          N (B columns)  K              A(m, k)         B(k, n)
//   CONV_FWD    Cout                output pixels  9 Cin          W[m][k]         input tap
//   CONV_DGRAD  Cin                 input pixels   taps x Cout    W[o][r][s][m]   output-gradient tap
//   CONV_WGRAD  9 Cin (tap, chan.)  Cout           output pixels  input tap       dZ[k][n]
//
// with k = (r 3 + s) Cin + c (the layout of W[o][3][3][c]) and likewise for
// Cout.  Backward-data of a stride-2 layer treats each parity class of the
// input pixels as a GEMM of its own with its one, two or four taps.  Every
// output of the forward and of backward-data is one K-order sum; backward-weight
// sums ranges of output pixels (four consecutive parts of a range by one
// wave each, added in order), one partial per range, which the update kernel
// adds in a fixed order.  So results depend on nothing but the inputs.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "conv.h"
#include "mfma_f32.h"

namespace oscars {
namespace {

// K groups loaded at once.
template <int MI, int NJ> struct Groups {
  static constexpr int G = MI + NJ >= 5 ? 1 : 2;
};
// Floats of a wave's LDS for the K-contiguous operands of a pixel tile.
template <int PASS, int MI, int NJ> constexpr int pixel_lds() {
  return Groups<MI, NJ>::G * ((PASS == CONV_FWD ? MI : 0) + NJ) * BLOCK_FLOATS;
}

// Stride-2 backward-data class `cls`: input rows 2 i + (cls >> 1), columns
// 2 j + (cls & 1); per dimension one tap (r = 1) for even, two (r = 0, 2) for
// odd positions.
__host__ __device__ inline int class_rows(const ConvArgs& a, int cls) {
  return (a.H - (cls >> 1) + 1) / 2;
}
__host__ __device__ inline int class_cols(const ConvArgs& a, int cls) {
  return (a.W - (cls & 1) + 1) / 2;
}
// the classes of a launch in workgroup order, the most taps first
__host__ __device__ inline int class_at(int i) { return i == 0 ? 3 : i == 1 ? 1 : i == 2 ? 2 : 0; }

// Pixels (N) of a forward or backward-data pass (class `cls`, or -1).
__host__ __device__ inline int pass_pixels(const ConvArgs& a, int pass, int cls) {
  if (pass == CONV_FWD) return a.B * a.Ho * a.Wo;
  return cls < 0 ? a.B * a.H * a.W : a.B * class_rows(a, cls) * class_cols(a, cls);
}

// Quotient and remainder by one divisor.  Exact for n < 2^21: (n + 1/2) / d is
// at least 1 / 2d from an integer, the product's error below n / d 2^-22.  (An
// integer division is some 35 vector instructions, and those of a tile's
// pixels took as long as a third of its products.)
struct Divisor {
  int d;
  float inv;
  __device__ explicit Divisor(int d_) : d(d_), inv(__builtin_amdgcn_rcpf(static_cast<float>(d_))) {}
  __device__ int operator()(int n, int& rem) const {
    const int q = static_cast<int>(fmaf(static_cast<float>(n), inv, 0.5f * inv));
    rem = n - __mul24(q, d);
    return q;
  }
};

// Positions of the pixels of a tile or range, counted from its first pixel n0
// (uniform): along the row, then down the image, so that each quotient is of a
// number below 2^21 (images have at most 4096 rows and columns) however many
// pixels an image has.
struct PixelWalk {
  int img0, i0, j0;  // of the first pixel
  Divisor by_col, by_row;
  __device__ PixelWalk(int n0, int rows, int cols) : by_col(cols), by_row(rows) {
    const int hw = rows * cols;
    img0 = n0 / hw;
    const int n = n0 - img0 * hw;
    i0 = __builtin_amdgcn_readfirstlane(n / cols);
    j0 = n - i0 * cols;
  }
  // image of pixel n0 + p, row i and column j in it
  __device__ int operator()(int p, int& i, int& j) const {
    const int down = by_col(j0 + p, j);
    return img0 + by_row(i0 + down, i);
  }
};

// The 3 x 3 taps (bit 3 r + s) around (h, w) that lie inside an H x W image;
// (h, w) itself does.
__device__ __forceinline__ uint32_t taps_inside(int h, int w, int H, int W) {
  const uint32_t s = (w > 0 ? 1u : 0u) | 2u | (w + 1 < W ? 4u : 0u);
  return (h > 0 ? s : 0u) | s << 3 | (h + 1 < H ? s << 6 : 0u);
}

// Forward (PASS = CONV_FWD) or backward-data of one wave's 16 MI x 16 NJ tile:
// rows m0 .. (output / input channels), pixels n0 .. of slot z.
//   UNI: the channels per tap are a multiple of 16, so a K group lies in one
//   tap and every address is a lane constant and a scalar; else each lane
//   follows its own (tap, channel).
//   GATHER (forward, not UNI): the images are dataset rows.
// An input tap outside its image is one bit per tap and pixel (taps past the
// last, past K, are outside): shifted to the top of the lane's offset it makes
// the load read zeros (NOWHERE).
template <int PASS, int MI, int NJ, bool UNI, bool GATHER>
__device__ __forceinline__ void conv_pixels_tile(const ConvArgs& a, int cls, int m0, int n0, int z,
                                                 int lane, float* lds) {
  constexpr bool FWD = PASS == CONV_FWD, TRANS = !FWD;
  static_assert(!GATHER || (FWD && !UNI), "gathered images: forward");
  const int c16 = lane & 15, gq = lane >> 4, lk = load_k(lane);
  const int rep = a.order[z];
  const int M = FWD ? a.Co : a.C, D = FWD ? a.C : a.Co;  // rows; channels per tap
  const int N = pass_pixels(a, PASS, cls);
  const int oddr = cls < 0 ? 0 : cls >> 1, oddc = cls < 0 ? 0 : cls & 1;
  const int K = (cls < 0 ? 9 : 1 << (oddr + oddc)) * D;
  const float* par = a.master_in + static_cast<int64_t>(rep) * a.master_in_slot;
  const float* W = par + a.w_off;
  const float* zero = GATHER ? zero_words() : nullptr;
  // the pixel grid of the tile, and the image that its taps read (PH x PW)
  const int rows = FWD ? a.Ho : cls < 0 ? a.H : class_rows(a, cls);
  const int cols = FWD ? a.Wo : cls < 0 ? a.W : class_cols(a, cls);
  const int PH = FWD ? a.H : a.Ho, PW = FWD ? a.W : a.Wo, st = FWD ? a.stride : 1;
  const float* src = FWD ? a.in + z * a.in_slot : a.dout + z * a.dout_slot;

  // Offsets are from the row of the tile's first pixel, moved back by a row and
  // a pixel (taps reach that far; a class's taps do not), so none is negative.
  const PixelWalk walk(n0, rows, cols);
  const int64_t base = (static_cast<int64_t>(walk.img0) * PH + st * walk.i0) * PW * D;
  const int back = cls < 0 ? (PW + 1) * D : 0;
  const Buf px = buffer(src + base - back, 0x7FFFFFFF);
  uint32_t at[NJ];    // byte offset of the tap at the centre (UNI: and this lane's channels)
  uint32_t out_of[NJ];  // bit t: tap t lies outside
  const float* ptr[NJ];  // GATHER: the centre
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = n0 + 16 * j + load_row(lane), nc = min(n, N - 1);
    int pi, pj;
    const int img = walk(nc - n0, pi, pj);
    uint32_t ok = 0;
    if (cls < 0) {
      ok = taps_inside(st * pi, st * pj, PH, PW);
      if (!FWD) ok = __builtin_bitreverse32(ok) >> 23;  // tap t reads around at 8 - t
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {  // tap (tr, ts) reads dZ (i + (odd and tr = 0), j + ...)
        const int tr = t >> oddc, ts = t - (tr << oddc);
        const int h = pi + (oddr & (tr == 0 ? 1 : 0)), w = pj + (oddc & (ts == 0 ? 1 : 0));
        ok |= static_cast<uint32_t>((t < (1 << (oddr + oddc))) & (h < PH) & (w < PW)) << t;
      }
    }
    out_of[j] = n < N ? ~ok : ~0u;
    if constexpr (GATHER) {
      ptr[j] = a.in + static_cast<int64_t>(a.gather[z * a.gather_slot + img]) * a.in_ld +
               (st * pi * PW + st * pj) * D - back;
    } else {
      const int64_t off = (static_cast<int64_t>(img) * PH + st * pi) * PW * D + st * pj * D - base;
      at[j] = 4u * (static_cast<uint32_t>(off) + (UNI ? lk : 0));
    }
  }
  // Weights: forward, K-contiguous rows (past M a valid one again: not stored);
  // backward-data, M-contiguous.
  uint32_t w_at[FWD ? MI : 4];
  const Buf w_rows = buffer(W + static_cast<int64_t>(m0) * 9 * a.C, 0x7FFFFFFF);
  if constexpr (FWD) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
      w_at[i] = 4u * (static_cast<uint32_t>(min(16 * i + load_row(lane), M - 1 - m0)) * (9 * a.C) + lk);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w_at[e] = 4u * (((UNI ? 4 * gq : 0) + e) * (9 * a.C) + MI * c16);
  }

  constexpr int G = Groups<MI, NJ>::G;
  constexpr int AB = FWD ? MI : 0, NB = G * (AB + NJ);  // blocks through LDS
  // A K position: tap t, channel c, stepped by 16 per group.  UNI: of the whole
  // group (scalar); else this lane's.
  struct Pos {
    int t, c;
  };
  const int dt = 16 / D, dc = 16 - dt * D;
  auto start = [&](int k) { return Pos{k / D, k - k / D * D}; };
  auto step = [&](Pos& p) {
    p.c += UNI ? 16 : dc;
    if (!UNI) p.t += dt;
    const bool wrap = p.c >= D;
    p.c = wrap ? p.c - D : p.c;
    p.t = wrap ? p.t + 1 : p.t;
  };
  // offset of tap t from the (moved) centre, in pixels; its place in the weights
  auto tap_at = [&](int t) {
    if (cls < 0) {
      const int r = t / 3, s = t - 3 * r;
      return FWD ? r * PW + s : (2 - r) * PW + 2 - s;
    }
    const int tr = t >> oddc, ts = t - (tr << oddc);
    return (oddr & (tr == 0 ? 1 : 0)) * PW + (oddc & (ts == 0 ? 1 : 0));
  };
  auto weight_tap = [&](int t) {
    if (cls < 0) return t;
    const int tr = t >> oddc, ts = t - (tr << oddc);
    return 3 * (oddr ? 2 * tr : 1) + (oddc ? 2 * ts : 1);
  };
  Pos pr = UNI ? Pos{0, 0} : start(lk), pc = UNI ? Pos{0, 0} : start(4 * gq);
  int kr = 0;  // K of the next rows' group
  f32x4 raw[NB];
  auto load_rows = [&]() {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if constexpr (FWD) {
        const uint32_t k4 = 4u * min(kr, K);
        const bool in = UNI ? kr < K : lk < K - kr;
        const Buf b = UNI ? buffer(W + static_cast<int64_t>(m0) * 9 * a.C, in ? 0x7FFFFFFF : 0) : w_rows;
#pragma unroll
        for (int i = 0; i < AB; ++i)
          raw[g * (AB + NJ) + i] = load_buffer<4>(b, UNI || in ? w_at[i] : NOWHERE, UNI && !in ? 0 : k4);
      }
      const int tap = tap_at(pr.t);
      const uint32_t off = 4u * (tap * D + pr.c);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f32x4& v = raw[g * (AB + NJ) + AB + j];
        const uint32_t gone = out_of[j] << (31 - (UNI ? pr.t : min(pr.t, 31)));  // top bit: outside
        if constexpr (GATHER) {
          const float* p = ptr[j] + (tap * D + pr.c);
          v = load_global<4>(static_cast<int32_t>(gone) < 0 ? zero : p);
        } else if constexpr (UNI) {
          v = load_buffer<4>(px, (gone & NOWHERE) | at[j], min(off, 0x7FFFFFFFu));
        } else {
          v = load_buffer<4>(px, (gone & NOWHERE) | (at[j] + off), 0);
        }
      }
      kr += 16;
      step(pr);
    }
  };
  struct Set {
    f32x4 rows[NB];
    float cols[TRANS ? G : 1][TRANS ? MI : 1][4];
  } f0, f1;
  auto load_cols = [&](Set& f) {
    if constexpr (TRANS) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const bool in = pc.t * D + pc.c < K;
        const int wt = weight_tap(pc.t);
        if constexpr (UNI) {
          const Buf b = buffer(W + (static_cast<int64_t>(pc.c) * 9 + wt) * a.C + m0,
                               in ? (15 * 9 * a.C + a.C - m0) * 4 : 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v[MI];
            load_buffer_vec<MI>(v, b, w_at[e], 0);
#pragma unroll
            for (int i = 0; i < MI; ++i) f.cols[g][i][e] = v[i];
          }
        } else {
          const Buf b = buffer(W + m0, (9LL * a.C * a.Co - m0) * 4);
          const uint32_t off = 4u * ((pc.c * 9 + wt) * a.C);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v[MI];
            load_buffer_vec<MI>(v, b, in ? w_at[e] + off : NOWHERE, 0);
#pragma unroll
            for (int i = 0; i < MI; ++i) f.cols[g][i][e] = v[i];
          }
        }
        step(pc);
      }
    }
  };
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto mma = [&](const Set& f) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            float w;
            if constexpr (TRANS) w = f.cols[g][i][e];
            else w = f.rows[g * (AB + NJ) + i][e];
            acc[i][j] = mfma16(w, f.rows[g * (AB + NJ) + AB + j][e], acc[i][j]);
          }
  };
  // Loads of group q + 2, the turn through LDS of q + 1 and the products of q
  // in flight together (zeros past K).
  constexpr int NM = 4 * G * MI * NJ, NV = NB + (TRANS ? 4 * G : 0);
  const int ng = (K + 15) / 16;
  load_rows();
  load_cols(f0);
  blocks_write(lds, raw, lane);
  load_rows();
  blocks_read(lds, f0.rows, lane);
  for (int q = 0; q < ng; q += 2 * G) {
    blocks_write(lds, raw, lane);
    load_rows();
    load_cols(f1);
    blocks_read(lds, f1.rows, lane);
    mma(f0);
    spread<NM, NB, NB, NV>();
    blocks_write(lds, raw, lane);
    load_rows();
    load_cols(f0);
    blocks_read(lds, f0.rows, lane);
    mma(f1);
    spread<NM, NB, NB, NV>();
  }

#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    // this lane's output pixel of block j: the offset of its channel 0
    const int n = n0 + 16 * j + c16, nc = n < N ? n : N - 1;
    int out = nc * M;
    if (!FWD && cls >= 0) {
      int pi, pj;
      const int img = walk(nc - n0, pi, pj);
      out = ((img * a.H + 2 * pi + oddr) * a.W + 2 * pj + oddc) * a.C;
    }
    f32x4 v[MI], x[MI], y[MI];
#pragma unroll
    for (int qd = 0; qd < MI; ++qd) {  // loads of every quad first
      const int m = m0 + quad_row<TRANS, MI>(qd, lane), mc = m < M ? m : 0;
      v[qd] = acc_quad<TRANS>(acc, j, qd);
      x[qd] = *reinterpret_cast<const f32x4*>(
          FWD ? par + a.b_off + mc : a.mask + z * a.mask_slot + out + mc);
      y[qd] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (a.skip) y[qd] = *reinterpret_cast<const f32x4*>(a.skip + z * a.skip_slot + out + mc);
    }
#pragma unroll
    for (int qd = 0; qd < MI; ++qd) {
      const int m = m0 + quad_row<TRANS, MI>(qd, lane);
      if (n >= N || m >= M) continue;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (FWD) {
          float zv = v[qd][e] + x[qd][e];
          if (a.skip) zv += y[qd][e];
          o[e] = zv > 0.0f ? zv : 0.0f;
        } else {
          const float gv = a.skip ? v[qd][e] + y[qd][e] : v[qd][e];
          o[e] = x[qd][e] > 0.0f ? gv : 0.0f;
        }
      }
      *reinterpret_cast<f32x4*>(a.out + z * a.out_slot + out + m) = o;
    }
  }
}

constexpr int FWD_WAVES = 4;  // per workgroup: consecutive pixel tiles of the same channels
template <int MI, int NJ, bool UNI, bool GATHER>
__global__ __launch_bounds__(64 * FWD_WAVES, 2) void conv_fwd_direct_kernel(ConvArgs a) {
  __shared__ __attribute__((aligned(16))) float stage[FWD_WAVES][pixel_lds<CONV_FWD, MI, NJ>()];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int work = xcd_item(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int z = work / gridDim.x, tile = work % gridDim.x;
  const int gm = (a.Co + 16 * MI - 1) / (16 * MI);
  const int n0 = (tile / gm * FWD_WAVES + wave) * 16 * NJ;
  if (n0 >= a.B * a.Ho * a.Wo) return;
  conv_pixels_tile<CONV_FWD, MI, NJ, UNI, GATHER>(a, -1, tile % gm * 16 * MI, n0, z, lane, stage[wave]);
}

// Backward-weight of 64 weight columns (tap, channel) x 16 NJ output channels
// over one range of output pixels: four waves take consecutive quarters of
// the range, their sums are added in order through LDS.  (Eight waves filled a
// CU with one workgroup, whose table and final sum nothing overlapped: 32x32
// CNN of 128 channels at eight replicas 11.8 against 11.2 ms per round.)  The positions of the
// range's pixels (offset of the centre tap, one bit per tap inside) are
// tabled in LDS once.
constexpr int BWD_WAVES = 4;
constexpr int WG_RANGE = 1024;  // longest range
struct PixelPos {
  uint32_t at, out_of;  // byte offset of the moved centre; bit t: tap t lies outside
};
struct WgradLds {
  union {
    PixelPos table[WG_RANGE + 64];
    uint64_t far[WG_RANGE + 64];       // GATHER: element offset | taps inside << 48
    float red[BWD_WAVES][32][64 + 4];  // [wave][output channel][column]
    float stage[BWD_WAVES][4 * BLOCK_FLOATS];  // backward-data: each wave's own
  };
  float bias[BWD_WAVES][64];
};

template <int NJ, bool GATHER>
__device__ __forceinline__ void conv_weights_tile(const ConvArgs& a, int tile, int z, WgradLds& sm) {
  constexpr int MI = 4, NP = NJ == 4 ? 2 : 1;  // phases of the final sum
  const int lane = threadIdx.x & 63, c16 = lane & 15, gq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int C9 = 9 * a.C, gm = (C9 + 63) / 64, go = (a.Co + 16 * NJ - 1) / (16 * NJ);
  const int split = tile / (gm * go), rest = tile - split * gm * go;
  const int m0 = rest % gm * 64, o0 = rest / gm * 16 * NJ;
  const int K = a.B * a.Ho * a.Wo, R = static_cast<int>(a.k_per_split);
  const int kbeg = split * R, kend = min(K, kbeg + R);
  // Offsets from the input row of the range's first pixel, moved back as in
  // conv_pixels_tile.
  const PixelWalk walk(kbeg, a.Ho, a.Wo);
  const int64_t base = (static_cast<int64_t>(walk.img0) * a.H + a.stride * walk.i0) * a.W * a.C;
  const int back = (a.W + 1) * a.C;
  for (int p = threadIdx.x; p < R + 64; p += 64 * BWD_WAVES) {
    int i, j;
    const int img = walk(min(p, K - 1 - kbeg), i, j);
    const int hi = a.stride * i, wi = a.stride * j;
    uint32_t ok = taps_inside(hi, wi, a.H, a.W);
    if (kbeg + p >= kend) ok = 0;
    if constexpr (GATHER) {
      const int64_t img_at = static_cast<int64_t>(a.gather[z * a.gather_slot + img]) * a.in_ld;
      sm.far[p] = static_cast<uint64_t>(ok) << 48 | static_cast<uint64_t>(img_at + (hi * a.W + wi) * a.C);
    } else {
      const int64_t off = (static_cast<int64_t>(img) * a.H + hi) * a.W * a.C + wi * a.C - base;
      sm.table[p] = {4u * static_cast<uint32_t>(off), ~ok};
    }
  }
  __syncthreads();

  // This lane's four columns: one tap, or (past 9 Cin) a tap that no pixel has.
  const int m = m0 + 4 * c16, tap = m < C9 ? m / a.C : 31, ch = m < C9 ? m - tap * a.C : 0;
  const float* in = a.in + z * a.in_slot;
  const float* zero = GATHER ? zero_words() : nullptr;
  const Buf px = buffer(in + base - back, 0x7FFFFFFF);
  const int tap_off = m < C9 ? (tap / 3 * a.W + tap % 3) * a.C + ch : 0;
  const uint32_t tap_at = 4u * tap_off, to_top = 31 - tap;
  const float* in_tap = in + tap_off - back;
  const float* dz = a.dout + z * a.dout_slot + o0;
  uint32_t d_at[4];  // channels past Cout: other pixels' values (not stored)
#pragma unroll
  for (int t = 0; t < 4; ++t) d_at[t] = 4u * ((4 * gq + t) * a.Co + NJ * c16);
  const int part_len = R / BWD_WAVES, p0 = wave * part_len;
  struct Set {
    float a[MI][4], b[NJ][4];
  } f0, f1;
  struct Pos {
    PixelPos e[4];
    uint64_t far[GATHER ? 4 : 1];
  } e0, e1;
  auto look = [&](Pos& e, int s) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int p = p0 + 16 * s + 4 * gq + t;
      if constexpr (GATHER) e.far[t] = sm.far[p];
      else e.e[t] = sm.table[p];
    }
  };
  auto load = [&](Set& f, const Pos& e, int s) {
    const int k = min(kbeg + p0 + 16 * s, kend), n = min(kend - k, 16);
    const Buf db = buffer(dz + static_cast<int64_t>(k) * a.Co, n > 0 ? (n * a.Co - o0) * 4 : 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float va[MI], vb[NJ];
      if constexpr (GATHER) {
        const uint32_t in_bits = static_cast<uint32_t>(e.far[t] >> 48);
        const float* p = in_tap + static_cast<int64_t>(e.far[t] & 0xFFFFFFFFFFFFull);
        load_vec<MI>(va, (in_bits >> tap & 1) ? p : zero);
      } else {
        load_buffer_vec<MI>(va, px, (e.e[t].out_of << to_top & NOWHERE) | (e.e[t].at + tap_at), 0);
      }
      load_buffer_vec<NJ>(vb, db, d_at[t], 0);
#pragma unroll
      for (int i = 0; i < MI; ++i) f.a[i][t] = va[i];
#pragma unroll
      for (int j = 0; j < NJ; ++j) f.b[j][t] = vb[j];
    }
  };
  f32x4 acc[MI][NJ];
  float db[NJ];  // bias gradient of the lane's channels over its pixels
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    db[j] = 0.0f;
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  auto mma = [&](const Set& f) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma16(f.a[i][t], f.b[j][t], acc[i][j]);
  };
  const bool with_bias = m0 == 0;
  auto add_bias = [&](const Set& f) {
    if (!with_bias) return;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < NJ; ++j) db[j] += f.b[j][t];
  };
  // the wave's own part: whole pairs of groups, at least one (R is a multiple of
  // 128).  (Tested before the first pair too, a round of the 32x32 CNN of 128
  // channels took 2312 us instead of 2301.)
  const int ng = part_len / 16;
  constexpr int RD = 2;  // LDS reads of four table entries
  look(e0, 0);
  look(e1, 1);
  load(f0, e0, 0);
  int s = 0;
  do {
    look(e0, s + 2);
    load(f1, e1, s + 1);
    mma(f0);
    spread<16 * NJ, 0, RD, 8>();
    add_bias(f0);
    look(e1, s + 3);
    load(f0, e0, s + 2);
    mma(f1);
    spread<16 * NJ, 0, RD, 8>();
    add_bias(f1);
    s += 2;
  } while (s < ng);

  // The waves' sums, added in order; a thread takes four consecutive
  // columns of one output channel.
  const int64_t MW = static_cast<int64_t>(a.Co) * C9;
  float* part = a.part + z * a.part_slot + split * (MW + a.Co);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    db[j] += __shfl_xor(db[j], 16);
    db[j] += __shfl_xor(db[j], 32);
    if (gq == 0) sm.bias[wave][NJ * c16 + j] = db[j];
  }
#pragma unroll
  for (int ph = 0; ph < NP; ++ph) {
    __syncthreads();  // the table, or the previous phase, is read
#pragma unroll
    for (int jj = 0; jj < NJ / NP; ++jj)
#pragma unroll
      for (int qd = 0; qd < MI; ++qd)
        *reinterpret_cast<f32x4*>(&sm.red[wave][16 * jj + c16][quad_row<true, MI>(qd, lane)]) =
            acc_quad<true>(acc, ph * (NJ / NP) + jj, qd);
    __syncthreads();
    const int col = 4 * (threadIdx.x & 15);
#pragma unroll
    for (int row = threadIdx.x >> 4; row < 16 * (NJ / NP); row += 4 * BWD_WAVES) {
      const int oo = o0 + NJ * (row & 15) + ph * (NJ / NP) + (row >> 4);
      if (oo >= a.Co || m0 + col >= C9) continue;
      f32x4 v = *reinterpret_cast<const f32x4*>(&sm.red[0][row][col]);
#pragma unroll
      for (int w = 1; w < BWD_WAVES; ++w)
        v = v + *reinterpret_cast<const f32x4*>(&sm.red[w][row][col]);
      *reinterpret_cast<f32x4*>(part + static_cast<int64_t>(oo) * C9 + m0 + col) = v;
    }
  }
  if (m0 == 0 && threadIdx.x < 16 * NJ && o0 + static_cast<int>(threadIdx.x) < a.Co) {
    float v = sm.bias[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < BWD_WAVES; ++w) v += sm.bias[w][threadIdx.x];
    part[MW + o0 + threadIdx.x] = v;
  }
}

// Backward-weight alone, of a first layer, whose images are dataset rows.
template <int WJ>
__global__ __launch_bounds__(64 * BWD_WAVES, 2) void conv_wgrad_direct_kernel(ConvArgs w) {
  __shared__ __attribute__((aligned(16))) WgradLds sm;
  conv_weights_tile<WJ, true>(w, xcd_item(blockIdx.x, gridDim.x), blockIdx.y, sm);
}

// Backward-data of d (workgroups below nd) and backward-weight
// of w in one launch: both read the layer's output gradient, neither reads
// what the other writes, and together they fill CUs that either leaves idle
// with one or two replicas.
template <int MI, int NJ, int WJ, bool UNI>
__global__ __launch_bounds__(64 * BWD_WAVES, 2) void conv_bwd_direct_kernel(ConvArgs d, ConvArgs w,
                                                                         int nd) {
  __shared__ __attribute__((aligned(16))) WgradLds sm;
  // Within each kind of work (and each class below) the workgroups of one XCD
  // take neighbouring tiles; over all of the launch they would take one kind
  // each, and the XCDs with the long ones would finish last.
  const int z = blockIdx.y;
  int tile = blockIdx.x;
  if (tile >= nd) {
    conv_weights_tile<WJ, false>(w, xcd_item(tile - nd, gridDim.x - nd), z, sm);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int gm = (d.C + 16 * MI - 1) / (16 * MI);
  constexpr int PX = 16 * NJ * BWD_WAVES;  // pixels per workgroup
  int cls = -1, tiles = nd;
  if (d.stride == 2) {
    for (int i = 0; i < 4; ++i) {
      cls = class_at(i);
      tiles = (pass_pixels(d, CONV_DGRAD, cls) + PX - 1) / PX * gm;
      if (tile < tiles) break;
      tile -= tiles;
    }
  }
  tile = xcd_item(tile, tiles);
  const int n0 = (tile / gm * BWD_WAVES + wave) * 16 * NJ;
  if (n0 >= pass_pixels(d, CONV_DGRAD, cls)) return;
  static_assert(pixel_lds<CONV_DGRAD, MI, NJ>() <= 4 * BLOCK_FLOATS, "a wave's stage");
  conv_pixels_tile<CONV_DGRAD, MI, NJ, UNI, false>(d, cls, tile % gm * 16 * MI, n0, z, lane, sm.stage[wave]);
}

// Wave tile of a pixel pass with M channels: 64, 32 or 16 channels by 64
// pixels, 32 where that leaves fewer than two waves per SIMD.
struct PixelTile {
  int mi, nj;
};
PixelTile pixel_tile(int M, int64_t pixels, int n_slots) {
  PixelTile t{M > 32 ? 4 : M > 16 ? 2 : 1, 4};
  auto waves = [&] {
    return static_cast<int64_t>((M + 16 * t.mi - 1) / (16 * t.mi)) *
           ((pixels + 16 * t.nj - 1) / (16 * t.nj)) * n_slots;
  };
  const int64_t simds = 1024;
  if (waves() < 2 * simds) t.nj = 2;
  if (t.mi == 4 && waves() < simds) t.mi = 2;
  return t;
}

int64_t dgrad_groups(const ConvArgs& d, const PixelTile& t) {
  const int64_t gm = (d.C + 16 * t.mi - 1) / (16 * t.mi), px = 16 * t.nj * BWD_WAVES;
  if (d.stride != 2) return (pass_pixels(d, CONV_DGRAD, -1) + px - 1) / px * gm;
  int64_t n = 0;
  for (int c = 0; c < 4; ++c) n += (pass_pixels(d, CONV_DGRAD, c) + px - 1) / px * gm;
  return n;
}

template <int MI, int NJ, bool UNI>
void bwd_launch(const dim3& grid, hipStream_t s, const ConvArgs& d, const ConvArgs& w, int nd) {
  const dim3 block(64 * BWD_WAVES);
  if (w.Co > 32)
    hipLaunchKernelGGL((conv_bwd_direct_kernel<MI, NJ, 4, UNI>), grid, block, 0, s, d, w, nd);
  else if (w.Co > 16)
    hipLaunchKernelGGL((conv_bwd_direct_kernel<MI, NJ, 2, UNI>), grid, block, 0, s, d, w, nd);
  else
    hipLaunchKernelGGL((conv_bwd_direct_kernel<MI, NJ, 1, UNI>), grid, block, 0, s, d, w, nd);
}

void wgrad_launch(const dim3& grid, hipStream_t s, const ConvArgs& w) {
  const dim3 block(64 * BWD_WAVES);
  if (w.Co > 32) hipLaunchKernelGGL(conv_wgrad_direct_kernel<4>, grid, block, 0, s, w);
  else if (w.Co > 16) hipLaunchKernelGGL(conv_wgrad_direct_kernel<2>, grid, block, 0, s, w);
  else hipLaunchKernelGGL(conv_wgrad_direct_kernel<1>, grid, block, 0, s, w);
}

}  // namespace

// Byte offsets below 2^31: those of a tile from its first pixel's row (the taps of
// 1024 output pixels of W-wide images, stride 2, span at most 4096 + 5 W pixels,
// of at most 65536 channels), and those in a layer's weights where a K group is
// not one tap's (backward-data, output channels no multiple of 16).
bool conv_direct(const ConvArgs& a) {
  return (a.C & 3) == 0 && (a.Co & 3) == 0 && a.C >= 4 &&
         static_cast<int64_t>(a.W) * a.C <= (1 << 25) && static_cast<int64_t>(a.Wo) * a.Co <= (1 << 25) &&
         (a.Co % 16 == 0 || 9LL * a.C * a.Co < (1 << 29));
}

int conv_direct_range(const ConvArgs& a) {
  // 1024 pixels (256 per wave): long enough that the partials are a small part
  // of the traffic; shorter where the layer has few pixels, so that it still
  // gives 16 ranges.  Layers with a tile per CU in one range have enough with
  // 256 pixels, and their partials, a copy of the weights per range, are large:
  // 512 to 512 channels on 8 x 8 images, batch 16, a round at four replicas with
  // 128 and 256 pixels 4.38 and 3.92 ms, at one 2.57 and 2.57.
  const int64_t pixels = static_cast<int64_t>(a.B) * a.Ho * a.Wo;
  const int64_t tiles = static_cast<int64_t>((9 * a.C + 63) / 64) * ((a.Co + 63) / 64);
  const int shortest = tiles < 256 || pixels <= 128 ? 128 : 256;
  int r = WG_RANGE;
  while (r > shortest && pixels < 16LL * r) r /= 2;
  return r;
}

hipError_t launch_conv_direct_fwd(const ConvArgs& a, int n_slots, hipStream_t s) {
  if (!conv_direct(a) || n_slots < 1 || a.B < 1) return hipErrorInvalidValue;
  const int64_t pixels = static_cast<int64_t>(a.B) * a.Ho * a.Wo;
  PixelTile t = pixel_tile(a.Co, pixels, n_slots);
  const bool uni = a.C % 16 == 0 && !a.gather;
  if (!uni) t.nj = 2;
  const int64_t px = 16 * t.nj * FWD_WAVES;
  const int64_t gx = (pixels + px - 1) / px * ((a.Co + 16 * t.mi - 1) / (16 * t.mi));
  if (gx * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(gx), n_slots), block(64 * FWD_WAVES);
#define FWD(mi, nj, un, ga) hipLaunchKernelGGL((conv_fwd_direct_kernel<mi, nj, un, ga>), grid, block, 0, s, a)
  if (uni) {
    if (t.mi == 4 && t.nj == 4) FWD(4, 4, true, false);
    else if (t.mi == 4) FWD(4, 2, true, false);
    else if (t.mi == 2 && t.nj == 4) FWD(2, 4, true, false);
    else if (t.mi == 2) FWD(2, 2, true, false);
    else if (t.nj == 4) FWD(1, 4, true, false);
    else FWD(1, 2, true, false);
  } else if (a.gather) {
    if (t.mi == 4) FWD(4, 2, false, true);
    else if (t.mi == 2) FWD(2, 2, false, true);
    else FWD(1, 2, false, true);
  } else {
    if (t.mi == 4) FWD(4, 2, false, false);
    else if (t.mi == 2) FWD(2, 2, false, false);
    else FWD(1, 2, false, false);
  }
#undef FWD
  return hipGetLastError();
}

hipError_t launch_conv_direct_bwd(const ConvArgs* d, const ConvArgs& w, int n_slots, hipStream_t s) {
  if (!conv_direct(w) || n_slots < 1 || w.B < 1 || w.k_per_split < 128 ||
      w.k_per_split > WG_RANGE || w.k_per_split % 128 != 0 ||
      static_cast<int64_t>(w.splits) * w.k_per_split < static_cast<int64_t>(w.B) * w.Ho * w.Wo ||
      (d != nullptr) == (w.gather != nullptr))  // a first layer, or a pair
    return hipErrorInvalidValue;
  const int nj = w.Co > 32 ? 4 : w.Co > 16 ? 2 : 1;
  const int64_t nw = static_cast<int64_t>((9 * w.C + 63) / 64) * ((w.Co + 16 * nj - 1) / (16 * nj)) *
                     w.splits;
  if (!d) {
    if (nw * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(nw), n_slots);
    wgrad_launch(grid, s, w);
    return hipGetLastError();
  }
  PixelTile t = pixel_tile(d->C, static_cast<int64_t>(d->B) * d->H * d->W, n_slots);
  const bool uni = d->Co % 16 == 0;
  if (!uni) t.nj = 2;
  const int64_t nd = dgrad_groups(*d, t);
  if ((nd + nw) * n_slots > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(nd + nw), n_slots);
  const int n = static_cast<int>(nd);
  if (uni) {
    if (t.mi == 4 && t.nj == 4) bwd_launch<4, 4, true>(grid, s, *d, w, n);
    else if (t.mi == 4) bwd_launch<4, 2, true>(grid, s, *d, w, n);
    else if (t.mi == 2 && t.nj == 4) bwd_launch<2, 4, true>(grid, s, *d, w, n);
    else if (t.mi == 2) bwd_launch<2, 2, true>(grid, s, *d, w, n);
    else if (t.nj == 4) bwd_launch<1, 4, true>(grid, s, *d, w, n);
    else bwd_launch<1, 2, true>(grid, s, *d, w, n);
  } else {
    if (t.mi == 4) bwd_launch<4, 2, false>(grid, s, *d, w, n);
    else if (t.mi == 2) bwd_launch<2, 2, false>(grid, s, *d, w, n);
    else bwd_launch<1, 2, false>(grid, s, *d, w, n);
  }
  return hipGetLastError();
}

}  // namespace oscars
