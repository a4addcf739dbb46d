// Learned pilot: a six-layer 3x3 convolutional network (2 -> 32 -> ... -> 32
// -> 1 channels, ReLU after the first five, residual output pilot = z - f)
// that stands in for stage 1 as the estimate driving the Wiener stage.
//
// All activations are bfloat16 NHWC with 32 channels (64 B per pixel; the
// two input channels and the single output channel are zero-padded), so every
// layer is the same 32 -> 32 convolution.  A convolution is an implicit GEMM
// on the bf16 matrix cores: for each 16-pixel row segment and each of the 9
// taps, D[out channel][pixel] += W_tap[out][in] * X[in][pixel shifted by the
// tap] with v_mfma_f32_16x16x32_bf16 (K = the 32 input channels of one tap),
// fp32 accumulation, and a fused epilogue (bias + ReLU, or the residual
// output).  A layer's backward pass is one kernel: the input gradient is the same
// convolution with flipped, transposed weights and the ReLU mask, the weight
// gradient a GEMM over pixels (K = 32 pixels of a tile row per MFMA) into
// per-workgroup partial sums that a second kernel adds in a fixed order.
#include <hip/hip_runtime.h>

#include "common.h"
#include "pilot.h"

namespace gbm3d {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kC = 32;          // channels of every activation tensor
constexpr int kTaps = 9;
constexpr int kTileY = 8, kTileX = 32;
constexpr int kWmat = kTaps * kC * kC;   // one packed weight set per layer

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__host__ __device__ inline int conv_items(int N, int H, int W) {
  return N * ((H + kTileY - 1) / kTileY) * ((W + kTileX - 1) / kTileX);
}

// What a layer reads: an activation tensor, the network's input (channel 0 = z
// of the u16 image, channel 1 = sigma) or the loss gradient (channel 0, one bf16
// per pixel).  The last two are expanded to the eights of channels of an
// activation tensor where a kernel loads them; as such tensors they were 64 MB
// each for 64 images of 128^2, written once and read twice (77 us of 749 in a
// gradient step).
enum Source { kAct, kInput, kLossGrad };

// Channels 8 c8 .. 8 c8 + 7 of pixel `pix` as they lie in memory, and from that
// as activations of an image of noise level sigma (apart, so that loads can be
// in flight).
template <Source SRC>
__device__ __forceinline__ uint4 load_channels(const uint16_t* __restrict__ p, size_t pix, int c8) {
  if constexpr (SRC == kAct) return *reinterpret_cast<const uint4*>(p + pix * kC + 8 * c8);
  return make_uint4(c8 == 0 ? p[pix] : 0, 0, 0, 0);
}
template <Source SRC>
__device__ __forceinline__ uint4 as_activations(uint4 v, float sigma, int c8) {
  if constexpr (SRC == kInput) {
    if (c8 == 0) v.x = f2bf(static_cast<float>(v.x) * (1.0f / 65535.0f)) | (static_cast<uint32_t>(f2bf(sigma)) << 16);
  }
  return v;
}

// v0 as bf16 to out[0 .. 3], v1 to out[16 .. 19]
__device__ __forceinline__ void store_channels(uint16_t* __restrict__ out, const float (&v0)[4], const float (&v1)[4]) {
  auto pair = [](float a, float b) { return f2bf(a) | (static_cast<uint32_t>(f2bf(b)) << 16); };
  *reinterpret_cast<uint2*>(out) = make_uint2(pair(v0[0], v0[1]), pair(v0[2], v0[3]));
  *reinterpret_cast<uint2*>(out + 16) = make_uint2(pair(v1[0], v1[1]), pair(v1[2], v1[3]));
}

// ---------------------------------------------------------------------------
// convolution 32 -> 32, 3x3, zero "same" padding
// MODE 0: forward, + bias, ReLU, bf16 out
// MODE 1: forward last layer: f = channel 0 + bias; pilot = z - f (fp32 / u16)
// ---------------------------------------------------------------------------
template <int MODE, Source SRC>
__global__ __launch_bounds__(256) void conv_kernel(const uint16_t* __restrict__ in, const float* __restrict__ sigma,
                                                   const uint16_t* __restrict__ wpk,
                                                   const float* __restrict__ bias,
                                                   uint16_t* __restrict__ out, const uint16_t* __restrict__ noisy,
                                                   float* __restrict__ pilot_f32, uint16_t* __restrict__ pilot_u16,
                                                   int N, int H, int W) {
  __shared__ __align__(16) uint16_t tile[kTileY + 2][kTileX + 2][kC];
  const int tx_n = (W + kTileX - 1) / kTileX, ty_n = (H + kTileY - 1) / kTileY;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;

  // A operands (weights) for all taps, both 16-channel output halves
  bf16x8 A[kTaps][2];
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      A[t][h] = as_bf16x8(*reinterpret_cast<const uint4*>(wpk + (t * kC + h * 16 + col) * kC + 8 * grp));
  float b0[4], b1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    b0[i] = bias ? bias[4 * grp + i] : 0.0f;
    b1[i] = bias ? bias[16 + 4 * grp + i] : 0.0f;
  }

  const int total = conv_items(N, H, W);
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int n = item / (tx_n * ty_n);
    const int rem = item - n * tx_n * ty_n;
    const int y0 = (rem / tx_n) * kTileY, x0 = (rem % tx_n) * kTileX;
    uint4* dst_t = reinterpret_cast<uint4*>(&tile[0][0][0]);
    for (int i = threadIdx.x; i < (kTileY + 2) * (kTileX + 2) * 4; i += blockDim.x) {
      const int pix = i >> 2, part = i & 3;
      const int r = pix / (kTileX + 2), c = pix - r * (kTileX + 2);
      const int y = y0 - 1 + r, x = x0 - 1 + c;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (y >= 0 && y < H && x >= 0 && x < W)
        v = as_activations<SRC>(load_channels<SRC>(in, (static_cast<size_t>(n) * H + y) * W + x, part),
                                SRC == kInput ? sigma[n] : 0.0f, part);
      dst_t[i] = v;
    }
    __syncthreads();

#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
      const int row = 2 * wave + (bi >> 1), xoff = (bi & 1) * 16;
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < kTaps; ++t) {
        const int ky = t / 3, kx = t % 3;
        const bf16x8 B = as_bf16x8(*reinterpret_cast<const uint4*>(&tile[row + ky][xoff + col + kx][8 * grp]));
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t][0], B, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t][1], B, acc1, 0, 0, 0);
      }
      // lane holds channels 4*grp + i (acc0) and 16 + 4*grp + i (acc1) of pixel (y, x)
      const int y = y0 + row, x = x0 + xoff + col;
      if (y < H && x < W) {
        const size_t p = (static_cast<size_t>(n) * H + y) * W + x;
        if constexpr (MODE == 0) {
          float v0[4], v1[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v0[i] = fmaxf(acc0[i] + b0[i], 0.0f);
            v1[i] = fmaxf(acc1[i] + b1[i], 0.0f);
          }
          store_channels(out + p * kC + 4 * grp, v0, v1);
        } else {
          if (grp == 0) {  // channel 0 sits in acc0[0] of lanes 0..15
            const float f = acc0[0] + b0[0];
            const float pil = static_cast<float>(noisy[p]) * (1.0f / 65535.0f) - f;
            if (pilot_f32) pilot_f32[p] = pil;
            if (pilot_u16) {
              const double d = static_cast<double>(fminf(fmaxf(pil, 0.0f), 1.0f));
              pilot_u16[p] = static_cast<uint16_t>(floor(d * 65535.0 + 0.5));
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// fused inference: the six layers of one 16 x 32 output tile in one
// workgroup, every intermediate activation in LDS.  Layer l is evaluated on
// the tile grown by 5 - l pixels on each side (the receptive field of the
// layers after it), so a tile reads only its 28 x 44 window of the noisy
// image and writes only its pilot pixels.  Positions outside the image are
// zero in every layer's output, as the zero "same" padding of the per-layer
// form has them.
//
// One wave per SIMD, each software-pipelining its pixel blocks (the operands
// of the next block are read from LDS and the previous block's results
// written while the current block's products run); the next layer's weights
// are loaded into registers while the current layer computes.
//
// LDS: the input window as (z, sigma) bf16 pairs, and two ping-pong
// activation buffers (layers 0, 2, 4 | 1, 3) of 64 B per pixel.  A pixel's
// 16-byte octet o holds channels 4o .. 4o+3 and 16+4o .. 16+4o+3: exactly
// the eight values one lane holds after the products (output rows 4 grp + i
// of both 16-channel halves), so a lane writes its pixel's results with one
// 16-byte store, and the next layer takes its K dimension in that order (its
// A operands are gathered to match).  Octet o of a pixel in region column x
// sits at slot o ^ ((x >> 1) & 3): the eight consecutive pixels that one
// 128-byte LDS cycle of a 16-byte access serves then hit eight different
// 16-byte bank groups.  A layer's output pixels are taken in raster order,
// 16 per MFMA column block; layer 0 packs its 9 taps x 2 input channels into
// one K = 32 product, and layer 5 computes one 16-channel half (its single
// output channel is row 0).  Bias enters as the initial accumulator.  Lanes
// of a region's last block that fall past its end store into a spare pixel
// at the end of the buffer, so the stores need no branch.
// ---------------------------------------------------------------------------
constexpr int kFY = 16, kFX = 32;                   // output tile
constexpr int kFWaves = 4, kFThreads = 64 * kFWaves;
constexpr int kZY = kFY + 2 * kPilotLayers, kZX = kFX + 2 * kPilotLayers;  // input window
__host__ __device__ constexpr int f_ry(int l) { return kFY + 2 * (kPilotLayers - 1 - l); }
__host__ __device__ constexpr int f_rx(int l) { return kFX + 2 * (kPilotLayers - 1 - l); }
constexpr int kFBufA = f_ry(0) * f_rx(0), kFBufB = f_ry(1) * f_rx(1);  // pixels
static_assert(kFBufA >= f_ry(2) * f_rx(2) && kFBufB >= f_ry(3) * f_rx(3), "ping-pong sizes");
static_assert(kFX % 16 == 0, "output rows are whole 16-pixel blocks");

__host__ __device__ inline int fused_tiles(int N, int H, int W) {
  return N * ((H + kFY - 1) / kFY) * ((W + kFX - 1) / kFX);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));  // round to nearest even
}

// A operands of one layer (HALVES = 1: the first 16 output channels only)
template <int HALVES>
struct FusedW {
  bf16x8 A[kTaps][HALVES];
};

template <int HALVES>
__device__ __forceinline__ void fused_load_w(const uint16_t* __restrict__ wf, int l, int col, int grp,
                                             FusedW<HALVES>& w) {
  // global address space, and opaque to the optimiser, so the loads stay
  // where they are issued instead of being hoisted out of the tile loop (the
  // weights of all layers at once do not fit in the registers)
  typedef const uint16_t __attribute__((address_space(1))) * gptr;
  gptr wl = (gptr)(wf + static_cast<size_t>(l) * kWmat);
  asm volatile("" : "+s"(wl));
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
      // K element 8 grp + e is input channel 4 grp + e (e < 4) or 16 + 4 grp + e - 4
      gptr row = wl + (t * kC + h * 16 + col) * kC;
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      typedef const u32x2 __attribute__((address_space(1))) * gptr2;
      const u32x2 lo = *(gptr2)(row + 4 * grp);
      const u32x2 hi = *(gptr2)(row + 16 + 4 * grp);
      w.A[t][h] = as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
}

// ReLU (all zero when keep is false: outside the image), bf16, into octet
// grp of pixel i (region column c).  The ReLU acts on the rounded bf16 pairs
// as signed 16-bit maxima: rounding keeps the sign, so this equals rounding
// the ReLU of the float sums.
__device__ __forceinline__ void fused_store(uint4* __restrict__ out, int i, int c, int grp, f32x4 a0, f32x4 a1,
                                            bool keep) {
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  const s16x2 zero = {0, 0};
  uint32_t q[4] = {pack_bf16(a0[0], a0[1]), pack_bf16(a0[2], a0[3]), pack_bf16(a1[0], a1[1]), pack_bf16(a1[2], a1[3])};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    q[k] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, q[k]), zero));
    q[k] = keep ? q[k] : 0u;
  }
  out[i * 4 + (grp ^ ((c >> 1) & 3))] = make_uint4(q[0], q[1], q[2], q[3]);
}

// A 3x3 layer over a region of RY x RX pixels (input row stride RX + 2), two
// rows at a time: a block is 16 pixels of a row pair's raster, and its lanes'
// four input rows serve both rows' taps, 12 LDS reads and one address
// computation for 18 and two.  (No single unit binds: the one wave per SIMD
// issues its reads, addresses and epilogues between its products, and the LDS
// cycles of the reads were twice the products', now 1.5 times; 32 x 512^2
// 1.55 -> 1.38 ms.)  A wave takes the blocks g = wave, wave + kFWaves, ...: an operand
// that the block has no more use for is replaced by the next block's, and the
// results of a block are stored while the products of the next run.
template <int RX, int RY, int HALVES, class Store>
__device__ __forceinline__ void fused_conv(const uint4* __restrict__ in, const FusedW<HALVES>& w, f32x4 b0, f32x4 b1,
                                           Store&& store) {
  static_assert(RY % 2 == 0, "row pairs");
  constexpr int S = RX + 2, NP = RY / 2 * RX, NG = (NP + 15) / 16;
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  int g = threadIdx.x >> 6;
  if (g >= NG) return;
  auto addr = [&](int gg, int (&e)[3]) {
    const int i = min(gg * 16 + col, NP - 1), r = i / RX, c = i - r * RX, pb = 2 * r * S + c;
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) e[kx] = (pb + kx) * 4 + (grp ^ (((c + kx) >> 1) & 3));
  };
  bf16x8 B[4][3];
  auto read = [&](const int (&e)[3], int row, int kx) { B[row][kx] = as_bf16x8(in[e[kx] + row * S * 4]); };
  struct Sums {
    f32x4 v[2][2];  // [row of the pair][half]
  };
  auto products = [&](bool more, const int (&e)[3]) {
    Sums a{{{b0, b1}, {b0, b1}}};
#pragma unroll
    for (int t = 0; t < kTaps; ++t) {
      const int ky = t / 3, kx = t % 3;
#pragma unroll
      for (int row = 0; row < 2; ++row)
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
          a.v[row][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.A[t][h], B[ky + row][kx], a.v[row][h], 0, 0, 0);
      if (more) {
        read(e, ky, kx);
        if (ky == 2) read(e, 3, kx);
      }
    }
    return a;
  };
  auto put = [&](int gg, const Sums& a) {
    const int i = gg * 16 + col, r = min(i, NP - 1) / RX, c = min(i, NP - 1) - r * RX;
#pragma unroll
    for (int row = 0; row < 2; ++row) store(2 * r + row, c, i < NP, a.v[row][0], a.v[row][1]);
  };
  int e[3];
  addr(g, e);
#pragma unroll
  for (int row = 0; row < 4; ++row)
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) read(e, row, kx);
  addr(min(g + kFWaves, NG - 1), e);
  Sums p = products(true, e);
  for (g += kFWaves; g + kFWaves < NG; g += kFWaves) {
    addr(g + kFWaves, e);
    const Sums a = products(true, e);
    put(g - kFWaves, p);
    p = a;
  }
  if (g < NG) {
    const Sums a = products(false, e);
    put(g - kFWaves, p);
    put(g, a);
  } else {
    put(g - kFWaves, p);
  }
}

// layers 1 .. 4: 32 -> 32, ReLU
template <int L, int DUMMY = (L & 1) ? kFBufB : kFBufA>
__device__ __forceinline__ void fused_mid(const uint4* __restrict__ in, uint4* __restrict__ out,
                                          const FusedW<2>& w, const f32x4* __restrict__ bias4, bool border, int y0,
                                          int x0, int H, int W) {
  constexpr int RX = f_rx(L), G = kPilotLayers - 1 - L;
  const int grp = (threadIdx.x & 63) >> 4;
  fused_conv<RX, f_ry(L), 2>(in, w, bias4[L * 8 + grp], bias4[L * 8 + 4 + grp],
                             [&](int r, int c, bool used, f32x4 a0, f32x4 a1) {
    bool keep = true;
    if (border) {
      const int y = y0 - G + r, x = x0 - G + c;
      keep = static_cast<unsigned>(y) < static_cast<unsigned>(H) && static_cast<unsigned>(x) < static_cast<unsigned>(W);
    }
    fused_store(out, used ? r * RX + c : DUMMY, c, grp, a0, a1, keep);
  });
}

__global__ __launch_bounds__(kFThreads) void fused_infer_kernel(const uint16_t* __restrict__ noisy,
                                                                const float* __restrict__ sigma,
                                                                const uint16_t* __restrict__ wf,
                                                                const float* __restrict__ bias, int N, int H, int W,
                                                                float* __restrict__ pilot_f32,
                                                                uint16_t* __restrict__ pilot_u16) {
  __shared__ __align__(16) uint4 bufA[(kFBufA + 1) * 4];
  __shared__ __align__(16) uint4 bufB[(kFBufB + 1) * 4];
  __shared__ uint32_t zb[kZY * kZX];
  __shared__ uint16_t zc[2][kFY * kFX];  // the tile's own noisy pixels (exact), current / next tile
  __shared__ f32x4 bias4[kPilotLayers * 8];  // [layer][half * 4 + grp]: output channels 16 half + 4 grp + 0..3

  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  const int tx_n = (W + kFX - 1) / kFX, ty_n = (H + kFY - 1) / kFY;
  const int total = fused_tiles(N, H, W);

  if (threadIdx.x < kPilotLayers * kC) {
    const int l = threadIdx.x / kC, ch = threadIdx.x % kC;
    bias4[l * 8 + ch / 4][ch % 4] = bias[l * kC + ch];
  }
  // layer 0 operands: K index 8 grp + e is tap (8 grp + e) / 2, input channel e % 2 (taps past 8 are zero)
  FusedW<2> w0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = (8 * grp + e) >> 1, ci = e & 1;
      w0.A[0][h][e] = t < kTaps ? __builtin_bit_cast(__bf16, wf[(t * kC + h * 16 + col) * kC + ci]) : __bf16(0.0f);
    }
  int zoff[4];  // window offset of the taps this lane's K octet holds (taps past 8: any finite entry)
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int t = 4 * grp + j;
    zoff[j] = t < kTaps ? (t / 3) * kZX + t % 3 : 0;
  }
  // the next layer's operands are loaded while the current layer computes
  FusedW<2> wa, wb;
  FusedW<1> w5;

  // the window of a tile: 28 x 44 (z, sigma) pairs, zero outside the image
  constexpr int kZPer = (kZY * kZX + kFThreads - 1) / kFThreads;
  uint32_t zr[kZPer];
  uint16_t cr[kZPer];
  auto fetch = [&](int item) {
    const int n = item / (tx_n * ty_n), rem = item - n * tx_n * ty_n;
    const int y0 = (rem / tx_n) * kFY - kPilotLayers, x0 = (rem % tx_n) * kFX - kPilotLayers;
    const uint32_t s = f2bf(sigma[n]);
    const uint16_t* src = noisy + static_cast<size_t>(n) * H * W;
#pragma unroll
    for (int k = 0; k < kZPer; ++k) {
      const int pix = threadIdx.x + k * kFThreads;
      const int r = pix / kZX, c = pix - r * kZX, y = y0 + r, x = x0 + c;
      uint16_t v = 0;
      const bool in = pix < kZY * kZX && y >= 0 && y < H && x >= 0 && x < W;
      if (in) v = src[static_cast<size_t>(y) * W + x];
      cr[k] = v;
      zr[k] = in ? (static_cast<uint32_t>(f2bf(static_cast<float>(v) * (1.0f / 65535.0f))) | (s << 16)) : 0u;
    }
  };
  auto park = [&](int buf) {
#pragma unroll
    for (int k = 0; k < kZPer; ++k) {
      const int pix = threadIdx.x + k * kFThreads;
      if (pix < kZY * kZX) {
        zb[pix] = zr[k];
        const int r = pix / kZX - kPilotLayers, c = pix % kZX - kPilotLayers;
        if (r >= 0 && r < kFY && c >= 0 && c < kFX) zc[buf][r * kFX + c] = cr[k];
      }
    }
  };

  int buf = 0;
  if (blockIdx.x < total) {
    fetch(blockIdx.x);
    park(0);
  }
  __syncthreads();
  for (int item = blockIdx.x; item < total; item += gridDim.x, buf ^= 1) {
    const int n = item / (tx_n * ty_n), rem = item - n * tx_n * ty_n;
    const int y0 = (rem / tx_n) * kFY, x0 = (rem % tx_n) * kFX;
    const bool border = y0 < kPilotLayers || x0 < kPilotLayers || y0 + kFY + kPilotLayers > H ||
                        x0 + kFX + kPilotLayers > W;

    fused_load_w(wf, 1, col, grp, wa);
    {  // layer 0: 2 -> 32 from the window, im2col over the K dimension; four blocks per step
      constexpr int RX = f_rx(0), NP = f_ry(0) * RX, NG = (NP + 15) / 16, G = kPilotLayers - 1;
      constexpr int kSteps = (NG + 4 * kFWaves - 1) / (4 * kFWaves);
      const f32x4 b0 = bias4[grp], b1 = bias4[4 + grp];
      const int wave = threadIdx.x >> 6;
      auto read = [&](int g) {
        const int i = min(g * 16 + col, NP - 1), r = i / RX, pb = r * kZX + (i - r * RX);
        return as_bf16x8(make_uint4(zb[pb + zoff[0]], zb[pb + zoff[1]], zb[pb + zoff[2]], zb[pb + zoff[3]]));
      };
      bf16x8 Bz[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) Bz[q] = read(wave + q * kFWaves);
      for (int st = 0; st < kSteps; ++st) {
        const int g0 = st * 4 * kFWaves + wave;
        f32x4 a0[4], a1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a0[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0.A[0][0], Bz[q], b0, 0, 0, 0);
          a1[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0.A[0][1], Bz[q], b1, 0, 0, 0);
          if (st + 1 < kSteps) Bz[q] = read(g0 + (4 + q) * kFWaves);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = (g0 + q * kFWaves) * 16 + col;
          if (i < NP) {
            const int r = i / RX, c = i - r * RX;
            bool keep = true;
            if (border) {
              const int y = y0 - G + r, x = x0 - G + c;
              keep = static_cast<unsigned>(y) < static_cast<unsigned>(H) &&
                     static_cast<unsigned>(x) < static_cast<unsigned>(W);
            }
            fused_store(bufA, i, c, grp, a0[q], a1[q], keep);
          }
        }
      }
    }
    __syncthreads();
    const int next = item + static_cast<int>(gridDim.x);
    if (next < total) fetch(next);  // in flight during layers 1 .. 4
    fused_load_w(wf, 2, col, grp, wb);
    fused_mid<1>(bufA, bufB, wa, bias4, border, y0, x0, H, W);
    __syncthreads();
    fused_load_w(wf, 3, col, grp, wa);
    fused_mid<2>(bufB, bufA, wb, bias4, border, y0, x0, H, W);
    __syncthreads();
    fused_load_w(wf, 4, col, grp, wb);
    fused_mid<3>(bufA, bufB, wa, bias4, border, y0, x0, H, W);
    __syncthreads();
    fused_load_w(wf, 5, col, grp, w5);
    fused_mid<4>(bufB, bufA, wb, bias4, border, y0, x0, H, W);
    if (next < total) park(buf ^ 1);  // the window buffer is free since layer 0
    __syncthreads();

    {  // layer 5: 32 -> 1 (row 0 of the first half), pilot = z - f
      const uint16_t* zcur = zc[buf];
      fused_conv<f_rx(5), f_ry(5), 1>(bufA, w5, bias4[5 * 8 + grp], bias4[5 * 8 + grp],
                                      [&](int r, int c, bool, f32x4 a0, f32x4) {
        const int y = y0 + r, x = x0 + c;
        if (grp == 0 && y < H && x < W) {
          const size_t p = (static_cast<size_t>(n) * H + y) * W + x;
          const float pil = static_cast<float>(zcur[r * kFX + c]) * (1.0f / 65535.0f) - a0[0];
          if (pilot_f32) pilot_f32[p] = pil;
          if (pilot_u16) {
            const double d = static_cast<double>(fminf(fmaxf(pil, 0.0f), 1.0f));
            pilot_u16[p] = static_cast<uint16_t>(floor(d * 65535.0 + 0.5));
          }
        }
      });
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// backward pass of a layer
// weight gradient: dW[t][ci][co] = sum_p x[p + off_t][ci] g[p][co], db[co] = sum_p g[p][co],
// as per-workgroup partials [grid][kWmat + kC]; with DX also the input gradient
// dx = (g convolved with the flipped, transposed weights) * (x > 0).
//
// The products of the weight gradient run over pixels, so both tensors are
// needed channel-major; a thread loads eight channels of eight pixels of a row,
// transposes them in registers (32 byte permutes) and stores eight 16-byte runs
// of pixels.  A wave owns 16 x 16 channels of all nine taps.  It goes down the
// tile's rows: an operand of x (eight pixels from column 8 grp on, and two more)
// gives the three column shifts in registers and meets the operands of the three
// rows of g it is a tap of, so a row is read from LDS once.  For the input
// gradient g's pixels are kept as they are too, each pixel's four 16-byte pieces
// permuted by its column so that eight lanes' reads of eight pixels fall on all
// banks, and a bit of every x for the mask (read from memory again, it would
// wait for the loads ahead).
// A tile's loads are in flight during the products of the one before.
// Bound by memory (both tensors with a tile's borders, and dx) and by the latency
// of eight waves per CU.  64 images of 128^2, us per 32 -> 32 layer: the weight
// gradient alone 86 with 2-byte stores into three shifted copies and two operand
// reads per product, 38 like this, and 43 for an input-gradient kernel beside it;
// together 71.  Both tensors read and one written once take 42 at the rate of a
// large copy.
// ---------------------------------------------------------------------------
constexpr int kXGroups = (kTileX + 2 + 7) / 8;          // eights of columns x0 - 1 .. : 5
constexpr int kXRow = 8 * kXGroups;
// channel pitch of 12 words modulo 32: eight lanes' 16-byte reads of eight
// channels fall on all banks; every eight channels start 8 words later, so that
// the stores of four lanes' eights of channels do too
constexpr int kXCh = (kTileY + 2) * kXRow + 8;
constexpr int kEights = 16;
static_assert(kXCh * 2 / 4 % 32 == 12, "conflict-free channel pitch");

__device__ __forceinline__ int channel_at(int ch, int pitch) { return ch * pitch + (ch >> 3) * kEights; }

// v[k] = channels 8 c8 .. 8 c8 + 7 of pixel k, to dst[channel * pitch + k]
__device__ __forceinline__ void store_transposed(uint16_t* dst, int pitch, const uint4 (&v)[8]) {
  auto word = [&](int k, int j) { return j == 0 ? v[k].x : j == 1 ? v[k].y : j == 2 ? v[k].z : v[k].w; };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    auto even = [&](int k) { return __builtin_amdgcn_perm(word(k + 1, j), word(k, j), 0x05040100u); };
    auto odd = [&](int k) { return __builtin_amdgcn_perm(word(k + 1, j), word(k, j), 0x07060302u); };
    *reinterpret_cast<uint4*>(dst + 2 * j * pitch) = make_uint4(even(0), even(2), even(4), even(6));
    *reinterpret_cast<uint4*>(dst + (2 * j + 1) * pitch) = make_uint4(odd(0), odd(2), odd(4), odd(6));
  }
}

// sixteen bits (one pixel) further along a row: q, then e
__device__ __forceinline__ bf16x8 shifted_by_one(uint4 q, unsigned e) {
  return as_bf16x8(make_uint4(__builtin_amdgcn_alignbit(q.y, q.x, 16), __builtin_amdgcn_alignbit(q.z, q.y, 16),
                              __builtin_amdgcn_alignbit(q.w, q.z, 16), __builtin_amdgcn_alignbit(e, q.w, 16)));
}

template <Source XS, Source GS, bool DX>
__global__ __launch_bounds__(256, 2) void backward_kernel(const uint16_t* __restrict__ x,
                                                          const float* __restrict__ sigma,
                                                          const uint16_t* __restrict__ g,
                                                          const uint16_t* __restrict__ wpk, int N, int H, int W,
                                                          float* __restrict__ partial, uint16_t* __restrict__ dx) {
  // column 0 is x0 - 1, row 0 y0 - 1
  __shared__ __align__(16) uint16_t xs[kC * kXCh + 4 * kEights], gs[kC * kXCh + 4 * kEights];
  __shared__ __align__(16) uint16_t gp[DX ? kTileY + 2 : 1][kTileX + 2][kC];
  __shared__ __align__(4) uint8_t positive[DX ? kTileY + 2 : 1][kTileX + 2][4];  // x's channels, a bit each
  const int tx_n = (W + kTileX - 1) / kTileX, ty_n = (H + kTileY - 1) / kTileY;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int co_t = wave >> 1, ci_t = wave & 1;
  f32x4 acc[kTaps];
#pragma unroll
  for (int t = 0; t < kTaps; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float db = 0.0f;  // bias-gradient partial of channel tid % 32 over tile rows tid / 32
  bf16x8 wt[DX ? kTaps : 1][2];
  if constexpr (DX) {
#pragma unroll
    for (int t = 0; t < kTaps; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wt[t][h] = as_bf16x8(*reinterpret_cast<const uint4*>(wpk + (t * kC + h * 16 + col) * kC + 8 * grp));
  }
  auto piece = [](int c, int c8) { return 8 * (c8 ^ ((c >> 1) & 3)); };  // of the pixel of tile column c

  const int total = conv_items(N, H, W);
  // eights of pixels; four threads take the channels of one
  constexpr int kUnits = (kTileY + 2) * kXGroups;
  static_assert(4 * kUnits <= 256, "one eight of pixels per thread");
  uint4 vx[8], vg[8];
  const int c8 = threadIdx.x & 3, u = threadIdx.x >> 2;
  const int ur = u / kXGroups, uc = 8 * (u - ur * kXGroups);
  unsigned inside = 0;  // the pixels of the eight that lie in the image
  float sigma_n = 0.0f;
  auto load = [&](int item) {
    const int n = item / (tx_n * ty_n);
    const int rem = item - n * tx_n * ty_n;
    const int y = (rem / tx_n) * kTileY - 1 + ur, xx = (rem % tx_n) * kTileX - 1 + uc;
    if constexpr (XS == kInput) sigma_n = sigma[n];
    const bool row = u < kUnits && y >= 0 && y < H;
    const size_t pix = (static_cast<size_t>(n) * H + y) * W + xx;
    inside = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      vx[k] = make_uint4(0, 0, 0, 0);
      vg[k] = make_uint4(0, 0, 0, 0);
      // (columns past the 34th are not used)
      if (row && xx + k >= 0 && xx + k < W && uc + k < kTileX + 2) {
        vx[k] = load_channels<XS>(x, pix + k, c8);
        vg[k] = load_channels<GS>(g, pix + k, c8);
        inside |= 1u << k;
      }
    }
  };
  if (static_cast<int>(blockIdx.x) < total) load(blockIdx.x);
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    if constexpr (XS == kInput) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (inside >> k & 1) vx[k] = as_activations<XS>(vx[k], sigma_n, c8);
    }
    if (u < kUnits) {
      const int at = channel_at(8 * c8, kXCh) + ur * kXRow + uc;
      store_transposed(xs + at, kXCh, vx);
      store_transposed(gs + at, kXCh, vg);
      if constexpr (DX) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (uc + k < kTileX + 2) {
            *reinterpret_cast<uint4*>(&gp[ur][uc + k][piece(uc + k, c8)]) = vg[k];
            const unsigned m[4] = {vx[k].x, vx[k].y, vx[k].z, vx[k].w};
            unsigned bits = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              bits |= (static_cast<int>(m[j] << 16) > 0 ? 1u << (2 * j) : 0u) |
                      (static_cast<int>(m[j]) > 0xffff ? 2u << (2 * j) : 0u);
            positive[ur][uc + k][c8] = static_cast<uint8_t>(bits);
          }
      }
    }
    // the next tile's loads are in flight during this one's products
    if (item + static_cast<int>(gridDim.x) < total) load(item + gridDim.x);
    __syncthreads();
    const uint16_t* xrow = xs + channel_at(ci_t * 16 + col, kXCh) + 8 * grp;
    const uint16_t* grow = gs + channel_at(co_t * 16 + col, kXCh) + 8 * grp;
    bf16x8 A[3];  // rows row, row - 1, row - 2 of the tile's g
#pragma unroll
    for (int row = 0; row < kTileY + 2; ++row) {
      A[2] = A[1];
      A[1] = A[0];
      if (row < kTileY) {
        const uint16_t* p = grow + (row + 1) * kXRow;
        A[0] = shifted_by_one(*reinterpret_cast<const uint4*>(p), *reinterpret_cast<const unsigned*>(p + 8));
      }
      const uint4 q = *reinterpret_cast<const uint4*>(xrow + row * kXRow);
      const unsigned e = *reinterpret_cast<const unsigned*>(xrow + row * kXRow + 8);
      const bf16x8 B[3] = {as_bf16x8(q), shifted_by_one(q, e), as_bf16x8(make_uint4(q.y, q.z, q.w, e))};
#pragma unroll
      for (int ky = 0; ky < 3; ++ky)
        if (row >= ky && row - ky < kTileY) {
#pragma unroll
          for (int kx = 0; kx < 3; ++kx)
            acc[3 * ky + kx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[ky], B[kx], acc[3 * ky + kx], 0, 0, 0);
        }
    }
    {  // bias gradient: thread (channel tid % 32, row tid / 32) sums one tile row
      const uint16_t* line = gs + channel_at(threadIdx.x & (kC - 1), kXCh) + ((threadIdx.x >> 5) + 1) * kXRow;
      float s = 0.0f;
#pragma unroll
      for (int c = 0; c < kXRow; c += 8) {
        const uint4 q = *reinterpret_cast<const uint4*>(line + c);
        const unsigned v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (c + k >= 1 && c + k <= kTileX) s += bf2f(static_cast<uint16_t>(v[k / 2] >> (16 * (k % 2))));
      }
      db += s;
    }
    if constexpr (DX) {
      const int n = item / (tx_n * ty_n);
      const int rem = item - n * tx_n * ty_n;
      const int y0 = (rem / tx_n) * kTileY, x0 = (rem % tx_n) * kTileX;
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) {
        const int row = 2 * wave + (bi >> 1), xoff = (bi & 1) * 16;
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < kTaps; ++t) {
          const int c = xoff + col + t % 3;
          const bf16x8 B = as_bf16x8(*reinterpret_cast<const uint4*>(&gp[row + t / 3][c][piece(c, grp)]));
          acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[t][0], B, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[t][1], B, acc1, 0, 0, 0);
        }
        // lane holds channels 4*grp + i (acc0) and 16 + 4*grp + i (acc1) of pixel (y, xx)
        const int y = y0 + row, xx = x0 + xoff + col;
        if (y < H && xx < W) {
          const size_t p = ((static_cast<size_t>(n) * H + y) * W + xx) * kC + 4 * grp;
          const unsigned m = *reinterpret_cast<const unsigned*>(positive[row + 1][xoff + col + 1]) >> (4 * grp);
          float v0[4], v1[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v0[i] = m >> i & 1 ? acc0[i] : 0.0f;
            v1[i] = m >> (16 + i) & 1 ? acc1[i] : 0.0f;
          }
          store_channels(dx + p, v0, v1);
        }
      }
    }
    __syncthreads();
  }
  // D[co][ci]: lane holds co = co_t*16 + 4*grp + i, ci = ci_t*16 + col; stored as [t][ci][co]
  float* dst = partial + static_cast<size_t>(blockIdx.x) * (kWmat + kC);
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[(t * kC + ci_t * 16 + col) * kC + co_t * 16 + 4 * grp + i] = acc[t][i];
  __shared__ float dbs[256];
  dbs[threadIdx.x] = db;
  __syncthreads();
  if (threadIdx.x < kC) {
    float s = 0.0f;
    for (int r = 0; r < kTileY; ++r) s += dbs[r * kC + threadIdx.x];
    dst[kWmat + threadIdx.x] = s;
  }
}

// grad (canonical layout of one layer) = sum over workgroups of the partials,
// in double.  Bound by memory latency: a thread that walked all the partials
// of an output alone had 512 dependent-in-time strided loads in only 37
// workgroups (125 us per 32 -> 32 layer).  Here a workgroup takes 64 outputs
// and each of its 16 waves every 16th partial, eight loads in flight, and the
// waves' sums are added in wave order: 4.8 us.
constexpr int kRedWaves = 16;
__global__ __launch_bounds__(64 * kRedWaves) void wgrad_reduce_kernel(const float* __restrict__ partial, int n_part,
                                                                      int ci_n, int co_n, float* __restrict__ grad) {
  __shared__ double sums[kRedWaves][64];
  const int n_w = kTaps * ci_n * co_n, n_out = n_w + co_n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane, o = min(i, n_out - 1);
  int src;
  if (o < n_w) {
    const int t = o / (ci_n * co_n), rem = o - t * ci_n * co_n;
    const int ci = rem / co_n, co = rem - ci * co_n;
    src = (t * kC + ci) * kC + co;
  } else {
    src = kWmat + (o - n_w);
  }
  double s = 0.0;
#pragma unroll 8
  for (int k = wave; k < n_part; k += kRedWaves) s += partial[static_cast<size_t>(k) * (kWmat + kC) + src];
  sums[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < n_out) {
#pragma unroll
    for (int w = 1; w < kRedWaves; ++w) s += sums[w][lane];
    grad[i] = static_cast<float>(s);
  }
}

// loss gradient of the (per-image weighted) mean squared error:
// dL/df = -2 w_b (pilot - target) / n with w_b = weight[pixel / hw] (1 if no
// weights), one bf16 per pixel; per-block partial sums of the weighted squared
// error in double.
__global__ __launch_bounds__(256) void loss_kernel(const float* __restrict__ pilot, const float* __restrict__ target,
                                                   const float* __restrict__ weight, size_t hw, size_t n,
                                                   uint16_t* __restrict__ g, double* __restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  const float scale = -2.0f / static_cast<float>(n);
  for (size_t p = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; p < n;
       p += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const float w = weight ? weight[p / hw] : 1.0f;
    const float d = pilot[p] - target[p];
    s += static_cast<double>(w) * d * d;
    g[p] = f2bf(scale * w * d);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// one workgroup: thread i adds partials i, i + 256, ..., then a tree over the
// threads: 4.7 us for 1024 partials (one thread adding all of them, a chain of
// loads, took 68 us)
__global__ __launch_bounds__(256) void loss_reduce_kernel(const double* __restrict__ part, int n_part, size_t n,
                                                          float* __restrict__ loss) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n_part; i += 256) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = static_cast<float>(red[0] / static_cast<double>(n));
}

// packed weights from the float32 master vector: forward [l][t][co][ci],
// backward [l][t'][ci][co] = W[8-t'][ci][co], biases [l][32]; zero padded
__global__ void pack_kernel(const float* __restrict__ master, uint16_t* __restrict__ wf, uint16_t* __restrict__ wb,
                            float* __restrict__ bias) {
  const int total = kPilotLayers * kWmat;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total + kPilotLayers * kC; i += gridDim.x * blockDim.x) {
    if (i >= total) {
      const int l = (i - total) / kC, co = (i - total) % kC;
      const int off = pilot_layer_offset(l), ci_n = pilot_cin(l), co_n = pilot_cout(l);
      bias[l * kC + co] = co < co_n ? master[off + kTaps * ci_n * co_n + co] : 0.0f;
      continue;
    }
    const int l = i / kWmat, rem = i % kWmat;
    const int t = rem / (kC * kC), a = (rem / kC) % kC, b = rem % kC;
    const int off = pilot_layer_offset(l), ci_n = pilot_cin(l), co_n = pilot_cout(l);
    // forward: (t, co = a, ci = b)
    wf[i] = (b < ci_n && a < co_n) ? f2bf(master[off + (t * ci_n + b) * co_n + a]) : 0;
    // backward: (t', ci = a, co = b) = W[8 - t'][ci][co]
    wb[i] = (a < ci_n && b < co_n) ? f2bf(master[off + ((8 - t) * ci_n + a) * co_n + b]) : 0;
  }
}

__global__ void adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, int n, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

}  // namespace

int pilot_conv_items(int N, int H, int W) { return conv_items(N, H, W); }

size_t pilot_packed_bytes() { return static_cast<size_t>(kPilotLayers) * kWmat * 2 * sizeof(uint16_t); }

size_t pilot_wgrad_partial_floats(int grid) { return static_cast<size_t>(grid) * (kWmat + kC); }

hipError_t launch_pilot_pack(const float* master, uint16_t* wf, uint16_t* wb, float* bias, hipStream_t st) {
  hipLaunchKernelGGL(pack_kernel, dim3(256), dim3(256), 0, st, master, wf, wb, bias);
  return hipGetLastError();
}

int pilot_fused_tiles(int N, int H, int W) { return fused_tiles(N, H, W); }

hipError_t launch_pilot_infer_fused(const uint16_t* noisy, const float* sigma, const uint16_t* wf, const float* bias,
                                    int N, int H, int W, float* pilot_f32, uint16_t* pilot_u16, int grid_cap,
                                    hipStream_t st) {
  const int grid = std::max(1, std::min(fused_tiles(N, H, W), grid_cap));
  hipLaunchKernelGGL(fused_infer_kernel, dim3(grid), dim3(kFThreads), 0, st, noisy, sigma, wf, bias, N, H, W,
                     pilot_f32, pilot_u16);
  return hipGetLastError();
}

hipError_t launch_pilot_conv(int layer, const uint16_t* in, const float* sigma, const uint16_t* w, const float* bias,
                             uint16_t* out, const uint16_t* noisy, float* pilot_f32, uint16_t* pilot_u16, int N,
                             int H, int W, int grid_cap, hipStream_t st) {
  const int grid = std::max(1, std::min(conv_items(N, H, W), grid_cap));
  if (layer == 0)
    hipLaunchKernelGGL((conv_kernel<0, kInput>), dim3(grid), dim3(256), 0, st, in, sigma, w, bias, out, noisy,
                       pilot_f32, pilot_u16, N, H, W);
  else if (layer < kPilotLayers - 1)
    hipLaunchKernelGGL((conv_kernel<0, kAct>), dim3(grid), dim3(256), 0, st, in, sigma, w, bias, out, noisy,
                       pilot_f32, pilot_u16, N, H, W);
  else
    hipLaunchKernelGGL((conv_kernel<1, kAct>), dim3(grid), dim3(256), 0, st, in, sigma, w, bias, out, noisy,
                       pilot_f32, pilot_u16, N, H, W);
  return hipGetLastError();
}

hipError_t launch_pilot_loss(const float* pilot, const float* target, const float* weight, size_t hw, size_t n,
                             uint16_t* g, double* part, int n_part, float* loss, hipStream_t st) {
  hipLaunchKernelGGL(loss_kernel, dim3(n_part), dim3(256), 0, st, pilot, target, weight, hw, n, g, part);
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, st, part, n_part, n, loss);
  return hipGetLastError();
}

hipError_t launch_pilot_backward(int layer, const uint16_t* x, const float* sigma, const uint16_t* g,
                                 const uint16_t* w, int N, int H, int W, int grid, float* partial, float* grad_layer,
                                 uint16_t* dx, hipStream_t st) {
  if (layer == 0)
    hipLaunchKernelGGL((backward_kernel<kInput, kAct, false>), dim3(grid), dim3(256), 0, st, x, sigma, g, w, N, H, W,
                       partial, dx);
  else if (layer < kPilotLayers - 1)
    hipLaunchKernelGGL((backward_kernel<kAct, kAct, true>), dim3(grid), dim3(256), 0, st, x, sigma, g, w, N, H, W,
                       partial, dx);
  else
    hipLaunchKernelGGL((backward_kernel<kAct, kLossGrad, true>), dim3(grid), dim3(256), 0, st, x, sigma, g, w, N, H, W,
                       partial, dx);
  const int ci_n = pilot_cin(layer), co_n = pilot_cout(layer);
  const int n_out = kTaps * ci_n * co_n + co_n;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((n_out + 63) / 64), dim3(64 * kRedWaves), 0, st, partial, grid, ci_n,
                     co_n, grad_layer);
  return hipGetLastError();
}

hipError_t launch_pilot_adam(float* w, float* m, float* v, const float* g, int n, float lr, float b1, float b2,
                             float eps, int step, hipStream_t st) {
  const float c1 = 1.0f - powf(b1, static_cast<float>(step));
  const float c2 = 1.0f - powf(b2, static_cast<float>(step));
  hipLaunchKernelGGL(adam_kernel, dim3(64), dim3(256), 0, st, w, m, v, g, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace gbm3d
