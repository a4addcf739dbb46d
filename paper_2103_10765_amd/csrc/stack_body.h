// The transform-domain patch stack of four image rows by 64 columns, the work of
// four waves: shared by the stack kernels and by the matching kernel, whose
// launch writes the stacks beside its own work.
#pragma once
#include "common.h"

namespace gbm3d {

namespace {

constexpr int kStackRows = 4;
constexpr int kStackThreads = kStackRows * kWave;       // one wave per output row
constexpr int kStackPixRows = kStackRows + kPatch - 1;  // 11
constexpr int kStackPixCols = kWave + kPatch - 1;       // 71
constexpr int kStagePitch = 65;                         // floats per parked block (odd: conflict-free)

// LDS of one item, PARTS = 64 / the positions a wave parks at a time
template <int PARTS>
struct StackLds {
  float pix[kStackPixRows][kStackPixCols + 1];
  float stage[kStackRows][kWave / PARTS * kStagePitch];
};

// one separable level on the leading L x L block: rows (x[a][0..L)), then columns
template <int L, typename F>
__device__ __forceinline__ void rows_cols(float (&x)[8][8], F&& line) {
#pragma unroll
  for (int a = 0; a < L; ++a) {
    float t[8];
    line(x[a], t);
#pragma unroll
    for (int b = 0; b < L; ++b) x[a][b] = t[b];
  }
#pragma unroll
  for (int b = 0; b < L; ++b) {
    float c[8], t[8];
#pragma unroll
    for (int a = 0; a < L; ++a) c[a] = x[a][b];
    line(c, t);
#pragma unroll
    for (int a = 0; a < L; ++a) x[a][b] = t[a];
  }
}

template <int KIND>
__device__ __forceinline__ void forward2d(float (&x)[8][8]) {
  if constexpr (KIND == 0) {
    constexpr Mat8 A8 = bior_analysis(8);
    constexpr Mat8 A4 = bior_analysis(4);
    constexpr Mat8 A2 = bior_analysis(2);
    rows_cols<8>(x, [&](const float* i, float* o) { apply_mat<8>(A8, i, o); });
    rows_cols<4>(x, [&](const float* i, float* o) { apply_mat<4>(A4, i, o); });
    rows_cols<2>(x, [&](const float* i, float* o) { apply_mat<2>(A2, i, o); });
  } else if constexpr (KIND == 1) {
    rows_cols<8>(x, [&](const float* i, float* o) { dct8_fwd(i, o); });
  } else {
    rows_cols<8>(x, [&](const float* i, float* o) { dct8_fwd_raw(i, o); });
  }
}

__host__ __device__ constexpr int stack_items(int H, int W) {
  return ((H + kStackRows - 1) / kStackRows) * ((W + kWave - 1) / kWave);
}

// One item by the four waves of threads t = 0 .. 255; every thread of the
// workgroup has to come here (barriers), those of a half without an item with
// item < 0.
// KIND 0: bior1.5; 1: DCT; 2: DCT as the Wiener groups want it, without its
// output factors dct8_scale(a) dct8_scale(b) for the pilot, with their squares
// for the noisy image (no multiplications for the first, and 26 instead of 40
// operations per line).
// LOADS_FIRST: every thread's pixel loads are issued before the first is
// used (one memory round trip for the tile); otherwise one item at a time.
template <int KIND, int PARTS, bool LOADS_FIRST>
__device__ __forceinline__ void stack_body(StackLds<PARTS>& lds, int t, const uint16_t* __restrict__ img_,
                                           float* __restrict__ out_, unsigned long long* __restrict__ block_weights_,
                                           bool noisy, int H, int W, int item) {
  constexpr int kPart = kWave / PARTS;
  auto& pix = lds.pix;
  auto& stage = lds.stage;
  if (item < 0) {
    __syncthreads();
    return;
  }
  const auto img = to_global(img_);
  const auto out = to_global(out_);
  const auto block_weights = to_global(block_weights_);
  const int xt = (W + kWave - 1) / kWave;
  const int y0 = (item / xt) * kStackRows;
  const int x0 = (item % xt) * kWave;
  const float scale = 1.0f / 65535.0f;
  // a tile reaches at most one period past the image that it is smaller than
  const bool once = H >= kStackPixRows && W >= kStackPixCols;
  auto wrap = [&](int r, int c) {
    const int y = y0 + r, x = x0 + c;
    return once ? static_cast<size_t>(y < H ? y : y - H) * W + (x < W ? x : x - W)
                : static_cast<size_t>(y % H) * W + x % W;
  };
  constexpr int kPix = kStackPixRows * kStackPixCols;
  if constexpr (LOADS_FIRST) {
    constexpr int kPixIter = (kPix + kStackThreads - 1) / kStackThreads;
    unsigned zv[kPixIter];
#pragma unroll
    for (int it = 0; it < kPixIter; ++it) {
      // (unconditional: threads past the tile's last pixel reload it)
      const int i = min(t + it * kStackThreads, kPix - 1);
      const int r = i / kStackPixCols, c = i - r * kStackPixCols;
      zv[it] = img[wrap(r, c)];
    }
#pragma unroll
    for (int it = 0; it < kPixIter; ++it) {
      const int i = t + it * kStackThreads;
      if (i < kPix) {
        const int r = i / kStackPixCols, c = i - r * kStackPixCols;
        pix[r][c] = static_cast<float>(zv[it]) * scale;
      }
    }
  } else {
    for (int i = t; i < kPix; i += kStackThreads) {
      const int r = i / kStackPixCols, c = i - r * kStackPixCols;
      pix[r][c] = static_cast<float>(img[wrap(r, c)]) * scale;
    }
  }
  __syncthreads();

  const int lane = t & (kWave - 1);
  const int w = t / kWave;
  float x[8][8];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) x[a][b] = pix[w + a][lane + b];
  forward2d<KIND>(x);
  if (KIND == 2 && noisy) {
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const double s = dct8_scale(a) * dct8_scale(b);
        x[a][b] *= static_cast<float>(s * s);
      }
  }
  const int y = y0 + w;
  const int n_pos = min(kWave, W - x0);  // positions of this row in the tile
  // the aggregation that follows adds into the block-start weights and the
  // numerator sums
  if (block_weights && y < H && lane < n_pos) {
    const size_t o = static_cast<size_t>(y) * W + x0 + lane;
    block_weights[o] = 0;
    block_weights[block_weight_entries(H, W) + o] = 0;
  }
  typedef float f32x4v __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) float lds_f32;
  const auto dst = (global_ptr<f32x4v>)(out + (static_cast<size_t>(y) * W + x0) * 64);
  // (addresses in registers of their own: as sums with the tile's place in LDS
  // every pair of accesses would have an addition)
  lds_f32* park = (lds_f32*)(stage[w] + (lane % kPart) * kStagePitch);
  const lds_f32* from = (const lds_f32*)(stage[w] + (lane >> 4) * kStagePitch + (lane & 15) * 4);
  asm volatile("" : "+v"(park), "+v"(from));
  const bool whole = y < H && n_pos == kWave;
#pragma unroll
  for (int part = 0; part < PARTS; ++part) {
    wave_lds_sync();  // the previous part's reads are done
    if (lane / kPart == part) {
#pragma unroll
      for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) park[a * 8 + b] = x[a][b];
    }
    wave_lds_sync();
    // in round i lane l stores float4 i * 64 + l of the part's run, of its
    // position 4 i + l / 16
    auto store = [&](int i) {
      const lds_f32* s = from + i * 4 * kStagePitch;
      dst[(part * kPart + i * 4) * 16 + lane] = f32x4v{s[0], s[1], s[2], s[3]};
    };
    if (whole) {
#pragma unroll
      for (int i = 0; i < kPart / 4; ++i) store(i);
    } else if (y < H) {
#pragma unroll
      for (int i = 0; i < kPart / 4; ++i)
        if (part * kPart + i * 4 + (lane >> 4) < n_pos) store(i);
    }
  }
}

}  // namespace

}  // namespace gbm3d
