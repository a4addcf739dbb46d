// Collaborative filtering of matched groups and their aggregation.
//
// A workgroup of 8 to 16 waves owns a tile of 8 to 64 references; each wave
// filters one group at a time with lane = 2-D coefficient index (64 lanes =
// 8x8 coefficients) and the group axis in registers:
//   decode the K block positions (lane k decodes slot k, the values are
//   broadcast as scalars), gather the K spectra from the patch stack (one
//   coalesced 256 B load per block), 1-D Haar along the group, shrink,
//   inverse Haar, inverse 2-D transform of the K blocks through a per-wave LDS
//   scratch (separable rows then columns, level by level, at most 16 blocks
//   at a time), group weight, and accumulation of w*U into an LDS image of
//   the tile's footprint (every block a reference of the tile can match lies
//   in it: rows 3p-R .. 3p+7+R).
// The denominator sum of w over the blocks covering a pixel is not spread
// over 64 pixels per block: w is added once per block at the block's
// top-left pixel of an image-sized array (global integer atomics, one
// instruction per group), and the pixel's denominator is the 8 x 8 box sum
// of that array (periodic).
// All sums are 64-bit fixed point (2^-40), so their value does not depend on
// the order in which waves add: results are bit-reproducible.  The footprint
// is added once per tile into the image's numerator sums (global integer
// atomics at the periodic positions); a second kernel forms the box sum,
// divides and optionally quantises.
//
// Stage 1 (Sec. 3.1, Sec. 5): bior1.5 stack, hard threshold |C| >= tau_l with
//   tau_l = sigma (a - b l) by Mallat level, 3-D DC kept, weight 1/(TV+eps)
//   (scaled by eps so that it lies in (0, 1]; the weighted average does not
//   change).
// Stage 2 (Sec. 4): DCT stacks of the noisy image and the pilot, Wiener gain
//   W = b^2 / (b^2 + sigma^2) of the pilot spectrum (W = 1 at the 3-D DC)
//   applied to the noisy spectrum, weight 1 / sum W^2.
#include "common.h"
#include "kernels.h"


namespace gbm3d {

namespace {

constexpr int kScratchPitch = 9;                  // LDS row pitch of a parked 8x8 block
constexpr int kBlockFloats = 8 * kScratchPitch;   // 72
constexpr int kReduceThreads = 256;
constexpr int kLdsBytes = 160 * 1024;             // LDS of one workgroup

using acc_t = unsigned long long;

// The reference tile of a workgroup and its footprint.
template <int PY, int PX>
struct Tile {
  static constexpr int refs = PY * PX, py = PY, px = PX;
  static constexpr int FYmax = kStep * (PY - 1) + kPatch + 2 * kMaxR;
  static constexpr int FXmax = kStep * (PX - 1) + kPatch + 2 * kMaxR;
  // cells per footprint row of every window (so that the rows of a block are
  // instruction offsets), 8 modulo 32
  static constexpr int FXP = FXmax + ((8 - FXmax) % 32 + 32) % 32;
  static constexpr int entries = FYmax * FXP;
};

struct GroupArgs {
  int H, W, R, S, nRy, nRx, nTx, nTy;
  int FY, FX;
  float invS;  // 1 / S for the rank decode
};

template <typename T>
__host__ __device__ inline GroupArgs make_args(int H, int W, int R) {
  GroupArgs g;
  g.H = H;
  g.W = W;
  g.R = R;
  g.S = 2 * R + 1;
  g.nRy = (H + kStep - 1) / kStep;
  g.nRx = (W + kStep - 1) / kStep;
  g.nTx = (g.nRx + T::px - 1) / T::px;
  g.nTy = (g.nRy + T::py - 1) / T::py;
  g.FY = kStep * (T::py - 1) + kPatch + 2 * R;
  g.FX = kStep * (T::px - 1) + kPatch + 2 * R;
  g.invS = 1.0f / static_cast<float>(g.S);
  return g;
}

// The tile's matched blocks, [reference t][K] (t = row-major place among the
// tile's references): stack position (pixel index) and first footprint cell
// (its byte offset).
// They are decoded from the ranks once, by all threads (per group and wave it
// would be 25 instructions for K active lanes).
template <int K, typename T>
struct Slots {
  alignas(16) int pos[T::refs * K];
  alignas(16) uint16_t fo[T::refs * K];

  // every thread's rank loads are issued before the first is used: one memory
  // round trip per tile.  References past the image's last row or column get a
  // clamped in-bounds entry that no group uses.  The caller's next barrier
  // publishes the slots.
  template <int THREADS>
  __device__ __forceinline__ void load(const GroupArgs& g, const int16_t* idx_, int tyi, int txi) {
    const auto idx = to_global(idx_);
    constexpr int n = T::refs * K;
    constexpr int iters = (n + THREADS - 1) / THREADS;
    int v[iters];
#pragma unroll
    for (int it = 0; it < iters; ++it) {
      const int e = min(static_cast<int>(threadIdx.x) + it * THREADS, n - 1);
      const int t = e / K, k = e % K;
      const int p = min(tyi * T::py + t / T::px, g.nRy - 1), q = min(txi * T::px + t % T::px, g.nRx - 1);
      v[it] = idx[(static_cast<size_t>(p) * g.nRx + q) * K + k];
    }
#pragma unroll
    for (int it = 0; it < iters; ++it) {
      const int e = static_cast<int>(threadIdx.x) + it * THREADS;
      if (e >= n) break;
      const int t = e / K, r = v[it];
      const int p = min(tyi * T::py + t / T::px, g.nRy - 1), q = min(txi * T::px + t % T::px, g.nRx - 1);
      // r / S in float: r + 1/2 lies at least 1/(2S) from a multiple of S and
      // r < S^2 <= 1521, far inside float's exact range
      const int dyi = static_cast<int>((static_cast<float>(r) + 0.5f) * g.invS), dxi = r - dyi * g.S;
      const int y = kStep * p + dyi - g.R, x = kStep * q + dxi - g.R;
      // -R <= y < H + R and H >= S > R + 1: at most one period away (same for x)
      const int yw = y < 0 ? y + g.H : (y >= g.H ? y - g.H : y);
      const int xw = x < 0 ? x + g.W : (x >= g.W ? x - g.W : x);
      pos[e] = yw * g.W + xw;
      const int cell = (kStep * (p - tyi * T::py) + dyi) * T::FXP + kStep * (q - txi * T::px) + dxi;
      fo[e] = static_cast<uint16_t>(cell * static_cast<int>(sizeof(acc_t)));
    }
  }
};

// Shapes of the group kernels.
enum GroupShape {
  kTwoTiles,  // 8 x 8 references by 16 waves (K = 32: 12), two tiles per CU
  kOneTile,   // 8 x 8 references by 16 waves, one tile per CU, the next group's spectra in flight
  kSmall,     // 4 x 4 references by 8 waves
  kTiny,      // 2 x 4 references by 8 waves
};

// Launch shape of a group kernel.  Tiles share a CU so that it has 32 waves (64
// registers: K <= 16; an even four groups per wave) or 24 (80: K = 32);
// inverse transforms go 8 blocks at a time through each wave's scratch, without
// a prefetch of the next group (the other waves hide the loads).  The Wiener
// kernel by 12 instead of 16 waves, us: K = 2, 4 (bound by latency) 1024^2 76 |
// 92 against 66 | 81, 2048^2 247 | 296 against 221 | 273; K = 8, 16 2048^2 388 |
// 599 against 379 | 594; at K = 32 sixteen waves leave room for one tile, 1097
// against 1044.  kOneTile is a choice of the autotuner for the
// hard-threshold kernel (K <= 16).  That kernel at K = 32 takes two tiles of
// twelve waves, 80 registers; 16 blocks at a time through the scratch of eight
// waves, two tiles a little too large for one CU's LDS ran one by one (kernel us
// 512^2 107 -> 85, 1024^2 405 -> 287, 2048^2 1503 -> 1002).
template <int K, bool HT, int SHAPE>
struct GroupCfg {
  using T = std::conditional_t<SHAPE == kTiny, Tile<2, 4>, std::conditional_t<SHAPE == kSmall, Tile<4, 4>, Tile<8, 8>>>;
  static constexpr bool prefetch = SHAPE == kOneTile;
  static constexpr int chunk = SHAPE == kOneTile ? K : (K > 8 ? 8 : K);
  using SlotTable = Slots<K, T>;
  static constexpr int waves = SHAPE == kOneTile ? 16 : SHAPE != kTwoTiles ? 8 : K <= 16 ? 16 : 12;
  static constexpr int tiles = SHAPE == kOneTile ? 1 : SHAPE == kTwoTiles ? 2 : 3;
  static constexpr int threads = waves * kWave;
  static constexpr int min_waves_per_simd = waves * tiles / 4;
  static_assert(SHAPE != kOneTile || (HT && K <= 16), "only the hard-threshold kernel of small groups prefetches");
  static_assert(tiles * (T::entries * static_cast<int>(sizeof(acc_t)) +
                         waves * chunk * kBlockFloats * static_cast<int>(sizeof(float)) +
                         static_cast<int>(sizeof(SlotTable))) <=
                    kLdsBytes,
                "LDS of the tiles sharing a CU");
};

__host__ __device__ inline int reduce_items(int H, int W) { return H * ((W + kReduceThreads - 1) / kReduceThreads); }

struct HtParams {
  float ht_a, ht_b;
  int weight_mode, keep_dc;
};

// Lines of the leading L x L block of each of K blocks parked at
// xw[k * BLOCK + a * PITCH + b], one line per lane: every row in place.
template <int K, int L, int BLOCK, int PITCH, typename F>
__device__ __forceinline__ void transform_rows(float* xw, int lane, F&& line) {
  constexpr int items = K * L;
#pragma unroll
  for (int it0 = 0; it0 < items; it0 += kWave) {
    const int it = it0 + lane;
    if (it < items) {
      float* row = xw + it / L * BLOCK + it % L * PITCH;
      float x[8], y[8];
#pragma unroll
      for (int j = 0; j < L; ++j) x[j] = row[j];
      line(x, y);
#pragma unroll
      for (int j = 0; j < L; ++j) row[j] = y[j];
    }
  }
  wave_lds_sync();
}

// Every column: put(pass, k, j, y), y the transformed column j of block k.
template <int K, int L, int BLOCK, int PITCH, typename F, typename P>
__device__ __forceinline__ void transform_columns(const float* xw, int lane, F&& line, P&& put) {
  constexpr int items = K * L;
#pragma unroll
  for (int it0 = 0; it0 < items; it0 += kWave) {
    const int it = it0 + lane;
    if (it < items) {
      const float* col = xw + it / L * BLOCK + it % L;
      float x[8], y[8];
#pragma unroll
      for (int i = 0; i < L; ++i) x[i] = col[i * PITCH];
      line(x, y);
      put(it0 / kWave, it / L, it % L, y);
    }
  }
}

// One separable level in place: rows, then columns.
template <int K, int L, int BLOCK = kBlockFloats, int PITCH = kScratchPitch, typename F>
__device__ __forceinline__ void transform_level(float* xw, int lane, F&& line) {
  transform_rows<K, L, BLOCK, PITCH>(xw, lane, line);
  transform_columns<K, L, BLOCK, PITCH>(xw, lane, line, [&](int, int k, int j, const float (&y)[8]) {
#pragma unroll
    for (int i = 0; i < L; ++i) xw[k * BLOCK + i * PITCH + j] = y[i];
  });
  wave_lds_sync();
}

// The footprint cell at a byte offset.
__device__ __forceinline__ acc_t* cell_at(acc_t* acc, unsigned bytes) {
  return reinterpret_cast<acc_t*>(reinterpret_cast<char*>(acc) + bytes);
}

// ws * u[k] (fixed point) into the footprint, block k at byte offset fo[k] (two
// to a word)
template <int K, typename T>
__device__ __forceinline__ void accumulate(acc_t* acc, const uint16_t* fo, const float (&u)[K], float ws, int lane) {
  const unsigned ab = ((lane >> 3) * T::FXP + (lane & 7)) * sizeof(acc_t);
  const unsigned* pairs = reinterpret_cast<const unsigned*>(fo);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const unsigned o = k % 2 ? pairs[k / 2] >> 16 : pairs[k / 2] & 0xffffu;
    atomicAdd(cell_at(acc, o + ab), static_cast<acc_t>(to_fixed_scaled(ws * u[k])));
  }
}

// w at the top-left pixel pos of each of the K blocks (lane k holds slot k's);
// integer addition, so the order of the atomics does not matter
template <int K>
__device__ __forceinline__ void add_block_weights(acc_t* bw, int pos_v, float w, int lane) {
  if (lane < K)
    __hip_atomic_fetch_add(to_global(bw) + pos_v, static_cast<acc_t>(to_fixed(w)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void zero_acc(acc_t* acc, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) acc[i] = 0;
  __syncthreads();
}

// The tile's footprint (origin fy0, fx0 in unwrapped image coordinates) added
// into the image's numerator sums at the periodic positions it covers, one
// agent-scope integer atomic per nonzero cell: integer addition, so the sums
// do not depend on the order in which tiles arrive.  A wave takes whole
// footprint rows, a lane the same columns of each.
template <typename T>
__device__ __forceinline__ void flush_acc(const acc_t* acc, const GroupArgs& g, int fy0, int fx0,
                                          acc_t* __restrict__ num) {
  __syncthreads();
  const auto gnum = to_global(num);
  const int lane = threadIdx.x & (kWave - 1);
  const int waves = static_cast<int>(blockDim.x) / kWave;
  // -R <= fy0 and fy0 + FY <= H + FY - R + 1: with H > FY every footprint row
  // is at most one period away (same for the columns)
  const bool once = g.H > g.FY && g.W > g.FX;
  constexpr int kPasses = (T::FXmax + kWave - 1) / kWave;
  int xs[kPasses];
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    const int x = fx0 + p * kWave + lane;
    xs[p] = once ? x + (x < 0 ? g.W : (x >= g.W ? -g.W : 0)) : pmod(x, g.W);
  }
  for (int fy = wave_id(); fy < g.FY; fy += waves) {
    int y = fy0 + fy;
    y = once ? y + (y < 0 ? g.H : (y >= g.H ? -g.H : 0)) : pmod(y, g.H);
    const auto row = gnum + static_cast<size_t>(y) * g.W;
    const acc_t* cells = acc + fy * T::FXP;
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int fx = p * kWave + lane;
      const acc_t v = fx < g.FX ? cells[fx] : 0;
      if (v != 0) __hip_atomic_fetch_add(row + xs[p], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();  // the accumulator is reused by the next item
}

// The groups a wave filters in a tile: reference t = wave + j * WAVES,
// j < kGroups.
template <typename T, int WAVES>
struct GroupWalk {
  static constexpr int kGroups = (T::refs + WAVES - 1) / WAVES;
  const GroupArgs& g;
  const int* pos;  // the tile's block positions in LDS [reference t][K]
  int tyi, txi, wave, lane;

  __device__ __forceinline__ int ref(int j) const { return wave + j * WAVES; }
  __device__ __forceinline__ bool exists(int j) const {
    const int t = ref(j);
    return j < kGroups && t < T::refs && tyi * T::py + t / T::px < g.nRy && txi * T::px + t % T::px < g.nRx;
  }
  // position of slot lane % K of group j (0 past the last)
  template <int K>
  __device__ __forceinline__ int slot(int j) const {
    const int t = ref(j);
    return t < T::refs ? pos[t * K + (lane & (K - 1))] : 0;
  }
  // stack rows of the group whose slots' positions the lanes hold:
  // v[k] = stack[pos_k * 64 + lane]
  template <int K, int NS>
  __device__ __forceinline__ void gather(int pos_v, const float* const (&stacks)[NS], float (&v)[NS][K]) const {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      // the block's base address is uniform: it goes into a buffer resource
      // (scalar arithmetic only), the lane offset into the load itself
      const size_t blk = static_cast<size_t>(__builtin_amdgcn_readlane(pos_v, k)) * 64;
#pragma unroll
      for (int s = 0; s < NS; ++s) v[s][k] = load_block_lane(stacks[s] + blk, lane);
    }
  }
  // the pixels of the group's blocks instead of their spectra: v[k] = z at
  // (row lane / 8, column lane % 8) of slot k's block (periodic),
  // z = Z / 65535 as the stack kernel reads it
  template <int K>
  __device__ __forceinline__ void gather_pixels(int pos_v, const uint16_t* __restrict__ img, float (&v)[1][K]) const {
    const int a = lane >> 3, b = lane & 7;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int pos = __builtin_amdgcn_readlane(pos_v, k);
      const int y = pos / g.W, x = pos - y * g.W;
      const int yy = y + a >= g.H ? y + a - g.H : y + a, xx = x + b >= g.W ? x + b - g.W : x + b;
      v[0][k] = static_cast<float>(to_global(img)[static_cast<size_t>(yy) * g.W + xx]) * (1.0f / 65535.0f);
    }
  }
};

// The forward 2-D bior1.5 transform (three periodic Mallat levels, rows then
// columns at each, as the stage-1 stack computes it) of K blocks whose
// pixels the lanes hold (lane = pixel a * 8 + b), CH blocks at a time
// through the wave's scratch (the same separable passes as the inverse);
// afterwards v[k] is coefficient `lane` of block k.
template <int K, int CH>
__device__ __forceinline__ void forward_blocks(float* xw, int lane, float (&v)[K]) {
  const int a = lane >> 3, b = lane & 7;
  constexpr Mat8 A8 = bior_analysis(8);
  constexpr Mat8 A4 = bior_analysis(4);
  constexpr Mat8 A2 = bior_analysis(2);
#pragma unroll
  for (int c0 = 0; c0 < K; c0 += CH) {
    wave_lds_sync();  // earlier reads of the scratch are done
#pragma unroll
    for (int k = 0; k < CH; ++k) xw[k * kBlockFloats + a * kScratchPitch + b] = v[c0 + k];
    wave_lds_sync();
    transform_level<CH, 8>(xw, lane, [&](const float* x, float* y) { apply_mat<8>(A8, x, y); });
    transform_level<CH, 4>(xw, lane, [&](const float* x, float* y) { apply_mat<4>(A4, x, y); });
    transform_level<CH, 2>(xw, lane, [&](const float* x, float* y) { apply_mat<2>(A2, x, y); });
#pragma unroll
    for (int k = 0; k < CH; ++k) v[c0 + k] = xw[k * kBlockFloats + a * kScratchPitch + b];
  }
}

// Runs filter(v, j, pos_v) on every group j of this wave in the tile, v the
// gathered spectra, lane k < K's pos_v slot k's position.  PREFETCH also keeps
// the next group's spectra in flight (otherwise the CU's other waves hide the
// loads).
template <int K, int NS, bool PREFETCH, typename W, typename F>
__device__ __forceinline__ void for_each_group(const W& walk, const float* const (&stacks)[NS], F&& filter) {
  if constexpr (PREFETCH) {
    int pos_c = walk.template slot<K>(0), pos_n = walk.template slot<K>(1);
    float cur[NS][K];
    bool ok_c = walk.exists(0);
    if (ok_c) walk.template gather<K, NS>(pos_c, stacks, cur);
    for (int j = 0; j < walk.kGroups; ++j) {
      const int pos_2 = walk.template slot<K>(j + 2);
      float nxt[NS][K];
      const bool ok_n = walk.exists(j + 1);
      if (ok_n) walk.template gather<K, NS>(pos_n, stacks, nxt);
      if (ok_c) filter(cur, j, pos_c);
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int k = 0; k < K; ++k) cur[s][k] = nxt[s][k];
      pos_c = pos_n;
      pos_n = pos_2;
      ok_c = ok_n;
    }
  } else {
    int pos_v = walk.template slot<K>(0);
    for (int j = 0; j < walk.kGroups; ++j) {
      const int pos_n = walk.template slot<K>(j + 1);
      if (walk.exists(j)) {
        float cur[NS][K];
        walk.template gather<K, NS>(pos_v, stacks, cur);
        filter(cur, j, pos_v);
      }
      pos_v = pos_n;
    }
  }
}

// |v| * haar_gain(k) >= tau, a float product, as |v| >= a threshold: haar_gain
// is 2^-m, or sqrt(1/2) 2^-m for which the smallest t with t sqrt(1/2) >= tau
// (rounded) lies within two units of the last place of tau sqrt(2).
constexpr float kSqrtHalf = static_cast<float>(kInvSqrt2);
__device__ __forceinline__ float smallest_kept(float tau) {
  const float t0 = tau * static_cast<float>(2 * kInvSqrt2);
  float t = __int_as_float(__float_as_int(t0) + 2);
#pragma unroll
  for (int d = 1; d >= -2; --d) {
    const float c = __int_as_float(__float_as_int(t0) + d);
    t = c * kSqrtHalf >= tau ? c : t;
  }
  return t;
}
// e of haar_gain2<K>(k) = 2^-e
template <int K>
__host__ __device__ constexpr int gain2_log(int k) {
  int e = 0;
  for (float g = haar_gain2<K>(k); g < 1.0f; g *= 2.0f) ++e;
  return e;
}
template <int K>
constexpr bool gains_are_scaled() {
  for (int k = 0; k < K; ++k) {
    const int e = gain2_log<K>(k);
    if (haar_gain<K>(k) * static_cast<float>(1 << (e / 2)) != (e % 2 ? kSqrtHalf : 1.0f)) return false;
  }
  return true;
}

// Unnormalised Haar inverse of v[k] haar_gain2<K>(k) K: the
// band [h, 2h) enters with its weight h (a power of two: an exact product).
template <int K>
__device__ __forceinline__ void haar_inv_banded(float* v) {
#pragma unroll
  for (int half = 1; half <= K / 2; half *= 2) {
    float t[K];
#pragma unroll
    for (int j = 0; j < half; ++j) {
      t[2 * j] = fmaf(static_cast<float>(half), v[half + j], v[j]);
      t[2 * j + 1] = fmaf(-static_cast<float>(half), v[half + j], v[j]);
    }
#pragma unroll
    for (int j = 0; j < 2 * half; ++j) v[j] = t[j];
  }
}

// The next lane's value (lanes 15, 31, ..: 0).
__device__ __forceinline__ float next_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x101, 0xf, 0xf, true));
}

// One work item = one tile of references: stage-1 groups.  RECOMPUTE: the
// blocks' spectra are computed here from the image's pixels instead of
// gathered from the bior1.5 stack.
// Bound by vector issue and LDS cycles (80 and 60 % of the kernel's).  What is
// the same for a band or a chunk is taken out of the group's arithmetic where
// the result stays the same to the bit: thresholds on unscaled coefficients,
// powers of two kept until the weight, the coarse transform levels of all K
// blocks at once, neighbours from the next lane's register, block positions
// decoded once per tile.  580 -> 480 vector and 130 -> 100 LDS instructions per
// group of 16; kernel us: 512^2 58 -> 50, 4096^2 2535 -> 2130, 64 mixed images
// 3760 -> 3110.
template <int K, bool RECOMPUTE, int SHAPE>
__device__ __forceinline__ void group_ht_body(acc_t* acc,
                                              float (*scratch)[GroupCfg<K, true, SHAPE>::chunk * kBlockFloats],
                                              typename GroupCfg<K, true, SHAPE>::SlotTable& slots, const ImgRec& r,
                                              int R, const HtParams& hp, int item) {
  using Cfg = GroupCfg<K, true, SHAPE>;
  using T = typename Cfg::T;
  const GroupArgs g = make_args<T>(r.H, r.W, R);
  const int tyi = item / g.nTx, txi = item % g.nTx;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  slots.template load<Cfg::threads>(g, r.idx, tyi, txi);
  zero_acc(acc, g.FY * T::FXP);
  const int fy0 = kStep * tyi * T::py - g.R;
  const int fx0 = kStep * txi * T::px - g.R;
  float* xw = scratch[wave];
  const int a = lane >> 3, b = lane & 7;
  const float tau = r.sigma * (hp.ht_a - hp.ht_b * static_cast<float>(bior_level(lane)));
  const bool dc_lane = hp.keep_dc && lane == 0;
  // |v[k]| from which coefficient k is kept: k = 0, then by band
  constexpr int kBands = __builtin_ctz(K);
  const float tau_sqrt = smallest_kept(tau);
  static_assert(gains_are_scaled<K>(), "a power of two, or times sqrt(1/2)");
  auto kept_from = [&](int k) {
    const int e = gain2_log<K>(k);
    return (e % 2 ? tau_sqrt : tau) * static_cast<float>(1 << (e / 2));
  };
  const float kept_dc = dc_lane ? 0.0f : kept_from(0);
  float kept[kBands];
#pragma unroll
  for (int i = 0; i < kBands; ++i) kept[i] = kept_from(1 << i);
  acc_t* bw = r.partials;  // block-start weights
  float* own = xw + a * kScratchPitch + b;
  const float* below = own + (a < 7 ? kScratchPitch : 0);
  const float has_right = b < 7 ? 1.0f : 0.0f;

  const GroupWalk<T, Cfg::waves> walk{g, slots.pos, tyi, txi, wave, lane};
  const float* const stacks[1] = {r.stack_a};
  auto filter = [&](const float (&cur)[1][K], int j, int pos_v) {
    float v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = cur[0][k];
    // unnormalised Haar: coefficient k of the orthonormal transform is
    // haar_gain(k) * v[k]; the thresholds are on v[k], and the inverse takes
    // the bands with their weights h = K haar_gain^2: from here to the
    // weight, values are K times the orthonormal ones (exactly)
    haar_fwd_raw<K>(v);
    auto keep = [&](int k, float x) { return fabsf(x) >= (k == 0 ? kept_dc : kept[k == 0 ? 0 : 31 - __builtin_clz(k)]); };
    int nnz = 0;
    if (hp.weight_mode == 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        float x = v[k];
        asm volatile("" : "+v"(x));  // (apart from the selection below, which then folds |x| into its comparison)
        nnz += keep(k, x) ? 1 : 0;
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = keep(k, v[k]) ? v[k] : 0.0f;
    haar_inv_banded<K>(v);
    // inverse 2-D transform.  The two coarse levels are a 4 x 4 corner: up to 16
    // blocks' corners go through the scratch together (fuller waves than a
    // chunk's), and come back in the registers ll, a column per lane.
    constexpr int CH = Cfg::chunk;
    constexpr Mat8 S2 = bior_synthesis(2);
    constexpr Mat8 S4 = bior_synthesis(4);
    constexpr Mat8 S8 = bior_synthesis(8);
    constexpr int kCorner = 20, kCornerPitch = 5;  // conflict-free rows and columns
    constexpr int KC = K > 16 ? 16 : K;
    static_assert(KC * kCorner <= CH * kBlockFloats && KC * 4 <= kWave, "the corners fit the scratch and a wave");
    float ll[K / KC][4];
    auto line4 = [&](const float* x, float* y) { apply_mat<4>(S4, x, y); };
#pragma unroll
    for (int part = 0; part < K / KC; ++part) {
      wave_lds_sync();  // earlier reads of the scratch are done
      if (a < 4 && b < 4) {
#pragma unroll
        for (int k = 0; k < KC; ++k) xw[k * kCorner + a * kCornerPitch + b] = v[part * KC + k];
      }
      wave_lds_sync();
      transform_level<KC, 2, kCorner, kCornerPitch>(xw, lane, [&](const float* x, float* y) { apply_mat<2>(S2, x, y); });
      transform_rows<KC, 4, kCorner, kCornerPitch>(xw, lane, line4);
      transform_columns<KC, 4, kCorner, kCornerPitch>(xw, lane, line4, [&](int, int, int, const float (&y)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ll[part][i] = y[i];
      });
    }
    // the fine level, kChunk blocks at a time; the spatial total-variation
    // terms are read while a chunk is parked there
    float u[K];
    float tv = 0.0f;
#pragma unroll
    for (int c0 = 0; c0 < K; c0 += CH) {
      wave_lds_sync();  // earlier reads of the scratch are done
#pragma unroll
      for (int k = 0; k < CH; ++k) own[k * kBlockFloats] = v[c0 + k];
      wave_lds_sync();
      const int it = lane - 4 * (c0 % KC);  // corner column it % 4 of the chunk's block it / 4
      if (it >= 0 && it < 4 * CH) {
        float* col = xw + it / 4 * kBlockFloats + it % 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) col[i * kScratchPitch] = ll[c0 / KC][i];
      }
      wave_lds_sync();
      transform_level<CH, 8>(xw, lane, [&](const float* x, float* y) { apply_mat<8>(S8, x, y); });
#pragma unroll
      for (int k = 0; k < CH; ++k) u[c0 + k] = own[k * kBlockFloats];
      if (hp.weight_mode == 0) {
        // (lanes without a neighbour add 0)
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          tv = fmaf(fabsf(next_lane(u[c0 + k]) - u[c0 + k]), has_right, tv);
          tv += fabsf(below[k * kBlockFloats] - u[c0 + k]);
        }
      }
    }
    float w;
    if (hp.weight_mode == 0) {
#pragma unroll
      for (int k = 0; k + 1 < K; ++k) tv += fabsf(u[k + 1] - u[k]);
      w = r.eps / fmaf(wave_sum(tv), 1.0f / K, r.eps);
    } else if (hp.weight_mode == 1) {
      w = 1.0f / static_cast<float>(max(wave_sum_int(nnz), 1));
    } else {
      w = 1.0f;
    }
    accumulate<K, T>(acc, slots.fo + walk.ref(j) * K, u, w * (kFixScaleF / K), lane);
    add_block_weights<K>(bw, pos_v, w, lane);
  };
  if constexpr (RECOMPUTE) {
    for (int j = 0; j < walk.kGroups; ++j) {
      if (!walk.exists(j)) continue;
      const int pos_v = walk.template slot<K>(j);
      float cur[1][K];
      walk.template gather_pixels<K>(pos_v, r.noisy, cur);
      forward_blocks<K, Cfg::chunk>(xw, lane, cur[0]);
      filter(cur, j, pos_v);
    }
  } else {
    for_each_group<K, 1, Cfg::prefetch>(walk, stacks, filter);
  }
  flush_acc<T>(acc, g, fy0, fx0, numerator_sums(r));
}

// Unnormalised Haar inverse of v[k] wt[k], in place of v.
template <int K>
__device__ __forceinline__ void haar_inv_weighted(float* v, const float* wt) {
#pragma clang fp contract(off)
  v[0] *= wt[0];
#pragma unroll
  for (int half = 1; half <= K / 2; half *= 2) {
    float t[K];
#pragma unroll
    for (int j = 0; j < half; ++j) {
      t[2 * j] = fmaf(v[half + j], wt[half + j], v[j]);
      t[2 * j + 1] = fmaf(-v[half + j], wt[half + j], v[j]);
    }
#pragma unroll
    for (int j = 0; j < 2 * half; ++j) v[j] = t[j];
  }
}

// One work item = one tile of references: stage-2 groups.
// Bound by vector issue.  No factor common to a block, band or coefficient is
// multiplied in by itself: the DCT's output factors s = dct8_scale(a)
// dct8_scale(b) are left out of the pilot's stack and squared in the noisy one
// (as the inverse without its input factors wants them), and with the Haar
// gains they are on the noise variance; the inverse Haar's band weights h are
// on the gains, which enter its butterflies as FMAs; the aggregation weight is
// on the conversion to fixed point.  The column transform leaves a lane eight
// pixels of one column of a block, which it adds into the footprint from
// there: one address per column, rows by instruction offsets, no trip back
// through the scratch.
// At 80 registers two tiles of twelve waves share a CU.  Against one tile of
// sixteen waves with scaled transforms, a pixel of every block per lane and an
// address per block, kernel us: 512^2 91 -> 67, 1001 x 750 285 -> 205, 4096^2
// 4837 -> 3420, 64 mixed images 7604 -> 5110.
template <int K, int SHAPE>
__device__ __forceinline__ void group_wiener_body(acc_t* acc,
                                                  float (*scratch)[GroupCfg<K, false, SHAPE>::chunk * kBlockFloats],
                                                  typename GroupCfg<K, false, SHAPE>::SlotTable& slots,
                                                  const ImgRec& r, int R, int item) {
#pragma clang fp contract(off)  // the same roundings in every shape
  using Cfg = GroupCfg<K, false, SHAPE>;
  using T = typename Cfg::T;
  const GroupArgs g = make_args<T>(r.H, r.W, R);
  const int tyi = item / g.nTx, txi = item % g.nTx;
  const int lane0 = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  slots.template load<Cfg::threads>(g, r.idx, tyi, txi);
  zero_acc(acc, g.FY * T::FXP);
  const int fy0 = kStep * tyi * T::py - g.R;
  const int fx0 = kStep * txi * T::px - g.R;
  // noise variance in the units of the lane's squared pilot coefficients
  float s2 = r.sigma * r.sigma;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float inv = static_cast<float>(1.0 / (dct8_scale(i) * dct8_scale(i)));
    s2 *= (lane0 / 8 == i ? inv : 1.0f) * (lane0 % 8 == i ? inv : 1.0f);
  }
  acc_t* bw = r.partials;  // block-start weights
  const float* __restrict__ stack_n = r.stack_a;
  const float* __restrict__ stack_p = r.stack_b;
  constexpr int CH = Cfg::chunk;

  const GroupWalk<T, Cfg::waves> walk{g, slots.pos, tyi, txi, wave, lane0};
#pragma unroll 1
  for (int j = 0; j < walk.kGroups; ++j) {
    if (!walk.exists(j)) continue;
    const int pos_v = walk.template slot<K>(j);
    // what follows from the lane is formed again for each group: kept through
    // the loop it would not fit the registers
    int lane = lane0;
    float sv = s2;
    asm volatile("" : "+v"(lane), "+v"(sv));
    float* xw = scratch[wave];
    const int a = lane >> 3, b = lane & 7;
    // the pilot's spectra, turned into the Wiener gains; the noisy spectra are
    // loaded after them, so that the two are never in flight together
    float wt[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
      wt[k] = load_block_lane(stack_p + static_cast<size_t>(__builtin_amdgcn_readlane(pos_v, k)) * 64, lane);
    haar_fwd_raw<K>(wt);
    // h b^2 / (b^2 + sigma^2), b^2 = haar_gain2 x and h = K haar_gain2 >= 1 the
    // band's weight (both powers of two); their squares' sum without h
    float sw2 = 0.0f, band = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float h = K * haar_gain2<K>(k), x = wt[k] * wt[k];
      wt[k] = x * __builtin_amdgcn_rcpf(fmaf(x, 1.0f / h, sv * (K / (h * h))));
      if (k == 0 && lane == 0) wt[k] = 1.0f;
      band = fmaf(wt[k], wt[k], band);
      if (k == 0 || k + 1 == K || haar_gain2<K>(k + 1) != haar_gain2<K>(k)) {
        sw2 = fmaf(band, 1.0f / (h * h), sw2);
        band = 0.0f;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    float v[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
      v[k] = load_block_lane(stack_n + static_cast<size_t>(__builtin_amdgcn_readlane(pos_v, k)) * 64, lane);
    const float w = 1.0f / wave_sum(sw2);
    haar_fwd_raw<K>(v);
    haar_inv_weighted<K>(v, wt);
    const double w_scaled = static_cast<double>(w) * (kFixScale / K);
#pragma unroll
    for (int c0 = 0; c0 < K; c0 += CH) {
      wave_lds_sync();  // earlier reads of the scratch are done
#pragma unroll
      for (int k = 0; k < CH; ++k) xw[k * kBlockFloats + a * kScratchPitch + b] = v[c0 + k];
      wave_lds_sync();
      // lane (a, b) of the chunk: row b, then column b, of block a
      if (CH == 8 || a < CH) {
        float* line = xw + a * kBlockFloats + b * kScratchPitch;
        float x[8], y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = line[i];
        dct8_inv_raw(x, y);
#pragma unroll
        for (int i = 0; i < 8; ++i) line[i] = y[i];
      }
      wave_lds_sync();
      if (CH == 8 || a < CH) {
        const float* col = xw + a * kBlockFloats + b;
        float x[8], y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = col[i * kScratchPitch];
        dct8_inv_raw(x, y);
        acc_t* cell = cell_at(acc, slots.fo[walk.ref(j) * K + c0 + a]) + b;
#pragma unroll
        for (int i = 0; i < 8; ++i) atomicAdd(cell + i * T::FXP, static_cast<acc_t>(to_fixed_product(y[i], w_scaled)));
      }
    }
    add_block_weights<K>(bw, pos_v, w, lane);
  }
  flush_acc<T>(acc, g, fy0, fx0, numerator_sums(r));
}

// (the second launch bound is the minimum number of waves per SIMD)
template <int K, bool BATCH, bool RECOMPUTE, int SHAPE>
__global__ __launch_bounds__((GroupCfg<K, true, SHAPE>::threads),
                             (GroupCfg<K, true, SHAPE>::min_waves_per_simd)) void group_ht_kernel(ImgRec one,
                                                                                                  WorkList wl, int R,
                                                                                                  HtParams hp) {
  using Cfg = GroupCfg<K, true, SHAPE>;
  __shared__ acc_t acc[Cfg::T::entries];
  __shared__ float scratch[Cfg::waves][Cfg::chunk * kBlockFloats];
  __shared__ typename Cfg::SlotTable slots;
  for_item<BATCH>(one, wl, [&](const ImgRec& r, int item) {
    group_ht_body<K, RECOMPUTE, SHAPE>(acc, scratch, slots, r, R, hp, item);
  });
}

// the block-start weights and numerator sums the aggregation adds into (the
// bior1.5 stack launch clears them otherwise)
__global__ void clear_weights_kernel(acc_t* __restrict__ w, size_t n) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    w[i] = 0;
}

template <int K, bool BATCH, int SHAPE>
__global__ __launch_bounds__((GroupCfg<K, false, SHAPE>::threads),
                             (GroupCfg<K, false, SHAPE>::min_waves_per_simd)) void group_wiener_kernel(ImgRec one,
                                                                                                       WorkList wl,
                                                                                                       int R) {
  using Cfg = GroupCfg<K, false, SHAPE>;
  __shared__ acc_t acc[Cfg::T::entries];
  __shared__ float scratch[Cfg::waves][Cfg::chunk * kBlockFloats];
  __shared__ typename Cfg::SlotTable slots;
  for_item<BATCH>(one, wl, [&](const ImgRec& r, int item) {
    group_wiener_body<K, SHAPE>(acc, scratch, slots, r, R, item);
  });
}

// One work item = 256 pixels of one row: the numerator sum of each pixel over
// the 8 x 8 box sum of the block-start weights ending at it, then normalise.
__device__ __forceinline__ void reduce_body(acc_t* colsum, const ImgRec& r, int final_stage, int item) {
  const auto bw = to_global(static_cast<const acc_t*>(r.partials));
  const auto nums = to_global(static_cast<const acc_t*>(numerator_sums(r)));
  const auto out = to_global(final_stage ? r.out : r.basic);
  const bool with_q = !final_stage && r.q != nullptr;
  const auto q = to_global(r.q);
  const int H = r.H, W = r.W;
  const int xb = (W + kReduceThreads - 1) / kReduceThreads;
  const int y = item / xb;
  const int xs = (item % xb) * kReduceThreads;
  const int x = xs + static_cast<int>(threadIdx.x);
  const bool active = x < W;
  const size_t o = static_cast<size_t>(y) * W + x;
  // the numerator's load is issued before the weights' column sums below, so
  // the two round trips overlap
  const acc_t num = active ? nums[o] : 0;
  // colsum[c] = sum over rows y-7..y of the weights at column xs - 7 + c
  // (H, W >= 8, so a row index wraps at most once; so does a column index
  // when W covers a chunk and its 7-column margin)
  const bool wide = W >= kReduceThreads + 7;
  constexpr int kCols = kReduceThreads + 7;
  auto column = [&](int c) {
    const int xi = xs - 7 + c;
    return wide ? xi + (xi < 0 ? W : (xi >= W ? -W : 0)) : pmod(xi, W);
  };
  auto rows_of = [&](int xi, acc_t (&v)[8]) {
#pragma unroll
    for (int dy = 0; dy < 8; ++dy) {
      const int yy = y - dy < 0 ? y - dy + H : y - dy;
      v[dy] = bw[static_cast<size_t>(yy) * W + xi];
    }
  };
  auto sum8 = [](const acc_t (&v)[8]) {
    acc_t sum = 0;
#pragma unroll
    for (int dy = 0; dy < 8; ++dy) sum += v[dy];
    return sum;
  };
  // column c = thread, and the last 7 columns in the first wave, whose two
  // sets of loads go out together (one round trip for the block)
  const int c0 = static_cast<int>(threadIdx.x);
  acc_t v0[8];
  rows_of(column(c0), v0);
  if (threadIdx.x < kWave) {
    const int c1 = min(c0 + kReduceThreads, kCols - 1);
    acc_t v1[8];
    rows_of(column(c1), v1);
    if (c0 + kReduceThreads < kCols) colsum[c1] = sum8(v1);
  }
  colsum[c0] = sum8(v0);
  static_assert(kCols - kReduceThreads <= kWave, "the extra columns fit the first wave");
  __syncthreads();
  if (active) {
    acc_t den = 0;
#pragma unroll
    for (int dx = 0; dx < 8; ++dx) den += colsum[threadIdx.x + 7 - dx];
    const float v = static_cast<float>(static_cast<double>(static_cast<long long>(num)) /
                                       static_cast<double>(static_cast<long long>(den)));
    out[o] = v;
    if (with_q) {
      const double d = static_cast<double>(fminf(fmaxf(v, 0.0f), 1.0f));
      q[o] = static_cast<uint16_t>(floor(d * 65535.0 + 0.5));
    }
  }
}

template <bool BATCH>
__global__ __launch_bounds__(kReduceThreads) void reduce_kernel(ImgRec one, WorkList wl, int final_stage) {
  __shared__ acc_t colsum[kReduceThreads + 8];
  for_item<BATCH>(one, wl, [&](const ImgRec& r, int item) { reduce_body(colsum, r, final_stage, item); });
}

__global__ void quantize_kernel(const float* __restrict__ in, uint16_t* __restrict__ out, size_t n) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const double d = static_cast<double>(fminf(fmaxf(in[i], 0.0f), 1.0f));
    out[i] = static_cast<uint16_t>(floor(d * 65535.0 + 0.5));
  }
}

}  // namespace

size_t partials_bytes(int H, int W) { return aggregation_entries(H, W) * sizeof(acc_t); }

template <typename T>
static int tiles_of(int H, int W) {
  const GroupArgs g = make_args<T>(H, W, 0);
  return g.nTy * g.nTx;
}

// items of the batch launches (two-tile shape)
int group_items_for(int H, int W) { return tiles_of<Tile<8, 8>>(H, W); }

int reduce_items_for(int H, int W) { return reduce_items(H, W); }

// The shapes of a single image's launches, by its tiles of 8 x 8 references and
// the 256 CUs.  A CU takes two tiles at a time.  Below 256 tiles CUs idle unless
// the tiles are smaller, from 193 on hardly any; just above, a few CUs work on
// two tiles while the rest have one.  Small tiles pay for it with more footprint
// cells to clear and add per reference, the more the wider the window.
// Kernel us, 8 x 8 | 4 x 4 | 2 x 4 references, windows of 39 and of 21:
//   tiles  first stage K = 16              Wiener K = 16                  Wiener K = 32
//     36   26 13 12    25 13 10            20 11 10    20 11 9            35 15 12    34 15 12
//     64   26 15 16    26 14 13            20 13 13    20 12 12           35 18 17    35 17 16
//    121   26 21 25    26 19 20            21 17 22    20 16 19           36 25 28    35 23 25
//    196   28 28 36    27 22 26            22 24 30    21 22 26           38 37 41    36 33 34
//    256   31 37 47    28 30 34            26 33 38    24 28 32           43 49 51    39 44 40
//    289   44 42 53    41 34 40            36 37 43    33 32 36           59 56 61    55 48 48
//    324   45 45 56    41 38 42            37 41 47    34 35 39           61 63 66    56 55 52
//    361   46 48 59    42 39 44            38 42 50    35 36 41           65 65 71    57 55 56
//    400   47 53 67    43 44 50            41 47 56    36 40 44           68 70 79    60 64 59
//   1849  161 213 263  141 152 175        177 194 241  162 164 183       290 307 349  262 248 266
// Smaller K go like K = 16, the first stage's K = 32 like the Wiener kernel's.
// From 257 tiles on, 4 x 4 references where they win: the first stage and Wiener
// groups of 32, up to 300 tiles, 380 for windows up to 31.
static GroupShape shape_for(int H, int W, int R, bool above_256) {
  const int t = tiles_of<Tile<8, 8>>(H, W);
  if (t <= 64) return kTiny;
  return t <= 192 || (above_256 && t > 256 && t <= (R > 15 ? 300 : 380)) ? kSmall : kTwoTiles;
}

template <int K, int SHAPE>
static hipError_t launch_ht_shape(const ImgRec& one, const WorkList* wl, int R, const HtParams& hp, int recompute,
                                  hipStream_t st) {
  using Cfg = GroupCfg<K, true, SHAPE>;
  if (!wl) {
    const dim3 grid(tiles_of<typename Cfg::T>(one.H, one.W));
    if (recompute)
      hipLaunchKernelGGL((group_ht_kernel<K, false, true, SHAPE>), grid, dim3(Cfg::threads), 0, st, one, WorkList{}, R,
                         hp);
    else
      hipLaunchKernelGGL((group_ht_kernel<K, false, false, SHAPE>), grid, dim3(Cfg::threads), 0, st, one, WorkList{},
                         R, hp);
  } else if constexpr (SHAPE <= kOneTile) {
    if (recompute) return hipErrorInvalidValue;  // batches read the stack
    if (wl->total <= 0) return hipSuccess;
    hipLaunchKernelGGL((group_ht_kernel<K, true, false, SHAPE>), batch_grid(wl->total), dim3(Cfg::threads), 0, st, one,
                       *wl, R, hp);
  }
  return hipGetLastError();
}

template <int K>
static hipError_t launch_ht_k(const ImgRec& one, const WorkList* wl, int R, const HtParams& hp, int recompute,
                              int shape, hipStream_t st) {
  if constexpr (K <= 16)
    if (shape == 1) return launch_ht_shape<K, kOneTile>(one, wl, R, hp, recompute, st);
  switch (wl ? kTwoTiles : shape_for(one.H, one.W, R, true)) {
    case kTiny: return launch_ht_shape<K, kTiny>(one, wl, R, hp, recompute, st);
    case kSmall: return launch_ht_shape<K, kSmall>(one, wl, R, hp, recompute, st);
    default: return launch_ht_shape<K, kTwoTiles>(one, wl, R, hp, recompute, st);
  }
}

hipError_t launch_group_ht(const ImgRec& one, const WorkList* wl, int R, int K, float ht_a, float ht_b,
                           int weight_mode, int keep_dc, int recompute, int shape, hipStream_t st) {
  const HtParams hp{ht_a, ht_b, weight_mode, keep_dc};
  switch (K) {
    case 2: return launch_ht_k<2>(one, wl, R, hp, recompute, shape, st);
    case 4: return launch_ht_k<4>(one, wl, R, hp, recompute, shape, st);
    case 8: return launch_ht_k<8>(one, wl, R, hp, recompute, shape, st);
    case 16: return launch_ht_k<16>(one, wl, R, hp, recompute, shape, st);
    case 32: return launch_ht_k<32>(one, wl, R, hp, recompute, shape, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_clear_weights(const ImgRec& one, hipStream_t st) {
  const size_t n = aggregation_entries(one.H, one.W);
  const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(clear_weights_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, one.partials, n);
  return hipGetLastError();
}

template <int K, int SHAPE>
static hipError_t launch_wiener_shape(const ImgRec& one, const WorkList* wl, int R, hipStream_t st) {
  using Cfg = GroupCfg<K, false, SHAPE>;
  if (!wl) {
    hipLaunchKernelGGL((group_wiener_kernel<K, false, SHAPE>), dim3(tiles_of<typename Cfg::T>(one.H, one.W)),
                       dim3(Cfg::threads), 0, st, one, WorkList{}, R);
  } else if constexpr (SHAPE == kTwoTiles) {
    if (wl->total <= 0) return hipSuccess;
    hipLaunchKernelGGL((group_wiener_kernel<K, true, SHAPE>), batch_grid(wl->total), dim3(Cfg::threads), 0, st, one,
                       *wl, R);
  }
  return hipGetLastError();
}

template <int K>
static hipError_t launch_wiener_k(const ImgRec& one, const WorkList* wl, int R, hipStream_t st) {
  switch (wl ? kTwoTiles : shape_for(one.H, one.W, R, K > 16)) {
    case kTiny: return launch_wiener_shape<K, kTiny>(one, wl, R, st);
    case kSmall: return launch_wiener_shape<K, kSmall>(one, wl, R, st);
    default: return launch_wiener_shape<K, kTwoTiles>(one, wl, R, st);
  }
}

hipError_t launch_group_wiener(const ImgRec& one, const WorkList* wl, int R, int K, hipStream_t st) {
  switch (K) {
    case 2: return launch_wiener_k<2>(one, wl, R, st);
    case 4: return launch_wiener_k<4>(one, wl, R, st);
    case 8: return launch_wiener_k<8>(one, wl, R, st);
    case 16: return launch_wiener_k<16>(one, wl, R, st);
    case 32: return launch_wiener_k<32>(one, wl, R, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_reduce(const ImgRec& one, const WorkList* wl, int final_stage, hipStream_t st) {
  if (!wl) {
    hipLaunchKernelGGL((reduce_kernel<false>), dim3(reduce_items(one.H, one.W)), dim3(kReduceThreads), 0, st, one,
                       WorkList{}, final_stage);
  } else {
    if (wl->total <= 0) return hipSuccess;
    hipLaunchKernelGGL((reduce_kernel<true>), batch_grid(wl->total), dim3(kReduceThreads), 0, st,
                       one, *wl, final_stage);
  }
  return hipGetLastError();
}

hipError_t launch_quantize(const float* in, uint16_t* out, size_t n, hipStream_t st) {
  const size_t blocks = std::min<size_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(quantize_kernel, dim3(static_cast<unsigned>(blocks > 0 ? blocks : 1)), dim3(256), 0, st, in,
                     out, n);
  return hipGetLastError();
}

}  // namespace gbm3d
