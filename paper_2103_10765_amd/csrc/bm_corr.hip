// Block matching in the correlation form of Theorem 1 (Sec. 2), on the
// matrix cores.  Same result as the shift-wise kernel: for every reference the
// K-1 smallest keys dist * 2048 + rank over the search window (dist the exact
// integer ||a - b||^2), reference in slot 0.
//
// A workgroup of eight waves owns a 4 x 4 tile of references (step 3); the
// union of their windows is a square of at most 48 x 48 candidate positions,
// taken in 4 x 4 blocks that are dealt to the waves.  Exact keys of all pairs
// cost an order of magnitude more vector instructions than the products
// themselves, and only K of 1521 are wanted, so the kernel first finds, from
// approximate distances, a set of little more than K candidates per reference
// that provably holds the answer, and forms exact keys for that set alone:
//
//  1. Pixels less the tile's centre pixel, halved, are rounded to f16 (a~),
//     and one f16 product of 16 candidates x 16 references with the
//     accumulator started at (N(a~) + N(b~)) / 2 (N the squared norm) leaves
//     the half distance ||a~ - b~||^2 / 2 of every pair without a vector
//     instruction.  Each lane keeps its 72 half distances, truncated to bf16
//     and packed in 36 registers, and the smallest of each of its four
//     columns: a reference has 8 waves x 4 rows x 4 columns = 128 group bests.
//  2. The K-th smallest of the 128 bests is a bound: K distinct candidates (one
//     may be the reference itself) are at least that good.  Candidates of a
//     group lie far apart, so neighbours, which are good together, fall into
//     different groups: on noisy images 18 candidates of 1521 pass the bound
//     for K = 16, on first estimates 37 for K = 32.  The bound is widened by
//     what the roundings can do (widened_bound), so that no candidate of
//     the exact answer is lost.
//  3. Candidates past the bound go to a queue in LDS, one thread forms each
//     one's exact integer distance from the u16 pixels, and a key's rank among
//     its reference's keys is its slot.
//
// Ties: candidates that are exactly as good are told apart by a position
// term far below one unit of distance, which survives while the norms are
// small (constant regions); elsewhere they all pass and the exact keys decide
// (long lists are cut by the (K-1)-th smallest of their first kSample keys
// before the ranks are counted).
//
// The widening grows with the reference's distance from the centre pixel and
// with the noise it does not shrink: on a tile of two flat levels, on text,
// graphics and periodic textures hundreds of candidates of a reference pass.
// Such a tile (hard_tile, kLongList) goes through an exact pass: <a, b> from four
// int8 products of the pixels' bytes, keys in float64 (integers below 2^49), the
// group bests' exact K-th smallest, position and all, as the limit, and a second
// pass over the products that marks the keys up to it: 18 / 40 candidates per
// reference again, whatever the image.  It costs such a tile 16 000 vector
// instructions.  Matching 512^2, K = 16 / 32, us, without the pass | with it |
// by the earlier kernel of exact keys alone, which any image took: two levels
// 4000 and 60000 with noise of 128 110 / 187 | 88 / 123 | 86 / 112, checkerboard
// 432 / 445 | 115 / 120 | 82 / 107, texture of period 8 186 / 355 | 123 / 146 | 88 / 111,
// strokes on white 150 / 273 | 121 / 169 | 90 / 115; noisy 47 / 59 | 47 / 59 | 91 / 115.
//
// Bound by LDS cycles and vector issue about equally: per tile 6 200 LDS
// cycles (the 144 blocks' operands 2 600 of them) and 9 000 vector
// instructions at K = 16, and by the latency of its eight phases, so three
// workgroups share a CU (80 registers, 53 KB of LDS; none in scratch memory but
// for one to three of the stacks' workgroups): with unpacked half distances and
// two workgroups per CU the 4096^2 image took 3.0 ms instead of 2.6, and with
// f16 copies 22 instead of 8 banks apart 2.6 instead of 2.45.
// Against the earlier kernel (exact float64 keys of all pairs from int8
// products and a norm table), K = 16 / 32, noisy images: 512^2 87 / 112 -> 46 / 59
// us, 4096^2 2.93 / 3.56 -> 2.46 / 3.0 ms, 128^2 26 / 31 -> 11 / 16 us.
#include "common.h"
#include "kernels.h"
#include "match_bound.h"
#include "stack_body.h"

namespace gbm3d {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kPrune = 64;                       // longer lists are cut before their keys are ranked
constexpr int kSample = 256;                      // by a bound from so many of their keys
// A tile goes through the exact pass where its lists hold more candidates than
// this in all, or three of them more than kLongList: lists of many hundreds are
// slow to cut and rank, and a thousand candidates more cost as much as the pass.
// (Noisy images have some 20 candidates per reference at K = 16, 45 at K = 32.  A
// first estimate has a few references with lists of 450 to 1000 in tiles of 1000 to
// 2000 in all, which are the tail of a small image's launch: sent through the pass
// for one long list they made two-stage calls of 128^2 up to 12 %, of 200 x 256 up
// to 7 % slower.  Two-stage calls of 16 noisy images of 512^2, of a 128^2 image of
// two flat levels, of one of strokes, us: one list, 1700 / 2500 in all at K = 16 / 32
// 260, 86, 109; three lists, 1824 / 2848 257, 103, 119; three, 2240 / 2880 258, 104,
// 127; four, 1824 / 2848 257, 105, 119, levels at 512^2 405 instead of 377; without
// the pass 262, 198, 180.)
__host__ __device__ constexpr int hard_tile(int K) { return 800 + 64 * K; }
constexpr int kLongList = 448;

constexpr int max2(int a, int b) { return a > b ? a : b; }
constexpr int min2(int a, int b) { return a < b ? a : b; }

// A tile's region and its LDS for a grid of 2 Q x 4 C candidate blocks, of which
// a wave takes Q x C.  Windows up to 7, 15, 23 and 39 have grids of their own: a
// fixed region of 12 x 12 blocks' size made every window up to 17 cost the same
// (1024^2, K = 2 / 8, us: window 7 92 / 98 -> 59 / 64, window 15 95 / 101 -> 76 / 81).
template <int Q, int C>
struct Geo {
  static constexpr int kSteps = Q * C;
  static constexpr int kCandRows = 8 * Q, kCandCols = 16 * C;  // candidate positions
  static constexpr int kRows = kCandRows + 7;                  // pixel rows
  static constexpr int kGroups = kCandCols / 4 + 1;            // 4-pixel column groups of the f16 planes
  static constexpr int kPixCols = kCandCols + 8;               // columns of the u16 planes
  static constexpr int kPixPitch = 2 * kPixCols;               // bytes per u16 plane row
  static constexpr int kPixPlane = kRows * kPixPitch;
  // The f16 plane is kept in four copies shifted by 0..3 pixels, so that the
  // eight pixels of a candidate row start at an 8-byte boundary of the copy its
  // column asks for.  The LDS serves 16 lanes of an 8-byte read at a time from 32
  // banks: with rows 26, 18 or 10 words apart and copies 8 words apart (modulo
  // 32) the four rows x four copies that 16 candidates read fall on all 32 banks
  // once.
  static constexpr int kF16Pitch = 8 * kGroups;
  static constexpr int kF16Copy = (kRows * kF16Pitch - 32 + 127) / 128 * 128 + 32;
  static_assert(kF16Pitch / 4 % 8 == 2 && kF16Copy % 128 == 32 && kF16Copy >= kRows * kF16Pitch, "copies eight banks apart");
  static constexpr int kInitPitch = 2 * kF16Pitch;   // bytes per row of the accumulator starts (float)
  static constexpr int kSumPitch = 4 * kCandCols;    // bytes per row of the horizontal norm sums (float)
  static constexpr int kBestPitch = 2 * kWaves * 16 + 8;  // bytes per reference of the 128 group bests (bf16)

  static constexpr int pix0 = 0;                         // u16 plane, and the same shifted by one pixel:
  static constexpr int pix1 = pix0 + kPixPlane;          // any candidate row starts at a word of one of them
  static constexpr int f16 = (pix1 + kPixPlane + 15) / 16 * 16;
  // the accumulator starts replace the horizontal norm sums they come from
  static constexpr int sums = (f16 + 4 * kF16Copy + 15) / 16 * 16;
  static constexpr int init = sums;
  static constexpr int codes = (sums + max2(kRows * kSumPitch, kCandRows * kInitPitch) + 15) / 16 * 16;
  static constexpr int best = codes;                     // dead before the codes are written
  // candidates with exact keys at a time (lists padded to eights); the keys take
  // the place of the products' operands, which are dead by then
  static constexpr int kQueue = min2(3072, (codes - f16) / 64 * 8);
  // The exact pass: norms with position (double, rows two entries longer than
  // the candidates' so that four rows fall on different banks) and, before them,
  // their horizontal sums, over the products' operands; 128 group bests
  // (double), over the starts and codes.
  static constexpr int kNormPitch = kCandCols + 2;
  static constexpr int norms = f16;
  static constexpr int kExactPitch = 8 * (kWaves * 16 + 2);
  static constexpr int exact = sums;
  static_assert(8 * kRows * kCandCols <= 4 * kF16Copy && 8 * kCandRows * kNormPitch <= 4 * kF16Copy, "norms fit the operands' area");
  static constexpr int bound = (max2(codes + max2(16 * kBestPitch, 2 * kQueue), exact + 16 * kExactPitch) + 15) / 16 * 16;
  // int[16]: packed half distances up to it pass
  static constexpr int count = bound + 64;               // int[16]: candidates past each reference's bound
  static constexpr int start = count + 64;               // int[16]: their first place in the queue
  static constexpr int kept = start + 64;                // int[16]: keys left of a long list
  static constexpr int limit = kept + 64;                // double[16]: exact keys up to it pass
  static constexpr int bytes = limit + 128;
  static constexpr int keys = f16;
  static constexpr int kMaxWindow = kCandRows < kCandCols ? kCandRows - 9 : kCandCols - 9;
  static_assert(kQueue >= kMaxWindow * kMaxWindow + 7, "one reference always fits the queue");
  static_assert(kGroups % 2 == 1 && kPixCols / 8 * 2 == kGroups + 1, "f16 planes end in half an eight-column item");
};
constexpr int kMaxNb = (2 * kMaxR + 10 + 3) / 4;  // candidate blocks per axis: 12
static_assert(Geo<6, 3>::bytes <= 160 * 1024 / 3 / 1280 * 1280, "three workgroups per CU");

__host__ __device__ constexpr int blocks_per_axis(int R) { return (2 * R + 10 + 3) / 4; }

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

__host__ __device__ constexpr int corr_items(int H, int W) {
  return ((H + kStep - 1) / kStep + 3) / 4 * (((W + kStep - 1) / kStep + 3) / 4);
}

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) float lds_float;

// 16 bytes at an 8-byte boundary
__device__ __forceinline__ f16x8 read_row(const lds_byte* p) {
  typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
  const u32x2 a = *(const lds_u32x2*)p, b = *(const lds_u32x2*)(p + 8);
  return __builtin_bit_cast(f16x8, u32x4{a.x, a.y, b.x, b.y});
}

__device__ __forceinline__ unsigned join(unsigned lo, unsigned hi) { return __builtin_amdgcn_alignbit(hi, lo, 16); }

// x[0]^2 + x[1]^2 of a pair of f16
__device__ __forceinline__ float square2(unsigned x) {
  const f16x2 h = __builtin_bit_cast(f16x2, x);
  return __builtin_amdgcn_fdot2(h, h, 0.0f, false);
}

// Exact key of reference block (ry, rx) and candidate (cy, cx) of the tile's
// pixel planes, rank the candidate's displacement rank.  |a - b| is formed on
// packed u16 and its square from byte digits, 65536 hh + 512 hl + ll, each
// sum of 64 terms below 2^23.
template <typename G>
__device__ __forceinline__ double exact_key(const unsigned char* smem, int ry, int rx, int cy, int cx, int rank) {
  const unsigned char* pa = smem + ((cx & 1) ? G::pix1 : G::pix0) + cy * G::kPixPitch + 2 * (cx & ~1);
  const unsigned char* pb = smem + ((rx & 1) ? G::pix1 : G::pix0) + ry * G::kPixPitch + 2 * (rx & ~1);
  unsigned hh = 0, hl = 0, ll = 0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const unsigned* a = reinterpret_cast<const unsigned*>(pa + r * G::kPixPitch);
    const unsigned* b = reinterpret_cast<const unsigned*>(pb + r * G::kPixPitch);
    unsigned d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u16x2 x = __builtin_bit_cast(u16x2, a[i]), y = __builtin_bit_cast(u16x2, b[i]);
      const u16x2 e = __builtin_elementwise_max(x, y) - __builtin_elementwise_min(x, y);
      d[i] = __builtin_bit_cast(unsigned, e);
    }
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      const unsigned h = __builtin_amdgcn_perm(d[i + 1], d[i], 0x07050301u);
      const unsigned l = __builtin_amdgcn_perm(d[i + 1], d[i], 0x06040200u);
      hh = __builtin_amdgcn_udot4(h, h, hh, false);
      hl = __builtin_amdgcn_udot4(h, l, hl, false);
      ll = __builtin_amdgcn_udot4(l, l, ll, false);
    }
  }
  const double dist = fma(static_cast<double>(hh), 65536.0, fma(static_cast<double>(hl), 512.0, static_cast<double>(ll)));
  return fma(dist, 2048.0, static_cast<double>(rank));
}

// The exact pass takes pixels as 256 h + l with signed bytes h and l, z - 32896:
// z's bytes with their top bits flipped.
constexpr int kMid = 32896;
// a key outside the window, and the high word of one (above it)
constexpr double kOutside = 1e300;
constexpr unsigned kOutsideHigh = 0x7FE00000u;

struct Digits {
  i32x4 h, l;
};

// two rows of eight pixels (at a word of a flipped plane), and their digits
struct Rows {
  unsigned a[4], b[4];
};
template <typename G>
__device__ __forceinline__ Rows read_rows(const lds_byte* p) {
  typedef const __attribute__((address_space(3))) unsigned* lds_words;
  const lds_words a = (lds_words)p, b = (lds_words)(p + G::kPixPitch);
  return {{a[0], a[1], a[2], a[3]}, {b[0], b[1], b[2], b[3]}};
}
__device__ __forceinline__ Digits digits_of(const Rows& r) {
  auto high = [](unsigned x, unsigned y) { return static_cast<int>(__builtin_amdgcn_perm(y, x, 0x07050301u)); };
  auto low = [](unsigned x, unsigned y) { return static_cast<int>(__builtin_amdgcn_perm(y, x, 0x06040200u)); };
  return {i32x4{high(r.a[0], r.a[1]), high(r.a[2], r.a[3]), high(r.b[0], r.b[1]), high(r.b[2], r.b[3])},
          i32x4{low(r.a[0], r.a[1]), low(r.a[2], r.a[3]), low(r.b[0], r.b[1]), low(r.b[2], r.b[3])}};
}

// m = 2 m + the lane's bit
__device__ __forceinline__ void shift_in(unsigned& m, unsigned long long bit) {
  unsigned long long carry;
  asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(m), "=s"(carry) : "0"(m), "s"(bit));
}

// The candidate row of a wave's block (q, k) in the exact pass.
__device__ __forceinline__ int exact_row(int wave, int q, int k) { return 8 * q + ((wave - q - 3 * k) & 7); }

// flips the top bits of the planes' bytes (and back)
template <typename G>
__device__ __forceinline__ void flip_digits(unsigned char* smem, int tid) {
  static_assert(G::pix0 == 0 && G::pix1 == G::kPixPlane && G::kPixPlane % 8 == 0, "one run of words");
  unsigned* w = reinterpret_cast<unsigned*>(smem);
  for (int i = tid; i < 2 * G::kPixPlane / 4; i += kThreads) w[i] ^= 0x80808080u;
}

__device__ __forceinline__ unsigned high_word(double x) {
  return static_cast<unsigned>(__builtin_bit_cast(unsigned long long, x) >> 32);
}

// How many of the first n entries of list (16-byte aligned, filled up to a
// multiple of eight with infinities) lie below key.
__device__ __forceinline__ int entries_below(const double* list, int n, double key) {
  const f64x2* p = reinterpret_cast<const f64x2*>(list);
  int below = 0;
  for (int i = 0; i < n; i += 8, p += 4) {
    const f64x2 a = p[0], b = p[1], c = p[2], d = p[3];
    below += (a.x < key) + (a.y < key) + (b.x < key) + (b.y < key) + (c.x < key) + (c.y < key) + (d.x < key) +
             (d.y < key);
  }
  return below;
}

// One work item: the 4 x 4 references of a tile (raster order).  Wave
// (wy, wx) = (wave / 4, wave % 4) takes the blocks of rows 2 q + wy and columns
// 4 k + wx, q < Q, k < C: a group's candidates (one wave, row g, column i) are
// at least 8 rows or 16 columns apart, so no two of a cluster share a group,
// and a block's place is its wave's plus a constant.  Q x C covers the grid of
// blocks_per_axis(R) squared; WIDE: it is 12 x 12 (R >= 18), where the blocks
// of the middle rows and columns lie inside every window.
template <int Q, int C, bool WIDE>
__device__ __forceinline__ void corr_body(unsigned char* smem, const uint16_t* __restrict__ img_,
                                          int16_t* __restrict__ idx_, int H, int W, int R, int K, int item) {
  using G = Geo<Q, C>;
  const auto img = to_global(img_);
  const auto idx = to_global(idx_);
  const int nRy = (H + kStep - 1) / kStep, nRx = (W + kStep - 1) / kStep;
  const int tiles_x = (nRx + 3) / 4;
  const int S = 2 * R + 1, nb = blocks_per_axis(R), rows = 4 * nb + 7;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
  const int g = lane >> 4, n = lane & 15, u = n >> 2, v = n & 3;
  const int p0 = item / tiles_x * 4, q0 = item % tiles_x * 4;
  const int y0 = kStep * p0 - R, x0 = kStep * q0 - R;

  // the u16 plane: rows y0 .., columns x0 .. x0 + 55, a wave a row and a lane
  // a column, all loads issued before the first store; rows and columns wrap
  // at most once when the image is larger than the region and its margin
  {
    static_assert(G::kPixCols <= kWave, "a row per wave");
    constexpr int kIter = (G::kRows + kWaves - 1) / kWaves;
    const int xl = x0 + lane, x = W >= kWave + kMaxR ? xl + (xl < 0 ? W : (xl >= W ? -W : 0)) : pmod(xl, W);
    unsigned short z[kIter];
    const bool near = H >= G::kRows + kMaxR;
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
      const int r = wave + it * kWaves;
      int y = y0 + r;
      y = near ? y + (y < 0 ? H : (y >= H ? -H : 0)) : pmod(y, H);
      if (r < rows) z[it] = (img + static_cast<size_t>(y) * W)[x];
    }
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
      const int r = wave + it * kWaves;
      if (r < rows && lane < G::kPixCols)
        *reinterpret_cast<uint16_t*>(smem + G::pix0 + r * G::kPixPitch + 2 * lane) = z[it];
    }
  }
  if (tid < 16) reinterpret_cast<int*>(smem + G::count)[tid] = 0;
  __syncthreads();

  // the shifted u16 plane, the f16 copies and the horizontal norm sums, eight
  // columns per item.  Sums of eight squares are formed in one association
  // for every column, so equal blocks get equal norms.
  {
    const unsigned centre = *reinterpret_cast<const uint16_t*>(smem + G::pix0 + (R + 8) * G::kPixPitch + 2 * (R + 8));
    const float shift = -0.5f * static_cast<float>(centre);
    constexpr int kCols = G::kPixCols / 8;  // 7
    static_assert(G::kRows * kCols <= kThreads, "one item per thread");
    const int r = tid / kCols, q = tid - r * kCols;
    if (r < rows) {
      const unsigned char* src = smem + G::pix0 + r * G::kPixPitch + 16 * q;
      // (the last item has no pixels past its own and repeats them)
      const unsigned char* src2 = src + (q < kCols - 1 ? 16 : 0);
      unsigned w[8], P[8], O[7];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u32x2 t = *reinterpret_cast<const u32x2*>(k < 2 ? src + 8 * k : src2 + 8 * (k - 2));
        w[2 * k] = t.x;
        w[2 * k + 1] = t.y;
      }
      u32x2* odd = reinterpret_cast<u32x2*>(smem + G::pix1 + r * G::kPixPitch + 16 * q);
      odd[0] = u32x2{join(w[0], w[1]), join(w[1], w[2])};
      odd[1] = u32x2{join(w[2], w[3]), join(w[3], w[4])};
#pragma unroll
      for (int k = 0; k < 8; ++k)
        P[k] = __builtin_bit_cast(
            unsigned, __builtin_convertvector(f32x2{fmaf(static_cast<float>(w[k] & 0xFFFFu), 0.5f, shift),
                                                    fmaf(static_cast<float>(w[k] >> 16), 0.5f, shift)},
                                              f16x2));
#pragma unroll
      for (int k = 0; k < 7; ++k) O[k] = join(P[k], P[k + 1]);
      unsigned char* dst = smem + G::f16 + r * G::kF16Pitch + 16 * q;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1 && q == kCols - 1) break;  // the f16 planes end in half an item
        const int e = 2 * h;
        *reinterpret_cast<u32x2*>(dst + 8 * h) = u32x2{P[e], P[e + 1]};
        *reinterpret_cast<u32x2*>(dst + 8 * h + G::kF16Copy) = u32x2{O[e], O[e + 1]};
        *reinterpret_cast<u32x2*>(dst + 8 * h + 2 * G::kF16Copy) = u32x2{P[e + 1], P[e + 2]};
        *reinterpret_cast<u32x2*>(dst + 8 * h + 3 * G::kF16Copy) = u32x2{O[e + 1], O[e + 2]};
      }
      if (q < kCols - 1) {
        float e[7], o[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) {
          e[k] = square2(P[k]);
          o[k] = square2(O[k]);
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          e[k] += e[k + 1];
          o[k] += o[k + 1];
        }
        f32x4* sums = reinterpret_cast<f32x4*>(smem + G::sums + r * G::kSumPitch + 32 * q);
        sums[0] = f32x4{e[0] + e[2], o[0] + o[2], e[1] + e[3], o[1] + o[3]};
        sums[1] = f32x4{e[2] + e[4], o[2] + o[4], e[3] + e[5], o[3] + o[5]};
      }
    }
  }
  __syncthreads();
  // accumulator starts N / 2 + position term, eight rows of a column per item
  {
    constexpr int kSegs = Q, kCand = G::kCandCols;
    static_assert(kSegs * kCand <= kThreads, "one item per thread");
    const int col = tid % kCand, seg = tid / kCand;
    const bool active = seg < kSegs && 8 * seg < 4 * nb && col < 4 * nb;
    float a[15];
    if (active) {
      const float* h = reinterpret_cast<const float*>(smem + G::sums) + 8 * seg * kCand + col;
#pragma unroll
      for (int k = 0; k < 15; ++k) a[k] = h[k * kCand];  // (rows past the region only reach unused outputs)
#pragma unroll
      for (int k = 0; k < 14; ++k) a[k] += a[k + 1];
#pragma unroll
      for (int k = 0; k < 12; ++k) a[k] += a[k + 2];
    }
    __syncthreads();
    if (active) {
      float* c = reinterpret_cast<float*>(smem + G::init + 8 * seg * G::kInitPitch) + col;
      const float row = kTieStep * static_cast<float>(S);
      float at = kTieStep * static_cast<float>(8 * seg * S + col);  // (exact: whole multiples below 2^11)
#pragma unroll
      for (int k = 0; k < 8; ++k, at += row) c[k * (G::kInitPitch / 4)] = fmaf(a[k] + a[k + 4], 0.5f, at);
    }
  }
  __syncthreads();

  // half distances: operand lane (g, m) holds row 4 h + g of candidate m
  // (block row m / 4, column m % 4) or, negated, of reference m, so product h
  // covers block rows 4 h .. 4 h + 3; result lane (g, n) holds candidates (row
  // g, columns 0..3) against reference n
  constexpr int kSteps = G::kSteps;
  const int wy = wave >> 2, wx = wave & 3;
  auto half_norm = [&](int ref) {
    return reinterpret_cast<const float*>(smem + G::init)[(R + 3 * (ref >> 2)) * (G::kInitPitch / 4) + R + 3 * (ref & 3)];
  };
  unsigned half[kSteps][2];  // bf16 pairs, truncated: columns 0, 1 and 2, 3
  {
    // the lanes whose window holds row g of block row q / column i of block column k
    unsigned long long row_in[Q], col_in[C][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      row_in[q] = __builtin_amdgcn_ballot_w64(static_cast<unsigned>(8 * q + 4 * wy + g - 3 * u) <= static_cast<unsigned>(2 * R));
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        col_in[k][i] =
            __builtin_amdgcn_ballot_w64(static_cast<unsigned>(16 * k + 4 * wx + i - 3 * v) <= static_cast<unsigned>(2 * R));
    const int rc = R + 3 * v;
    const lds_byte* rp = (const lds_byte*)(smem + G::f16 + (rc & 3) * G::kF16Copy + (R + 3 * u + g) * G::kF16Pitch + (rc >> 2) * 8);
    const f16x8 b0 = -read_row(rp), b1 = -read_row(rp + 4 * G::kF16Pitch);
    const float hn = half_norm(n);
    // (one address register per row of blocks: the reads of a row reach their
    // columns by instruction offsets)
    const lds_byte* ap[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      ap[q] = (const lds_byte*)(smem + G::f16 + v * G::kF16Copy + (8 * q + 4 * wy + u + g) * G::kF16Pitch + 8 * wx);
      asm("" : "+v"(ap[q]));
    }
    const lds_byte* cp = (const lds_byte*)(smem + G::init + (4 * wy + u) * G::kInitPitch + 16 * wx + 4 * v);
    constexpr float kInf = __builtin_huge_valf();
    float best[4] = {kInf, kInf, kInf, kInf};
    // the accumulator starts, N(a~) / 2 + N(b~) / 2, as a float product of
    // depth 4: lanes g = 0 hold N(a~) / 2 of candidate m and one, lanes g = 1
    // one and N(b~) / 2 of reference n (reading the start of every result
    // would take four times the LDS cycles, and an addition per result)
    const float start_b = g == 0 ? 1.0f : g == 1 ? hn : 0.0f, start_a = g == 1 ? 1.0f : 0.0f;
    const unsigned long long first_row = __builtin_amdgcn_ballot_w64(g == 0);
    struct Operands {
      f16x8 a0, a1;
      float norm;
    };
    auto load = [&](int s) {
      const int q = s / C, k = s % C;
      return Operands{read_row(ap[q] + 32 * k), read_row(ap[q] + 32 * k + 4 * G::kF16Pitch),
                      *(const lds_float*)(cp + 8 * q * G::kInitPitch + 64 * k)};
    };
    // the next block's operands are read while this one's products run (and
    // no further ahead: the registers are the occupancy)
    Operands o = load(0);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int q = s / C, k = s % C;
      const float start = __builtin_amdgcn_inverse_ballot_w64(first_row) ? o.norm : start_a;
      f32x4 c = __builtin_amdgcn_mfma_f32_16x16x4f32(start, start_b, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_f16(o.a0, b0, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_f16(o.a1, b1, c, 0, 0, 0);
      if (s + 1 < kSteps) o = load(s + 1);
      const bool rows_in = WIDE && (q == 2 || q == 3), cols_in = WIDE && k == 1;
      float d[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned long long in = rows_in ? col_in[k][i] : cols_in ? row_in[q] : row_in[q] & col_in[k][i];
        d[i] = c[i];
        if (!(rows_in && cols_in)) d[i] = __builtin_amdgcn_inverse_ballot_w64(in) ? d[i] : kInf;
        best[i] = fminf(best[i], d[i]);
      }
      half[s][0] = __builtin_amdgcn_perm(__float_as_uint(d[1]), __float_as_uint(d[0]), 0x07060302u);
      half[s][1] = __builtin_amdgcn_perm(__float_as_uint(d[3]), __float_as_uint(d[2]), 0x07060302u);
      asm volatile("" : "+v"(half[s][0]), "+v"(half[s][1]));  // packed here, not at the use
      __builtin_amdgcn_sched_barrier(0);
    }
    // the group bests (not below zero, so that their bit patterns are ordered)
#pragma unroll
    for (int i = 0; i < 4; ++i) best[i] = fmaxf(best[i], 0.0f);
    *reinterpret_cast<u32x2*>(smem + G::best + n * G::kBestPitch + (wave * 4 + g) * 8) =
        u32x2{__builtin_amdgcn_perm(__float_as_uint(best[1]), __float_as_uint(best[0]), 0x07060302u),
              __builtin_amdgcn_perm(__float_as_uint(best[3]), __float_as_uint(best[2]), 0x07060302u)};
  }
  __syncthreads();
  // the K-th smallest of a reference's 128 bests: two references per wave,
  // their bests two to a lane, bit by bit from the top (the largest prefix
  // with fewer than K bests below it)
  constexpr unsigned kInfBits = 0x7F80u;
  {
    const unsigned* bp = reinterpret_cast<const unsigned*>(smem + G::best + 2 * wave * G::kBestPitch) + lane;
    const unsigned w0 = bp[0], w1 = bp[G::kBestPitch / 4];
    const unsigned x[2][2] = {{w0 & 0xFFFFu, w0 >> 16}, {w1 & 0xFFFFu, w1 >> 16}};
    unsigned kth[2] = {0, 0};
#pragma unroll
    for (int bit = 14; bit >= 0; --bit)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const unsigned t = kth[j] | 1u << bit;
        const int below = __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[j][0] < t)) +
                          __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[j][1] < t));
        kth[j] = below < K ? t : kth[j];
      }
    if (lane < 2) {
      const int ref = 2 * wave + lane;
      const unsigned k = lane ? kth[1] : kth[0];
      auto root = [](float x) { return __builtin_amdgcn_sqrtf(x); };
      unsigned b = kInfBits - 1;  // fewer than K groups have a candidate: all pass
      if (k < kInfBits) b = min(b, __float_as_uint(widened_bound(__uint_as_float(k << 16 | 0xFFFFu), half_norm(ref), root)) >> 16);
      reinterpret_cast<unsigned*>(smem + G::bound)[ref] = b << 16 | b;
    }
  }
  __syncthreads();
  // candidates past the bound: one bit per half distance, and each lane's
  // place among its reference's candidates
  int* count = reinterpret_cast<int*>(smem + G::count);
  int* start = reinterpret_cast<int*>(smem + G::start);
  constexpr int kPer = kSteps % 6 == 0 ? 6 : kSteps % 4 == 0 ? 4 : kSteps;  // blocks per mask word
  constexpr int kWords = kSteps / kPer, kLow = 16 - 2 * kPer;
  static_assert(kSteps % kPer == 0 && kWords <= 3, "whole mask words");
  unsigned pass[kWords];
  int n_pass, place;
  auto mark = [&] {
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    const s16x2 bound = __builtin_bit_cast(s16x2, reinterpret_cast<const unsigned*>(smem + G::bound)[n]);
    n_pass = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
      unsigned m = 0;
      // (the signs of bound - half, shifted into both halves from the top)
#pragma unroll
      for (int t = 0; t < 2 * kPer; ++t) {
        const s16x2 d = __builtin_elementwise_sub_sat(bound, __builtin_bit_cast(s16x2, half[w * kPer + t / 2][t & 1]));
        m = m >> 1 | (__builtin_bit_cast(unsigned, d) & 0x80008000u);
      }
      pass[w] = ~m & (((1u << 2 * kPer) - 1) << kLow) * 0x10001u;
      n_pass += __builtin_popcount(pass[w]);
    }
    place = n_pass ? atomicAdd(count + n, n_pass) : 0;
  };
  // lane (g, n): the lengths of the references' lists up to n, each padded to a
  // multiple of eight and those before `first` left out (along the 16 lanes of a row)
  auto lengths_up_to = [&](int c8) {
    int upto = c8;
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xF, 0xF, true);  // row_shr:1
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xF, 0xF, true);  // row_shr:2
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xF, 0xF, true);  // row_shr:4
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xF, 0xF, true);  // row_shr:8
    return upto;
  };
  auto hard = [&] {
    const int c = count[n];
    // (four lanes hold each length)
    return __builtin_popcountll(__builtin_amdgcn_ballot_w64(c > kLongList)) > 4 * 2 ||
           __builtin_amdgcn_readlane(lengths_up_to((c + 7) & ~7), 15) > hard_tile(K);
  };
  mark();
  __syncthreads();
  const bool exact = hard();
  if (exact) {
    // The exact pass.  Norms: sum over 8 x 8 pixels of (z - 32896)^2, times 2048,
    // plus the position row * S + column; rows of eight sums per thread first.
    double* norms = reinterpret_cast<double*>(smem + G::norms);
    constexpr int kCand = G::kCandCols, kPitch = G::kNormPitch;
    {
      constexpr int kCols = kCand / 8;
      static_assert(G::kRows * kCols <= kThreads, "one item per thread");
      const int r = tid / kCols, q = tid - r * kCols;
      if (r < G::kRows) {
        const u32x2* src = reinterpret_cast<const u32x2*>(smem + G::pix0 + r * G::kPixPitch + 16 * q);
        double e[16];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const u32x2 w = src[k];
          const unsigned z[4] = {w.x & 0xFFFFu, w.x >> 16, w.y & 0xFFFFu, w.y >> 16};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const double d = static_cast<double>(static_cast<int>(z[j]) - kMid);
            e[4 * k + j] = d * d;
          }
        }
#pragma unroll
        for (int k = 0; k < 15; ++k) e[k] += e[k + 1];
#pragma unroll
        for (int k = 0; k < 13; ++k) e[k] += e[k + 2];
        double* h = norms + r * kCand + 8 * q;
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = e[k] + e[k + 4];
      }
    }
    __syncthreads();
    {
      const int col = tid % kCand, seg = tid / kCand;
      const bool active = seg < Q;
      double a[15];
      if (active) {
        const double* h = norms + 8 * seg * kCand + col;
#pragma unroll
        for (int k = 0; k < 15; ++k) a[k] = h[k * kCand];
#pragma unroll
        for (int k = 0; k < 14; ++k) a[k] += a[k + 1];
#pragma unroll
        for (int k = 0; k < 12; ++k) a[k] += a[k + 2];
      }
      flip_digits<G>(smem, tid);
      __syncthreads();
      if (active) {
        double* c = norms + 8 * seg * kPitch + col;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          c[k * kPitch] = fma(a[k] + a[k + 4], 2048.0, static_cast<double>((8 * seg + k) * S + col));
      }
    }
    __syncthreads();
    // key = norms - 4096 <a, b>, with signed byte digits <a, b> = 65536 hh +
    // 256 (hl + lh) + ll.  Here a block is 16 columns of a row, 8 Q x C of them,
    // of which wave w takes rows 8 q + (w - q - 3 k) mod 8: positions that a
    // period of 2 to 16 pixels apart are alike fall into different groups too
    // (of 4 x 4 blocks, a texture of period 8 has all its repeats in two groups).
    // Operand lane (g, m) holds rows 2 g and 2 g + 1 of candidate (column) or
    // reference m, result lane (g, n) candidates 4 g .. 4 g + 3 against
    // reference n.
    typedef const __attribute__((address_space(3))) f64x2* lds_pairs;
    const lds_byte* px = (const lds_byte*)(smem + (n & 1 ? G::pix1 : G::pix0) + 2 * g * G::kPixPitch + 2 * (n & ~1));
    const lds_byte* np = (const lds_byte*)(norms + 4 * g);
    const int rc = R + 3 * v;
    const Digits ref =
        digits_of(read_rows<G>((const lds_byte*)smem + (rc & 1 ? G::pix1 : G::pix0) + (R + 3 * u + 2 * g) * G::kPixPitch + 2 * (rc & ~1)));
    const double ref_norm = norms[(R + 3 * u) * kPitch + rc] - static_cast<double>((R + 6 * u) * S + R + 6 * v);
    // use(key, in): keys less ref_norm and the lanes whose window holds them, from
    // the last block to the first; end() after each mask word's blocks
    auto exact_keys = [&](auto&& use, auto&& end) {
      const int row = -3 * u, col = 4 * g - 3 * v;
      unsigned long long col_in[C][4];
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          col_in[k][i] = __builtin_amdgcn_ballot_w64(static_cast<unsigned>(col + 16 * k + i) <= static_cast<unsigned>(2 * R));
      static_assert(kPer % C == 0, "whole rows of blocks per mask word");
      constexpr int kQ = kPer / C;
      auto rows = [&](int q, int k) { return read_rows<G>(px + exact_row(wave, q, k) * G::kPixPitch + 32 * k); };
      // (the next block's rows are read while this one's products run, where the
      // registers are not the occupancy)
      constexpr bool kAhead = kSteps > 8;
      Rows next = rows(Q - 1, C - 1);
#pragma unroll 1
      for (int w = kWords - 1; w >= 0; --w) {
#pragma unroll
        for (int t = kPer - 1; t >= 0; --t) {
          const int q = w * kQ + t / C, k = t % C, r = exact_row(wave, q, k);
          if (!kAhead) next = rows(q, k);
          const Digits a = digits_of(next);
          if (kAhead) next = t > 0 ? rows(w * kQ + (t - 1) / C, (t - 1) % C) : rows(max(w * kQ - 1, 0), C - 1);
          const unsigned long long row_in = __builtin_amdgcn_ballot_w64(static_cast<unsigned>(row + r) <= static_cast<unsigned>(2 * R));
          i32x4 x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, ref.h, i32x4{0, 0, 0, 0}, 0, 0, 0);
          const i32x4 ll = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, ref.l, i32x4{0, 0, 0, 0}, 0, 0, 0);
          x <<= 8;
          x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, ref.l, x, 0, 0, 0);
          x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, ref.h, x, 0, 0, 0);
          const lds_pairs nr = (lds_pairs)(np + 8 * (r * kPitch + 16 * k));
          const f64x2 nk[2] = {nr[0], nr[1]};
          double key[4];
          unsigned long long in[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            key[i] = fma(static_cast<double>(ll[i]), -4096.0, nk[i / 2][i % 2]);
            key[i] = fma(static_cast<double>(x[i]), -1048576.0, key[i]);
            in[i] = row_in & col_in[k][i];
          }
          use(key, in);
          __builtin_amdgcn_sched_barrier(0);
        }
        end();
      }
    };
    double best[4] = {kOutside, kOutside, kOutside, kOutside};
    exact_keys([&](const double (&key)[4], const unsigned long long (&in)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // (the high word alone decides that a key is outside)
        const unsigned long long bits = __builtin_bit_cast(unsigned long long, key[i]);
        const unsigned hi = __builtin_amdgcn_inverse_ballot_w64(in[i]) ? static_cast<unsigned>(bits >> 32) : kOutsideHigh;
        best[i] = fmin(best[i], __builtin_bit_cast(double, static_cast<unsigned long long>(hi) << 32 | static_cast<unsigned>(bits)));
      }
    }, [] {});
    {
      f64x2* to = reinterpret_cast<f64x2*>(smem + G::exact + n * G::kExactPitch + (wave * 4 + g) * 32);
      to[0] = f64x2{best[0], best[1]} + ref_norm;
      to[1] = f64x2{best[2], best[3]} + ref_norm;
    }
    __syncthreads();
    // The K-th smallest of the 128 group bests: two references per wave, their
    // bests (not below zero) two to a lane as integers, bit by bit from the top
    // (fewer than K groups with a candidate: the limit comes out above kOutside)
    if (tid < 16) count[tid] = 0;
    {
      const unsigned long long* bp = reinterpret_cast<const unsigned long long*>(smem + G::exact + 2 * wave * G::kExactPitch) + lane;
      unsigned hi[2][2], lo[2][2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const unsigned long long x = bp[j * (G::kExactPitch / 8) + e * kWave];
          hi[j][e] = static_cast<unsigned>(x >> 32);
          lo[j][e] = static_cast<unsigned>(x);
        }
      unsigned kth[2] = {0, 0}, kth_lo[2] = {0, 0};
      auto below = [](const unsigned (&x)[2], unsigned t) {
        return __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[0] < t)) + __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[1] < t));
      };
#pragma unroll 1
      for (unsigned bit = 1u << 30; bit != 0; bit >>= 1)
#pragma unroll
        for (int j = 0; j < 2; ++j) kth[j] = below(hi[j], kth[j] | bit) < K ? kth[j] | bit : kth[j];
      // the low word where several bests have this high word (near and exact ties);
      // the last four bits of an integer below 2^49 are zero
      int left[2];
      bool ties = false;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        left[j] = K - below(hi[j], kth[j]);
        ties |= below(hi[j], kth[j] + 1) - below(hi[j], kth[j]) > 1;
#pragma unroll
        for (int e = 0; e < 2; ++e) lo[j][e] = hi[j][e] == kth[j] ? lo[j][e] : ~0u;
      }
      if (ties) {
#pragma unroll 1
        for (unsigned bit = 1u << 31; bit != 8u; bit >>= 1)
#pragma unroll
          for (int j = 0; j < 2; ++j) kth_lo[j] = below(lo[j], kth_lo[j] | bit) < left[j] ? kth_lo[j] | bit : kth_lo[j];
      } else {
        kth_lo[0] = kth_lo[1] = ~0u;
      }
      if (lane < 2)
        reinterpret_cast<unsigned long long*>(smem + G::limit)[2 * wave + lane] =
            static_cast<unsigned long long>(lane ? kth[1] : kth[0]) << 32 | (lane ? kth_lo[1] : kth_lo[0]);
    }
    __syncthreads();
    const double limit = reinterpret_cast<const double*>(smem + G::limit)[n] - ref_norm;
    unsigned even = 0, odd = 0;  // columns 0, 2 and 1, 3 of a word's blocks: a bit each, the first block's last
    n_pass = 0;
    exact_keys([&](const double (&key)[4], const unsigned long long (&in)[4]) {
#pragma unroll
      for (int i = 3; i >= 0; --i)
        shift_in(i & 1 ? odd : even, __builtin_amdgcn_ballot_w64(key[i] <= limit) & in[i]);
    }, [&] {
#pragma unroll
      for (int w = kWords - 1; w > 0; --w) pass[w] = pass[w - 1];
      pass[0] = (even | odd << 16) << kLow;
      n_pass += __builtin_popcount(pass[0]);
      even = odd = 0;
    });
    place = n_pass ? atomicAdd(count + n, n_pass) : 0;
    __syncthreads();
    flip_digits<G>(smem, tid);
  }

  // exact keys and slots, as many references at a time as the queue holds
  // (nearly always all 16): their candidates' codes (reference << 12 |
  // row << 6 | column) end to end, each list padded to a multiple of eight
  uint16_t* codes = reinterpret_cast<uint16_t*>(smem + G::codes);
  double* keys = reinterpret_cast<double*>(smem + G::keys);
  constexpr unsigned kPad = 0xFFFFu;
  for (int first = 0; first < 16;) {
    const int c = count[n], c8 = n >= first ? (c + 7) & ~7 : 0;
    const int upto = lengths_up_to(c8);
    const int my_start = upto - c8;
    const unsigned full = static_cast<unsigned>(__builtin_amdgcn_ballot_w64(upto > G::kQueue)) & 0xFFFFu;
    const int last = full ? __builtin_ctz(full) : 16;  // > first: a list always fits an empty queue
    const int total = __builtin_amdgcn_readlane(upto, last - 1);
    const bool here = n >= first && n < last;
    const bool long_lists = wave_any(here && c > kPrune);
    if (wave == 0 && here) {
      if (g == 0) start[n] = my_start;
      for (int e = (c & ~7) + g; e < c8; e += 4)
        if (e >= c) codes[my_start + e] = kPad;
    }
    if (n_pass && here) {
      int at = my_start + place;
      auto list = [&](auto&& position) {  // position(q, k): row << 6 | column of the lane's first candidate
#pragma unroll
        for (int w = 0; w < kWords; ++w)
          for (unsigned m = pass[w]; m != 0; m &= m - 1) {
            const int bit = __builtin_ctz(m), t = (bit & 15) - kLow, s = w * kPer + (t >> 1), q = s / C, k = s - q * C;
            codes[at++] = static_cast<uint16_t>((n << 12) + position(q, k) + 2 * (t & 1) + (bit >> 4));
          }
      };
      if (exact) {
        list([&](int q, int k) { return exact_row(wave, q, k) << 6 | (16 * k + 4 * g); });
      } else {
        const int mine = (4 * wy + g) << 6 | 4 * wx;
        list([&](int q, int k) { return mine + 512 * q + 16 * k; });
      }
    }
    __syncthreads();
    for (int f = tid; f < total; f += kThreads) {
      const unsigned code = codes[f], k = code >> 12, cy = code >> 6 & 63, cx = code & 63;
      const int dy = static_cast<int>(cy) - 3 * static_cast<int>(k >> 2), dx = static_cast<int>(cx) - 3 * static_cast<int>(k & 3);
      // (the reference itself takes no slot among the others)
      double key = __builtin_huge_val();
      if (code != kPad && (dy != R || dx != R))
        key = exact_key<G>(smem, R + 3 * (k >> 2), R + 3 * (k & 3), cy, cx, dy * S + dx);
      keys[f] = key;
    }
    __syncthreads();
    if (long_lists) {
      // a long list, a wave each: the (K-1)-th smallest high word of its first
      // kSample keys (positive, so ordered as integers), rounded up to eight bits
      // of mantissa, is a bound, and the keys up to it move to the list's front.
      // (Ranking longer lists whole, or cutting them by all threads from 128
      // ranked keys, made the tiles with such lists the launch's tail: K = 32 on
      // 640 x 360 56.6 -> 52.5 us, the two-stage 512^2 image 264 -> 256 us; a
      // sample of 512 and all 31 bits cost the smaller images 2 %, cutting from
      // 48 keys on instead of 64 up to 2 %.)
      constexpr int kBoundBit = 12;
      for (int k = first + wave; k < last; k += kWaves) {
        const int n_list = __builtin_amdgcn_readfirstlane(count[k]);
        if (n_list <= kPrune) continue;
        double* list = keys + __builtin_amdgcn_readfirstlane(start[k]);
        auto bound_of = [&](auto blocks) {
          constexpr int kBlocks = decltype(blocks)::value;
          unsigned x[kBlocks], kth = 0;
#pragma unroll
          for (int i = 0; i < kBlocks; ++i) {
            const int e = lane + kWave * i;
            x[i] = e < n_list ? high_word(list[e]) : ~0u;
          }
#pragma unroll 1
          for (int bit = 30; bit >= kBoundBit; --bit) {
            const unsigned t = kth | 1u << bit;
            int below = 0;
#pragma unroll
            for (int i = 0; i < kBlocks; ++i) below += __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[i] < t));
            kth = below < K - 1 ? t : kth;
          }
          return kth | ((1u << kBoundBit) - 1);
        };
        const unsigned kth = n_list <= 2 * kWave ? bound_of(std::integral_constant<int, 2>{})
                                                 : bound_of(std::integral_constant<int, kSample / kWave>{});
        int n_kept = 0;
        for (int e0 = 0; e0 < n_list; e0 += kWave) {
          // (a block's keys are read before any is written at or before its place)
          const double key = e0 + lane < n_list ? list[e0 + lane] : __builtin_huge_val();
          const bool keep = key < __builtin_huge_val() && high_word(key) <= kth;
          const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
          wave_lds_sync();
          if (keep)
            list[n_kept + __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(m), 0))] = key;
          n_kept += __builtin_popcountll(m);
          wave_lds_sync();
        }
        for (int e = n_kept + lane; e < ((n_list + 7) & ~7); e += kWave) list[e] = __builtin_huge_val();
        if (lane == 0) reinterpret_cast<int*>(smem + G::kept)[k] = n_kept;
      }
      __syncthreads();
    }
    // a key's slot is the number of smaller keys of its reference
    for (int f = tid; f < total; f += kThreads) {
      const double key = keys[f];
      const int k = codes[f] >> 12, p = p0 + (k >> 2), q = q0 + (k & 3);
      if (key == __builtin_huge_val()) continue;
      const int n_keys = count[k] > kPrune ? reinterpret_cast<const int*>(smem + G::kept)[k] : count[k];
      const int rank = entries_below(keys + start[k], n_keys, key);
      if (rank < K - 1 && p < nRy && q < nRx)
        idx[(static_cast<size_t>(p) * nRx + q) * K + 1 + rank] =
            static_cast<int16_t>(key - 2048.0 * floor(key * (1.0 / 2048.0)));
    }
    first = last;
    if (first < 16) __syncthreads();  // the queue is reused
  }
  if (tid < 16 && p0 + (tid >> 2) < nRy && q0 + (tid & 3) < nRx)
    idx[(static_cast<size_t>(p0 + (tid >> 2)) * nRx + q0 + (tid & 3)) * K] = static_cast<int16_t>(R * S + R);
}

// Stack work beside the matching (every thread's pixel loads first at every size,
// unlike a stack launch of its own: one by one the two-stage call takes 260
// instead of 257 us at 512^2, 13.27 instead of 13.17 ms at 4096^2): `pairs`
// workgroups of two stack items each,
// spread evenly over the launch.  Workgroups come in groups of eight (one per
// XCD); group g holds stack items where floor(g * share / 2^32) steps,
// share / 2^32 just above their part of all groups.
struct StackShare {
  int pairs = 0, per_plane = 0;  // workgroups of stack items; of one of its planes
  unsigned share = 0;
};

// waves per SIMD: 80 registers for the largest grid and for the stacks' workgroups
// (three workgroups per CU), 64 otherwise (four)
constexpr int min_waves(int steps, int kind) { return kind < 0 && steps <= 8 ? 8 : 6; }

template <int Q, int C, bool WIDE, bool BATCH, int KIND>
__global__ __launch_bounds__(kThreads, min_waves(Q * C, KIND)) void bm_corr_kernel(ImgRec one, WorkList wl,
                                                                                   WorkList stack_wl, StackShare ss,
                                                                                   int R, int K, int use_pilot) {
  using Lds = StackLds<4>;
  __shared__ __align__(16) unsigned char smem[KIND < 0 ? Geo<Q, C>::bytes : max2(Geo<Q, C>::bytes, 2 * sizeof(Lds))];
  unsigned b = blockIdx.z * gridDim.x + blockIdx.x;
  if constexpr (KIND >= 0) {
    const unsigned g = b >> 3, sg = __umulhi(g, ss.share);
    if (__umulhi(g + 1, ss.share) != sg) {
      const int s = static_cast<int>(sg * 8 + (b & 7));
      if (s >= ss.pairs) return;
      const int plane = s >= ss.per_plane ? 1 : 0;
      const int half = wave_id() / kStackRows;
      Lds& lds = reinterpret_cast<Lds*>(smem)[half];
      const int t = static_cast<int>(threadIdx.x) & (kStackThreads - 1);
      int item = 2 * (s - plane * ss.per_plane) + half;
      if constexpr (!BATCH) {
        if (item >= stack_items(one.H, one.W)) item = -1;
        stack_body<KIND, 4, true>(lds, t, plane ? one.pilot : one.noisy, plane ? one.stack_b : one.stack_a,
                                  plane ? nullptr : one.partials, plane == 0, one.H, one.W, item);
      } else {
        int first = item + 1;
        const bool any = item < stack_wl.total;
        const const_rec_ptr r = find_item(stack_wl, any ? item : 0, first);
        stack_body<KIND, 4, true>(lds, t, plane ? r->pilot : r->noisy, plane ? r->stack_b : r->stack_a,
                                  plane ? nullptr : r->partials, plane == 0, r->H, r->W,
                                  any ? item - first : -1);
      }
      return;
    }
    b -= sg * 8;
  }
  if constexpr (!BATCH) {
    // Workgroups go to the eight XCDs in turn (g -> XCD g mod 8): XCD x takes
    // the x-th eighth of the items, a band of reference rows, so each XCD's
    // L2 fetches its band's pixels instead of the whole image.  The grid is
    // 8 q; items past the last exit at once.
    const int n = corr_items(one.H, one.W), q = (n + 7) / 8;
    const int item = static_cast<int>((b & 7) * q + (b >> 3));
    if (static_cast<int>(b >> 3) >= q || item >= n) return;
    corr_body<Q, C, WIDE>(smem, use_pilot ? one.pilot : one.noisy, one.idx, one.H, one.W, R, K, item);
  } else {
    if (b >= static_cast<unsigned>(wl.total)) return;
    int first;
    const int item = static_cast<int>(b);
    const const_rec_ptr r = find_item(wl, item, first);
    corr_body<Q, C, WIDE>(smem, use_pilot ? r->pilot : r->noisy, r->idx, r->H, r->W, R, K, item - first);
  }
}

// kind < 0: matching only; else the stacks of stack_wl (or of the image) beside it
template <int Q, int C, bool WIDE, int KIND>
hipError_t launch_corr_kind(const ImgRec& one, const WorkList* wl, const WorkList* stack_wl, int R, int K,
                            int use_pilot, hipStream_t st) {
  const int n = wl ? wl->total : corr_items(one.H, one.W);
  if (n <= 0) return hipSuccess;
  const int match_groups = (n + 7) / 8;
  int groups = match_groups;
  StackShare ss;
  if constexpr (KIND >= 0) {
    const int planes = KIND == 0 ? 1 : 2;
    ss.per_plane = ((wl ? stack_wl->total : stack_items(one.H, one.W)) + 1) / 2;
    ss.pairs = planes * ss.per_plane;
    const int stack_groups = (ss.pairs + 7) / 8;
    groups += stack_groups;
    ss.share = static_cast<unsigned>(((static_cast<unsigned long long>(stack_groups) << 32) + groups - 1) / groups);
  }
  const dim3 grid = batch_grid(8 * groups);
  if (wl)
    hipLaunchKernelGGL((bm_corr_kernel<Q, C, WIDE, true, KIND>), grid, dim3(kThreads), 0, st, one, *wl,
                       stack_wl ? *stack_wl : WorkList{}, ss, R, K, use_pilot);
  else
    hipLaunchKernelGGL((bm_corr_kernel<Q, C, WIDE, false, KIND>), grid, dim3(kThreads), 0, st, one, WorkList{},
                       WorkList{}, ss, R, K, use_pilot);
  return hipGetLastError();
}

template <int Q, int C, bool WIDE>
hipError_t launch_corr_grid(const ImgRec& one, const WorkList* wl, const WorkList* stack_wl, int R, int K,
                            int use_pilot, int stack_kind, hipStream_t st) {
  if (stack_kind < 0) return launch_corr_kind<Q, C, WIDE, -1>(one, wl, stack_wl, R, K, use_pilot, st);
  return stack_kind == 0 ? launch_corr_kind<Q, C, WIDE, 0>(one, wl, stack_wl, R, K, use_pilot, st)
                         : launch_corr_kind<Q, C, WIDE, 2>(one, wl, stack_wl, R, K, use_pilot, st);
}

}  // namespace

int corr_items_for(int H, int W) { return corr_items(H, W); }

long corr_tiles(int H, int W) { return static_cast<long>(corr_items(H, W)); }

hipError_t launch_bm_corr(const ImgRec& one, const WorkList* wl, const WorkList* stack_wl, int R, int K, int use_pilot,
                          int stack_kind, hipStream_t st) {
  if (K < 2 || K > 32 || R < 0 || R > kMaxR || stack_kind == 1 ||
      (wl && stack_kind >= 0 && !stack_wl)) return hipErrorInvalidValue;
  const int nb = blocks_per_axis(R);
  if (nb <= 4) return launch_corr_grid<2, 1, false>(one, wl, stack_wl, R, K, use_pilot, stack_kind, st);
  if (nb <= 6) return launch_corr_grid<3, 2, false>(one, wl, stack_wl, R, K, use_pilot, stack_kind, st);
  if (nb <= 8) return launch_corr_grid<4, 2, false>(one, wl, stack_wl, R, K, use_pilot, stack_kind, st);
  if (nb < kMaxNb) return launch_corr_grid<6, 3, false>(one, wl, stack_wl, R, K, use_pilot, stack_kind, st);
  return launch_corr_grid<6, 3, true>(one, wl, stack_wl, R, K, use_pilot, stack_kind, st);
}

}  // namespace gbm3d
