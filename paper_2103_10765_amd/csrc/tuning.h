// The autotuner's records and the launch choices made from them, on the host
// alone.
#pragma once

#include <cstdlib>
#include <map>

#include "../../include/gbm3d.h"

namespace gbm3d {

// Tuning key: group size, search window, shape class of the image(s).
struct TuneKey {
  int K, search, cls;
  bool operator<(const TuneKey& o) const {
    return K != o.K ? K < o.K : (search != o.search ? search < o.search : cls < o.cls);
  }
};

// A block-matching launch choice.
struct TuneEntry {
  int method = GBM3D_BM_SHIFT, split = 1;
  float ms = 0.0f;
};

// A stage-1 group-kernel shape.
struct ShapeEntry {
  int shape = 0;
  float ms = 0.0f;
};

struct Tuning {
  std::map<TuneKey, TuneEntry> matching;
  std::map<TuneKey, ShapeEntry> shapes;  // keyed by k_ht
};

// Shape class of a launch: floor(log2) of its 4x4 reference tiles.
inline int tile_class(long tiles) {
  int c = 0;
  while (tiles >= (2L << c)) ++c;
  return c;
}

// The matching kernel where neither the caller nor a tuning record chooses.  The
// correlation kernel's work per tile hardly shrinks below its smallest grid of
// candidate blocks, the shift-wise kernel's does with the window's area, but it
// leaves the stacks to a launch of their own.  Matching | whole first stage at
// K = 8, correlation against shift-wise, us: 1024^2 window 5 64 | 217 against 26 |
// 174, window 7 64 | 217 against 52 | 199, window 11 81 | 234 against 82 | 225,
// window 13 81 | 235 against 130 | 279; 512^2 window 5 21 | 66 against 12 | 61,
// window 7 21 | 66 against 20 | 69; 256^2 window 5 10 | 31 against 10 | 33.
inline int default_method(int search, long tiles) {
  const bool shift = (search <= 5 && tiles > 1000) || (search <= 11 && tiles > 3000);
  return shift ? GBM3D_BM_SHIFT : GBM3D_BM_CORR;
}

struct BmChoice {
  int method, split;  // split 0: by size inside the launcher
};

// Explicit choices (method, split) win.  Zeros take the tuned choice of the
// class (same K and search); without one, the method of the nearest tuned
// class of the same K and search (split then by size), else the default.
inline BmChoice choose_bm(const Tuning& t, int method, int split, int search, long tiles, int K) {
  BmChoice c{method, split};
  const int cls = tile_class(tiles);
  const auto it = t.matching.find({K, search, cls});
  if (it != t.matching.end()) {
    if (c.method == GBM3D_BM_AUTO) c.method = it->second.method;
    if (c.split == 0 && c.method == it->second.method) c.split = it->second.split;
  } else if (c.method == GBM3D_BM_AUTO) {
    int best = 1 << 30;
    for (const auto& kv : t.matching) {
      const int d = std::abs(kv.first.cls - cls);
      if (kv.first.K == K && kv.first.search == search && d < best) {
        best = d;
        c.method = kv.second.method;
      }
    }
  }
  if (c.method == GBM3D_BM_AUTO) c.method = default_method(search, tiles);
  return c;
}

// The first class whose images all take 8 x 8 reference tiles in shape 0 (the
// group kernels' rule: more than 380 of those tiles, four times as many of
// 4 x 4).  A record of a smaller class has compared the one-tile shape with
// smaller tiles, which only single images of that size take.
constexpr int kTwoTileClass = 11;

// The stage-1 group-kernel shape: the tuned one of the class, else that of
// the nearest tuned class of the same k_ht and search, else 0 (tiles sharing a
// CU).  A record of a class below kTwoTileClass speaks for single images of its
// class alone.
inline int choose_shape(const Tuning& t, int k_ht, int search, long tiles, bool batch) {
  const int cls = tile_class(tiles);
  int best = 1 << 30, shape = 0;
  for (const auto& kv : t.shapes) {
    const int c = kv.first.cls, d = std::abs(c - cls);
    if (kv.first.K != k_ht || kv.first.search != search || d >= best) continue;
    if (c >= kTwoTileClass ? batch || cls >= kTwoTileClass : !batch && d == 0) {
      best = d;
      shape = kv.second.shape;
    }
  }
  return shape;
}

}  // namespace gbm3d
