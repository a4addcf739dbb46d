// The correlation matcher's bound on approximate half distances: its constants
// and the widening by what the roundings can do, apart from the kernel so that
// the host can check them against exact distances.
#pragma once

namespace gbm3d {

// Position term of a half distance, per unit of row * S + column (at most
// 1880): a half distance is a whole multiple of 1/8 on this scale, the term
// stays below half of that.
constexpr float kTieStep = 1.0f / 32768.0f;

// The widened bound on the approximate half distances of a reference, from
// the K-th best of its group bests, `half`, and hn = N(b~) / 2; root a square
// root that is off by less than 10^-6 of it.  With
// t = |a~ - b~| the distance that half stands for and e = 2^-11 the relative
// rounding of f16, a candidate at approximate distance <= t has true distance
// at most t + e (|a| + |b|), and a candidate truly that close has approximate
// distance at most t + e (4 |b~| + 2 t) to first order in e (|a| <= |b| + t
// for both).  The accumulation of a half distance, 64 products and the start
// value, is off by less than 2^-17 (|b~| + t)^2 (65 roundings of 2^-23 of sums
// below (|b~| + t)^2); this counts twice.
template <typename Root>
constexpr float widened_bound(float half, float hn, Root root) {
  const float nb = root(2.0f * hn) * 1.000002f, t = root(2.0f * half) * 1.000002f;
  const float t2 = t + (1.01f / 2048.0f) * (4.0f * nb + 2.0f * t);
  return 0.500002f * t2 * t2 + 1.0f / 65536.0f * (nb + t2) * (nb + t2);
}

}  // namespace gbm3d
