// Three-way cut of a uniform at the two Metropolis thresholds with one
// multiply-add (host part: plain C++, no HIP).
//
// A site needs [u < t4] and [u < t8] (t8 < t4).  The map
//     f(u) = u X + C,  X = floor(2^60 / (t4 - t8)),
//     C = 2^60 - t8 X + rho,  rho = 2^60 - (t4 - t8) X
// is increasing, has f(t8) = 2^60 + rho and f(t4) = 2^61, and moves by X per
// step of u, so with rho < X the top four bits of f(u) are 0 exactly for
// u < t8, 1 exactly for t8 <= u < t4 and 2 or more for u >= t4, as long as f
// stays inside [0, 2^64) for every u that occurs.  All of it is integer
// arithmetic: no uniform is rounded or cut short.  f fits for
// t8 <= t4 - t8 (the codes below t8 are one) and for t4 - t8 of at least
// about (2^32 - t4) / 14 (the codes from t4 up are at most 14): with
// t4 / 2^32 = e^{-4 beta} that is 1.516 <= T <= 5.77.
//
// The per-thread LCG's uniforms go up to 2^31 only (|int32(x)| against
// thresholds of that scale, both plus one): the multiplier, which is below
// 2^32, reaches differences of 2^28, so 2.08 <= T <= 5.77.
#pragma once

#include <stdint.h>

namespace ising {

struct Cut {
  uint32_t x;  // X, or 0: this pair of thresholds has no such map
  uint32_t pad;
  uint64_t c;  // C
};

// The cut for uniforms 0 .. u_max.
inline Cut make_cut(uint32_t t4, uint32_t t8, uint32_t u_max = 0xFFFFFFFFu) {
  const Cut none = {0u, 0u, 0ull};
  if (t4 <= t8) return none;
  const uint64_t d = t4 - t8, one = 1ull << 60;
  const uint64_t X = one / d, rho = one - d * X;
  if (X > 0xFFFFFFFFull || rho >= X) return none;
  const unsigned __int128 tx = (unsigned __int128)t8 * X;
  if (tx > (unsigned __int128)one + rho) return none;
  const uint64_t C = (uint64_t)((unsigned __int128)one + rho - tx);
  if (((unsigned __int128)u_max * X + C) >> 64) return none;
  const Cut cut = {(uint32_t)X, 0u, C};
  return cut;
}

}  // namespace ising
