// The sign that a layer's split products carry (lp_split.h). Plain C++ (constexpr
// functions run on the host and on the device), so that a host program can evaluate it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace lp {

// Level l of a solve with coarsening factor c evaluates the layers n = 0, c^l, 2 c^l, ..
// and the signs have to balance on all of these progressions, for any c. Layers 2 k and
// 2 k + 1 have opposite signs, so the finest level is even after every second layer;
// which of the two is positive is the upper half of k times an odd constant modulo
// 2^32, which walks evenly round the circle in steps of any length. The constant is the
// best of 600000 tried: over the first 16384 layers the signs of every progression with
// c = 2 .. 32 and a step up to 4096 add up to at most 14 at any point. (The parity of n's
// one bits does better for powers of two, 1, but leaves 1458 of 5462 for c = 3.)
constexpr float layer_sign(size_t n) { return ((uint32_t)(n >> 1) * 0xc9e47593u >> 31 ^ (uint32_t)(n & 1)) ? -1.f : 1.f; }

}  // namespace lp
