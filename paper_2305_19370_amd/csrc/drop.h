// The residual-branch dropout masks, regenerated wherever they are needed.
#pragma once

#include "common.h"
#include "internal.h"

namespace bpt {

BPT_DEV u32x4 philox4x32_10(u32x4 c, uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
    const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
    c = u32x4{hi1 ^ c[1] ^ k0, lo1, hi0 ^ c[3] ^ k1, lo0};
  }
  return c;
}

// keep factors (0 or scale) of columns n..n+3 of token t
BPT_DEV void drop_factors(const DropArgs& a, int64_t t, int64_t n, float f[4]) {
  const u32x4 w = philox4x32_10(u32x4{(uint32_t)(n >> 2), (uint32_t)t, a.site, 0u}, a.k0, a.k1);
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = w[e] >= a.threshold ? a.scale : 0.0f;
}

}  // namespace bpt
