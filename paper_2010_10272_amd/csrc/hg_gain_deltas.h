// hg_gain_deltas.h -- gain-cache updates of one pin (subsection "Gain Caching").
#pragma once

#include "hg_device.h"
#include "hg_internal.h"

namespace hg {

// Pin v of a net of weight w: p_i(v) gets +w where block i lost its last pin of the
// net and -w where it gained its first, and b(v), if v did not move, +w where its
// block now holds exactly one pin of the net and -w where it no longer does.
// chg(x), x in [0, 4 WK): changed and old Lambda, changed and new S, WK words each.
template <int WK, typename Word>
__device__ __forceinline__ void pin_deltas(const InstDesc& D, int v, int w, Word chg) {
  int* cp = D.cache + cache_pbase(D.n) + (long long)v * cache_stride(D.k);
  unsigned any = 0;
#pragma unroll
  for (int x = 0; x < WK; ++x) {
    unsigned d = chg(x);
    const unsigned old = chg(WK + x);
    any |= chg(2 * WK + x);
    while (d) {
      const int bit = __ffs(d) - 1;
      d &= d - 1;
      atomicAdd(&cp[x * 32 + bit], ((old >> bit) & 1u) ? w : -w);
    }
  }
  if (any && !D.moved[v]) {
    const int c = D.part[v];
    if ((unsigned)c < (unsigned)D.k) {
      const int x = c >> 5, bit = c & 31;
      if ((chg(2 * WK + x) >> bit) & 1u)
        atomicAdd(&D.cache[v], ((chg(3 * WK + x) >> bit) & 1u) ? w : -w);
    }
  }
}

}  // namespace hg
