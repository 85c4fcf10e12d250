// hg_bits.h -- bit-sliced per-block counters held in registers.
//
// For a vertex u, conn_i = w({e in I(u) : i in Lambda(e)}) is needed for every
// block i; then p_i(u) = w(I(u)) - conn_i (section "Parallel Gain
// Calculation").  When w(I(u)) <= 255 every conn_i fits in 8 bits, so the k
// counters are stored transposed: plane p holds bit p of all counters, one
// 32-bit word per 32 blocks.  Adding w(e) to every block of Lambda(e) is an
// add of the bitset into the planes (several nets' bitsets at a time), and the arg-max over a set
// of blocks is a walk from the top plane down.  Everything stays in VGPRs:
// one thread per vertex, no LDS, full occupancy for the random net gathers.
#pragma once

#include "hg_internal.h"

namespace hg {

template <int WK>
struct BitCounters {
  unsigned c[kPlanes][WK];

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int p = 0; p < kPlanes; ++p)
#pragma unroll
      for (int w = 0; w < WK; ++w) c[p][w] = 0u;
  }

  // a + b + c as sum and carry bits (one three-input logic operation each).
  static __device__ __forceinline__ void full_add(unsigned a, unsigned b, unsigned c,
                                                  unsigned& sum, unsigned& carry) {
    const unsigned x = a ^ b;
    carry = (a & b) | (c & x);
    sum = x ^ c;
  }

  // counter_i += 2^J for every i in each of the U (4 or 8) masks of word w.  The masks
  // are added among themselves first (a tree of full adders), so the counters
  // take one carry ripple per call: 18 operations a word for four masks, 24
  // for eight, where a ripple per mask takes 16 each.
  template <int J, int U>
  __device__ __forceinline__ void add_masks(int w, const unsigned (&m)[U]) {
    static_assert(U == 4 || U == 8, "masks per call");
    unsigned carry, s, k1, k2;
    if constexpr (U == 4) {
      full_add(m[0], m[1], m[2], s, k1);
      full_add(c[J][w], s, m[3], c[J][w], k2);
      if constexpr (J + 1 < kPlanes) {
        full_add(c[J + 1][w], k1, k2, c[J + 1][w], carry);
        ripple<J + 2>(w, carry);
      }
    } else {
      unsigned s2, k3, k4, l1, l2;
      full_add(m[0], m[1], m[2], s, k1);
      full_add(m[3], m[4], m[5], s2, k2);
      full_add(s, s2, m[6], s, k3);
      full_add(c[J][w], s, m[7], c[J][w], k4);
      if constexpr (J + 1 < kPlanes) {
        full_add(k1, k2, k3, s, l1);
        full_add(c[J + 1][w], s, k4, c[J + 1][w], l2);
        if constexpr (J + 2 < kPlanes) {
          full_add(c[J + 2][w], l1, l2, c[J + 2][w], carry);
          ripple<J + 3>(w, carry);
        }
      }
    }
  }

  template <int FROM>
  __device__ __forceinline__ void ripple(int w, unsigned carry) {
#pragma unroll
    for (int p = FROM; p < kPlanes; ++p) {
      const unsigned t = c[p][w] & carry;
      c[p][w] ^= carry;
      carry = t;
    }
  }

  // counter_i += 1 for every i in each mask (unit net weights).
  template <int U>
  __device__ __forceinline__ void add_ones(const unsigned (&m)[U][WK]) {
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      unsigned x[U];
#pragma unroll
      for (int q = 0; q < U; ++q) x[q] = m[q][w];
      add_masks<0, U>(w, x);
    }
  }

  // counter_i += wgt[q] for every i in mask q (weights in [0, 255]), one bit of
  // the weights at a time, up to the highest bit that a lane of the wavefront
  // has.
  template <int U>
  __device__ __forceinline__ void add_weighted(const unsigned (&m)[U][WK],
                                               const unsigned (&wgt)[U]) {
    unsigned any = 0;
#pragma unroll
    for (int q = 0; q < U; ++q) any |= wgt[q];
    weighted_bits<0, U>(m, wgt, any);
  }

  template <int J, int U>
  __device__ __forceinline__ void weighted_bits(const unsigned (&m)[U][WK],
                                                const unsigned (&wgt)[U], unsigned any) {
    if constexpr (J < kPlanes) {
      if (__any((any >> J) != 0)) {
#pragma unroll
        for (int w = 0; w < WK; ++w) {
          unsigned x[U];
#pragma unroll
          for (int q = 0; q < U; ++q)
            x[q] = m[q][w] & (unsigned)((int)(wgt[q] << (31 - J)) >> 31);
          add_masks<J, U>(w, x);
        }
        weighted_bits<J + 1, U>(m, wgt, any);
      }
    }
  }

  // Blocks with a non-zero counter.
  __device__ __forceinline__ void nonzero(unsigned (&out)[WK]) const {
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      unsigned x = 0;
#pragma unroll
      for (int p = 0; p < kPlanes; ++p) x |= c[p][w];
      out[w] = x;
    }
  }

  // Narrow `set` to the blocks whose counter is maximal within it; returns
  // that maximum.  `set` must be non-empty.
  __device__ __forceinline__ unsigned narrow_to_max(unsigned (&set)[WK]) const {
    unsigned best = 0;
#pragma unroll
    for (int p = kPlanes - 1; p >= 0; --p) {
      unsigned t[WK];
      unsigned any = 0;
#pragma unroll
      for (int w = 0; w < WK; ++w) {
        t[w] = set[w] & c[p][w];
        any |= t[w];
      }
      if (any) {
#pragma unroll
        for (int w = 0; w < WK; ++w) set[w] = t[w];
        best |= 1u << p;
      }
    }
    return best;
  }

  // Counter of block 32*w + b (w a compile-time word index).
  __device__ __forceinline__ unsigned value(int w, int b) const {
    unsigned v = 0;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) v |= ((c[p][w] >> b) & 1u) << p;
    return v;
  }
};

}  // namespace hg
