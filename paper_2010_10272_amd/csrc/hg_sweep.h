// hg_sweep.h -- what the vertex sweeps (LP select, gains) read per incident
// net, from either the full net record or the compact Lambda/S view.
#pragma once

#include "hg_bits.h"
#include "hg_device.h"
#include "hg_internal.h"

namespace hg {

// 32-bit words of a net entry: one for the views of up to 32 bits, Lambda and S
// otherwise, with w in front where nets are weighted.
constexpr __host__ __device__ int entry_words(int wk, int view) {
  return view == kView32 ? 2 : view == kView64 ? 4
         : view == kViewUnit ? 2 * wk : view == kViewFull ? 1 + 2 * wk : 1;
}

// Entry of net e.
template <int WK, int VIEW>
__device__ __forceinline__ void read_entry(const unsigned* __restrict__ netstate, int rw,
                                           const void* __restrict__ view, unsigned e,
                                           unsigned (&x)[entry_words(WK, VIEW)]) {
  if constexpr (VIEW == kView4) {
    x[0] = global_ptr((const unsigned char*)view)[e];
  } else if constexpr (VIEW == kView8) {
    x[0] = global_ptr((const unsigned short*)view)[e];
  } else if constexpr (VIEW == kView16) {
    x[0] = global_ptr((const unsigned*)view)[e];
  } else if constexpr (VIEW == kView32) {
    const u32x2 v = global_ptr((const u32x2*)view)[e];
    x[0] = v.x;
    x[1] = v.y;
  } else if constexpr (VIEW == kView64) {
    const u32x4 v = global_ptr((const u32x4*)view)[e];
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  } else {
    // record words 0 (w), 1 (lambda, not needed), 2 .. 2 + 2 WK (Lambda, S)
    constexpr int N = 2 + 2 * WK;
    unsigned r[(N + 3) / 4 * 4];
    const auto q = global_ptr(reinterpret_cast<const u32x4*>(netstate + (long long)e * rw));
#pragma unroll
    for (int i = 0; i < (N + 3) / 4; ++i) {
      const u32x4 v = q[i];
      r[4 * i] = v.x;
      r[4 * i + 1] = v.y;
      r[4 * i + 2] = v.z;
      r[4 * i + 3] = v.w;
    }
    constexpr int first = VIEW == kViewFull ? 1 : 0;
    if constexpr (VIEW == kViewFull) x[0] = r[0];
#pragma unroll
    for (int i = 0; i < 2 * WK; ++i) x[first + i] = r[2 + i];
  }
}

// Lambda(e), the S(e) word that holds block a's bit (aw = a / 32) and w(e) of an
// entry; nothing of it where `on` is 0 (all ones otherwise).
template <int WK, int VIEW>
__device__ __forceinline__ void open_entry(const unsigned (&x)[entry_words(WK, VIEW)], unsigned on,
                                           int aw, unsigned (&L)[WK], unsigned& S, unsigned& w) {
  if constexpr (VIEW == kView4 || VIEW == kView8 || VIEW == kView16) {
    constexpr int half = VIEW == kView4 ? 4 : VIEW == kView8 ? 8 : 16;
    const unsigned v = x[0] & on;
    L[0] = v & ((1u << half) - 1u);
    S = v >> half;
    w = 1;
  } else {
    constexpr int first = VIEW == kViewFull ? 1 : 0;
    w = VIEW == kViewFull ? x[0] & on : 1u;
    S = x[first + WK];
#pragma unroll
    for (int i = 0; i < WK; ++i) {
      L[i] = x[first + i] & on;
      if (i == aw) S = x[first + WK + i];
    }
    S &= on;
  }
}

// What the sweeps accumulate per vertex u in block a: conn counters, w(I(u)),
// b(u), and whether w(I(u)) left the counters' range (a heavy vertex; unit
// nets: the row's length bounds it).
template <int WK, int VIEW>
struct RowSums {
  BitCounters<WK> C;
  int tot, ben;
  bool heavy;

  __device__ __forceinline__ void clear() {
    C.clear();
    tot = ben = 0;
    heavy = false;
  }

  // The next U nets of the row; `ash` is a % 32.  False once the row is heavy.
  template <int U>
  __device__ __forceinline__ bool add(const unsigned (&L)[U][WK], const unsigned (&S)[U],
                                      const unsigned (&w)[U], int ash) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const unsigned single = (S[q] >> ash) & 1u;
      ben += VIEW == kViewFull ? (single ? (int)w[q] : 0) : (int)single;
    }
    if constexpr (VIEW == kViewFull) {
#pragma unroll
      for (int q = 0; q < U; ++q) tot += (int)w[q];
      if (tot > kLightLimit) {
        heavy = true;
        return false;
      }
      C.add_weighted(L, w);
    } else {
      C.add_ones(L);
    }
    return true;
  }
};

// Nets at positions [j, j + U) of the incidence row [at, at + deg), in 16-byte
// loads: a wavefront's rows lie side by side, so U single loads would each
// touch every line of them (netlist select 166 -> 150 us, matrix 69 -> 65).
// Positions past the row repeat its entry j (the caller masks them); rows
// within U entries of the array's end (P entries in all) load one by one.
template <int U>
__device__ __forceinline__ void read_row(const int* __restrict__ vnets, long long at, int deg,
                                         int j, long long P, int (&e)[U]) {
  const auto row = global_ptr(vnets + at);
  if (at + j + U <= P) {
    i32x4u v[U / 4];
#pragma unroll
    for (int h = 0; h < U / 4; ++h) v[h] = load4_unaligned(vnets + at + j + 4 * h);
#pragma unroll
    for (int q = 0; q < U; ++q) e[q] = v[q / 4][q % 4];
  } else {
#pragma unroll
    for (int q = 0; q < U; ++q) e[q] = row[j + q < deg ? j + q : j];
  }
#pragma unroll
  for (int q = 1; q < U; ++q) e[q] = j + q < deg ? e[q] : e[0];
}

// The sums of row [b0, b0 + deg) of a vertex in block a, walked by one lane: U entries in flight
// (slots past the row's end load an entry again and are masked, so that no
// load sits in a branch of its own), the next nets' ids on their way while
// these entries arrive.
template <int WK, int VIEW, int U>
__device__ __forceinline__ void walk_row(const InstDesc& D, const void* __restrict__ view,
                                         long long b0, int deg, int a, RowSums<WK, VIEW>& R) {
  R.clear();
  const int aw = a >> 5, ash = a & 31;
  int e[U];
  if (deg > 0) read_row<U>(D.vnets, b0, deg, 0, D.P, e);
  for (int j = 0; j < deg; j += U) {
    unsigned x[U][entry_words(WK, VIEW)], L[U][WK], S[U], w[U];
#pragma unroll
    for (int q = 0; q < U; ++q) read_entry<WK, VIEW>(D.netstate, D.rw, view, (unsigned)e[q], x[q]);
    const int next = j + U < deg ? j + U : j;
    read_row<U>(D.vnets, b0, deg, next, D.P, e);
#pragma unroll
    for (int q = 0; q < U; ++q)
      open_entry<WK, VIEW>(x[q], j + q < deg ? ~0u : 0u, aw, L[q], S[q], w[q]);
    if (!R.template add<U>(L, S, w, ash)) break;
  }
  if constexpr (VIEW != kViewFull) R.tot = deg;
}

}  // namespace hg
