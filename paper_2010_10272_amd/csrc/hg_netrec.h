// hg_netrec.h -- reading and writing one net's record (w, lambda, Lambda bits,
// S bits) and its compact views.
#pragma once

#include "hg_device.h"

namespace hg {

// Words of a record with WK words per bitset (net_words of such k).
constexpr __host__ __device__ int record_words(int wk) {
  return wk == 1 ? 4 : wk == 2 ? 8 : wk == 4 ? 16 : 32;
}

// Net e's record as it stands: w, lambda, Lambda and S.
template <int WK>
__device__ __forceinline__ void read_record(const InstDesc& D, long long e, int& w, int& lambda,
                                            unsigned (&lam)[WK], unsigned (&one)[WK]) {
  constexpr int N = 2 + 2 * WK, Q = (N + 3) / 4;
  unsigned r[4 * Q];
  const auto rec =
      global_ptr(reinterpret_cast<const u32x4*>(D.netstate + e * record_words(WK)));
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const u32x4 v = rec[i];
    r[4 * i] = v.x;
    r[4 * i + 1] = v.y;
    r[4 * i + 2] = v.z;
    r[4 * i + 3] = v.w;
  }
  w = (int)r[0];
  lambda = (int)r[1];
#pragma unroll
  for (int i = 0; i < WK; ++i) {
    lam[i] = r[2 + i];
    one[i] = r[2 + WK + i];
  }
}

// Net e's whole record (zero padding) and views, written by one lane.  FRESH:
// nothing was written before (pin counts); a round leaves the unused copy of
// weighted nets alone.
template <int WK, bool FRESH>
__device__ __forceinline__ void write_record(const InstDesc& D, long long e, int w, int lambda,
                                             const unsigned (&lam)[WK],
                                             const unsigned (&one)[WK]) {
  constexpr int RW = record_words(WK);
  unsigned r[RW];
#pragma unroll
  for (int i = 0; i < RW; ++i) r[i] = 0;
  r[0] = (unsigned)w;
  r[1] = (unsigned)lambda;
#pragma unroll
  for (int i = 0; i < WK; ++i) {
    r[2 + i] = lam[i];
    r[2 + WK + i] = one[i];
  }
  const auto rec = global_out(reinterpret_cast<u32x4*>(D.netstate + e * RW));
#pragma unroll
  for (int i = 0; i < RW / 4; ++i) {
    const u32x4 q = {r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]};
    rec[i] = q;
  }
  if constexpr (WK == 1) {
    if (D.view == kView16) {
      global_out(D.view_ptr)[e] = (lam[0] & 0xffffu) | (one[0] << 16);
      if (D.sweep == kView8)
        global_out(reinterpret_cast<unsigned short*>(D.sview))[e] =
            (unsigned short)(lam[0] | (one[0] << 8));
      else if (D.sweep == kView4)
        global_out(D.sview)[e] = (unsigned char)(lam[0] | (one[0] << 4));
      return;
    }
    if (D.view == kView32) {
      const u32x2 q = {lam[0], one[0]};
      *global_out(reinterpret_cast<u32x2*>(D.view_ptr + 2 * e)) = q;
      return;
    }
  }
  if constexpr (WK == 2) {
    if (D.view == kView64) {
      const u32x4 q = {lam[0], lam[1], one[0], one[1]};
      *global_out(reinterpret_cast<u32x4*>(D.view_ptr + 4 * e)) = q;
      return;
    }
  }
  // the compact copy is not used for weighted nets: keep it defined (zero)
  if constexpr (FRESH) {
    const int vw = view_words(D.k);
    for (int i = 0; i < vw; ++i) D.view_ptr[e * vw + i] = 0u;
  }
}

}  // namespace hg
