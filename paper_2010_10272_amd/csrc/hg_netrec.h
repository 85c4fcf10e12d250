// hg_netrec.h -- building one net's record (w, lambda, Lambda bits, S bits)
// from its pin counts with a group of G lanes (G in {4,8,16,32,64}).
//
// Lane gl of the group handles blocks gl, gl+G, ...; the bitsets come from
// two wave ballots per chunk of G blocks (Phi > 0 and Phi == 1).  Every lane
// ends up holding the record word with index gl, so the record is written
// with one coalesced store per lane.
#pragma once

#include "hg_device.h"

namespace hg {

struct NetBits {
  int lambda;
  unsigned word;   // record word with index = lane-in-group (valid for 1 <= gl < 2+2W)
};

// The bits from the counts cv[c] = Phi(e, c * G + gl) of this lane (MC of them,
// at least ceil(k / G); those past k are ignored).
template <int G, int MC>
__device__ __forceinline__ NetBits net_bits_of(int k, int gl, const int (&cv)[MC]) {
  const int wk = bit_words(k);
  const int shift = (G == kWave) ? 0 : (lane_id() / G) * G;
  const unsigned long long gmask = (G == kWave) ? ~0ull : ((1ull << (G % kWave)) - 1);
  NetBits r;
  r.lambda = 0;
  r.word = 0;
#pragma unroll
  for (int c = 0; c < MC; ++c) {
    if (c * G >= k) break;                  // the same for every lane
    const int x = c * G + gl < k ? cv[c] : 0;
    const unsigned long long nz = (__ballot(x > 0) >> shift) & gmask;
    const unsigned long long one = (__ballot(x == 1) >> shift) & gmask;
    r.lambda += __popcll(nz);
    if (G <= 32) {                    // chunk c fills bits [c*G % 32, +G) of word c*G/32
      const int wd = (c * G) >> 5, sh = (c * G) & 31;
      if (gl == 2 + wd) r.word |= (unsigned)nz << sh;
      if (gl == 2 + wk + wd) r.word |= (unsigned)one << sh;
    } else {
      const int j0 = 2 * c;
      if (gl == 2 + j0) r.word = (unsigned)nz;
      if (gl == 3 + j0) r.word = (unsigned)(nz >> 32);
      if (gl == 2 + wk + j0) r.word = (unsigned)one;
      if (gl == 3 + wk + j0) r.word = (unsigned)(one >> 32);
    }
  }
  if (gl == 1) r.word = (unsigned)r.lambda;
  return r;
}

// Record bits of one net with G lanes; get(i) -> Phi(e,i).  Every chunk's count
// is requested up front (indices past k clamped), as many as k has chunks of G
// blocks rounded up to 1, 2, 4 or 8.  k is the same for every lane of the
// wavefront, so the branch does not diverge.
template <int G, int MC, typename Get>
__device__ __forceinline__ NetBits net_bits_mc(int k, int gl, Get get) {
  int cv[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c) {
    const int i = c * G + gl;
    cv[c] = get(i < k ? i : k - 1);
  }
  return net_bits_of<G, MC>(k, gl, cv);
}

template <int G, typename Get>
__device__ __forceinline__ NetBits net_bits(int k, int gl, Get get) {
  const int nchunks = (k + G - 1) / G;
  if (nchunks <= 1) return net_bits_mc<G, 1>(k, gl, get);
  if (nchunks <= 2) return net_bits_mc<G, 2>(k, gl, get);
  if (nchunks <= 4) return net_bits_mc<G, 4>(k, gl, get);
  return net_bits_mc<G, 8>(k, gl, get);
}

// Write net e's entry of the compact Lambda/S views (NetView) from the record
// words held by the group's lanes (lane 2.. holds Lambda, then S): the one
// behind the records, and the refine call's own narrower one when there is
// one.  All lanes of the wavefront must call it; only `live` groups write.
__device__ __forceinline__ void write_views(const InstDesc& D, long long e, int gl,
                                            const NetBits& b, bool live) {
  if (D.view == kViewFull || D.view == kViewUnit) return;
  const unsigned next = __shfl(b.word, lane_id() + 1);   // the word of lane gl + 1
  if (!live) return;
  if (D.view == kView16) {
    if (gl == 2) {
      D.view_ptr[e] = (b.word & 0xffffu) | (next << 16);
      if (D.sweep == kView8)
        reinterpret_cast<unsigned short*>(D.sview)[e] = (unsigned short)(b.word | (next << 8));
      else if (D.sweep == kView4)
        D.sview[e] = (unsigned char)(b.word | (next << 4));
    }
  } else if (D.view == kView32) {
    if (gl == 2 || gl == 3) D.view_ptr[e * 2 + (gl - 2)] = b.word;
  } else if (D.view == kView64) {
    if (gl >= 2 && gl < 6) D.view_ptr[e * 4 + (gl - 2)] = b.word;
  }
}

// Net e's whole record (zero padding) and views, written by one lane.
template <int WK>
__device__ __forceinline__ void write_record(const InstDesc& D, long long e, int w, int lambda,
                                             const unsigned (&lam)[WK],
                                             const unsigned (&one)[WK]) {
  constexpr int N = 2 + 2 * WK;
  constexpr int RW = N <= 4 ? 4 : N <= 8 ? 8 : N <= 16 ? 16 : 32;   // net_words
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
  u32x4* rec = reinterpret_cast<u32x4*>(D.netstate + e * RW);
#pragma unroll
  for (int i = 0; i < RW / 4; ++i) {
    const u32x4 q = {r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]};
    rec[i] = q;
  }
  if constexpr (WK == 1) {
    if (D.view == kView16) {
      D.view_ptr[e] = (lam[0] & 0xffffu) | (one[0] << 16);
      if (D.sweep == kView8)
        reinterpret_cast<unsigned short*>(D.sview)[e] = (unsigned short)(lam[0] | (one[0] << 8));
      else if (D.sweep == kView4)
        D.sview[e] = (unsigned char)(lam[0] | (one[0] << 4));
      return;
    }
    if (D.view == kView32) {
      const u32x2 q = {lam[0], one[0]};
      *reinterpret_cast<u32x2*>(D.view_ptr + 2 * e) = q;
      return;
    }
  }
  if constexpr (WK == 2) {
    if (D.view == kView64) {
      const u32x4 q = {lam[0], lam[1], one[0], one[1]};
      *reinterpret_cast<u32x4*>(D.view_ptr + 4 * e) = q;
      return;
    }
  }
  // the compact copy is not used for weighted nets: keep it defined (zero)
  const int vw = view_words(D.k);
  for (int i = 0; i < vw; ++i) D.view_ptr[e * vw + i] = 0u;
}

}  // namespace hg
