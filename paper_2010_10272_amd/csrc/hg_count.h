// hg_count.h -- pin counts of a wavefront's nets in LDS, shared by the pin-count
// sweep (consecutive nets) and the finalize (the nets that movers touched).
//
// The nets' pins are laid end to end as one run and counted 64 at a time, every
// lane a pin, into byte counters in LDS; then each lane builds its net's bitsets
// from its counters and the Phi rows leave as whole lines.  Nets of more than
// 255 pins, whose counts might not fit a byte, are counted one at a time in
// 32-bit words.
#pragma once

#include "hg_device.h"
#include "hg_internal.h"
#include "hg_netrec.h"

namespace hg {

constexpr int kCountFlight = 4;              // pins in flight per lane
constexpr int kCountStep = kCountFlight * kWave;
constexpr int kByteNet = 255;                // longest net whose counts surely fit a byte

// Most nets a wavefront counts at a time (64 nets' counters fill the LDS for
// k > 128).
__host__ __device__ inline int count_nets(int k) { return k > 128 ? 32 : 64; }
// Words of a net's byte counters in LDS: odd, so that lanes reading their own
// nets' word i use all banks.
__host__ __device__ inline int count_stride(int k) { return ((k + 3) / 4) | 1; }
// LDS words of one wavefront that counts `nets` nets at a time: the counters,
// k words for a long net, a flag byte per position in flight, one word a net.
__host__ __device__ inline int count_words(int k, int nets) {
  return nets * count_stride(k) + k + kCountStep / 4 + kWave;
}

// A run of pins is walked kCountStep places at a time.  It has fewer than 2^31
// places, but its last step may end beyond: places and steps are unsigned.
typedef unsigned RunPlace;
__host__ __device__ inline bool run_left(RunPlace s, int total) { return s < (RunPlace)total; }
// Place `first` within the step at s; kCountStep or more: not in it.
__host__ __device__ inline RunPlace in_step(int first, RunPlace s) { return (RunPlace)first - s; }

struct CountLds {
  unsigned* cnt;               // [nets][stride], zero between calls
  int* big;                    // [k]
  unsigned char* flag;         // [kCountStep], zero between calls
  int* shift;                  // [kWave]: first pin - place in the run, per net
  int stride;
};

// The wavefront's share of the LDS words at `base`, cleared.
__device__ __forceinline__ CountLds count_lds(unsigned* base, int k, int nets) {
  CountLds M;
  M.stride = count_stride(k);
  M.cnt = base;
  M.big = reinterpret_cast<int*>(base + nets * M.stride);
  M.flag = reinterpret_cast<unsigned char*>(M.big + k);
  M.shift = M.big + k + kCountStep / 4;
  for (int i = lane_id(); i < nets * M.stride; i += kWave) M.cnt[i] = 0;
  reinterpret_cast<unsigned*>(M.flag)[lane_id()] = 0;
  return M;
}
static_assert(kCountFlight == 4, "one word of flags per lane");

// Counters -> bits: bit i of `nz` / `one` for byte i of x non-zero / equal to one.
__device__ __forceinline__ void byte_bits(unsigned x, unsigned& nz, unsigned& one) {
  constexpr unsigned low7 = 0x7f7f7f7fu;
  const unsigned a = (((x & low7) + low7) | x) & ~low7;               // bytes != 0
  const unsigned y = x ^ 0x01010101u;
  const unsigned b = ~((((y & low7) + low7) | y) | low7);             // bytes == 1
  // the four top bits to bits 0..3
  nz = ((a >> 7) * 0x10204080u) >> 28;
  one = ((b >> 7) * 0x10204080u) >> 28;
}

// The partition as the counting kernels gather it: part8 (a quarter or an eighth
// of part's bytes, so more of it stays in the L1s) where it is valid, that is
// where the block-weight sweep just wrote it or the rounds since then kept it, and
// no block was out of range; else part.
struct Blocks {
  const int* part;
  const unsigned char* part8;
  bool packed, nibbles;
  __device__ __forceinline__ unsigned operator()(int v) const {
    if (!packed) return (unsigned)part[v];
    if (!nibbles) return part8[v];
    return (part8[(unsigned)v >> 1] >> (4 * (v & 1))) & 15u;
  }
};

__device__ __forceinline__ Blocks blocks_of(const InstDesc& D, bool valid) {
  return Blocks{D.part, D.part8, valid && (*D.err_flags & kErrPart) == 0, D.k <= 16};
}

// Vertex u moves from block a to block t: its place in part8 (two vertices share
// a byte, and other movers their word: an exclusive or).
__device__ __forceinline__ void move_packed(const InstDesc& D, int u, int a, int t) {
  if (D.k > 16) {
    D.part8[u] = (unsigned char)t;
  } else {
    atomicXor(reinterpret_cast<unsigned*>(D.part8) + ((unsigned)u >> 3),
              (unsigned)((a ^ t) & 15) << (4 * (u & 7)));
  }
}

// One net's sets: Lambda, S and lambda.
template <int WK>
struct NetSets {
  unsigned lam[WK], one[WK];
  int lambda;
};

// The pins of the wavefront's nets -- lane's net is pins [b, b + len), len = 0:
// none -- laid end to end, kCountFlight per lane at a time: `load(v, q)` is called
// for the pins of a step (v = -1 past the end) once all of its pins are on their
// way, then `take(net, q)` with the lane index of each pin's net.  So a step waits
// once for its pins and once for what load fetches (netlist, 56.5M pins: pin counts
// 483 us with load called pin by pin, 370 so).  RUN: the nets are neighbours,
// their pins one run already.  A position's net is the count of net starts at or
// before it: a flag per position in LDS, one ballot.  Nets come in the first
// lanes, each of at least one pin (else the flags would miss one).  Every lane
// calls.
template <bool RUN, typename LoadF, typename TakeF>
__device__ __forceinline__ void for_pins(const int* __restrict__ pins, const CountLds& M,
                                         long long b, int len, LoadF load, TakeF take) {
  const int lane = lane_id();
  const int incl = wave_incl_scan(len);
  const int total = last_lane(incl), first = incl - len;   // this net's place in the run
  if constexpr (RUN) pins += __shfl(b, 0);
  else M.shift[lane] = (int)b - first;                     // pin positions are below 2^31
  int before = -1;                                         // last net starting before this step
  for (RunPlace s = 0; run_left(s, total); s += kCountStep) {
    int net[kCountFlight], v[kCountFlight];
    auto nets_of = [&]() {
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const int here = M.flag[q * kWave + lane];
        M.flag[q * kWave + lane] = 0;
        const unsigned long long starts = __ballot(here != 0);
        net[q] = lanes_below(starts, before) + here;
        before += __popcll(starts);
      }
    };
    if constexpr (RUN) {
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const RunPlace p = s + q * kWave + lane;
        v[q] = run_left(p, total) ? pins[p] : -1;
      }
    }
    if (len > 0 && in_step(first, s) < kCountStep) M.flag[in_step(first, s)] = 1;
    if constexpr (!RUN) {
      nets_of();
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const RunPlace p = s + q * kWave + lane;
        v[q] = run_left(p, total) ? pins[(RunPlace)M.shift[net[q]] + p] : -1;
      }
    }
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q) load(v[q], q);
    if constexpr (RUN) nets_of();
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q) take(net[q], q);
    wave_lds_sync();
  }
}

// Counts of one net longer than kByteNet by the whole wavefront, in 32-bit
// words: its Phi row, and the counts left in M.big.
template <typename Block>
__device__ void count_long_net(const InstDesc& D, const CountLds& M, long long e, long long b,
                               long long t, Block block) {
  const int lane = lane_id(), k = D.k;
  for (int i = lane; i < k; i += kWave) M.big[i] = 0;
  wave_lds_sync();
  for (long long p = b + lane; p < t; p += kWave) {
    const unsigned v = block(D.pins[p]);
    if (v < (unsigned)k) atomicAdd(&M.big[v], 1);
  }
  wave_lds_sync();
  for (int i = lane; i < k; i += kWave) D.phi[e * k + i] = M.big[i];
}

// Pin counts of the wavefront's `nets` nets: lane i < nets owns net e, pins
// [b, b + len) (len = 0 in the other lanes).  block(v) is v's block, anything
// >= k where it counts nowhere; pin(v) is called once for every pin of the nets.
// Writes the Phi rows and leaves lane's sets in N.  Pins of a net in one block
// are often neighbours, so each run of equal (net, block) adds once.  vec_phi:
// rows are 16-byte aligned and leave as 16-byte streaming stores.  Every lane
// calls.
template <int WK, bool RUN, typename Block, typename Pin>
__device__ __forceinline__ void count_batch(const InstDesc& D, const CountLds& M, long long e,
                                            long long b, int len, int nets, bool vec_phi,
                                            Block block, Pin pin, NetSets<WK>& N) {
  const int lane = lane_id(), k = D.k, stride = M.stride;
  const unsigned long long is_long = __ballot(len > kByteNet);
  wave_lds_sync();
  unsigned id[kCountFlight];
  for_pins<RUN>(
      D.pins, M, b, len,
      [&](int v, int q) {
        id[q] = ~0u;
        if (v >= 0) {
          pin(v);
          id[q] = block(v);
        }
      },
      [&](int net, int q) {
        bool live = id[q] < (unsigned)k;
        if (is_long) live = live && !((is_long >> (net & 63)) & 1ull);
        // one add per run of equal (net, block) in neighbouring lanes
        const unsigned key = live ? ((unsigned)net << 8) | id[q] : ~0u;
        const unsigned prev = lane_before(key);
        const unsigned long long heads = __ballot(lane == 0 || key != prev);
        if (live && ((heads >> lane) & 1ull)) {
          const unsigned long long later = heads >> lane >> 1;
          const int run_len = later ? __ffsll((long long)later) : kWave - lane;
          atomicAdd(&M.cnt[net * stride + (id[q] >> 2)], (unsigned)run_len << (8 * (id[q] & 3)));
        }
      });
  // lane's net: bitsets from its counters
  N.lambda = 0;
#pragma unroll
  for (int w = 0; w < WK; ++w) {
    N.lam[w] = N.one[w] = 0;
    if (lane < nets) {
      for (int j = 0; j < 8 && w * 32 + 4 * j < k; ++j) {
        unsigned nz, on;
        byte_bits(M.cnt[lane * stride + w * 8 + j], nz, on);
        N.lam[w] |= nz << (4 * j);
        N.one[w] |= on << (4 * j);
      }
    }
    N.lambda += __popc(N.lam[w]);
  }
  // Phi rows, 16 bytes (or one count) per lane and step; M.shift now holds the
  // nets' ids
  M.shift[lane] = (int)e;
  wave_lds_sync();
  if (vec_phi) {
    const int words = k >> 2, all = nets * words;
    int row = lane / words, col = lane % words;             // words <= 64
    const int drow = kWave / words, dcol = kWave % words;
    for (int i = lane; i < all; i += kWave) {
      const unsigned x = M.cnt[row * stride + col];
      const i32x4 o = {(int)(x & 255u), (int)((x >> 8) & 255u), (int)((x >> 16) & 255u),
                       (int)(x >> 24)};
      if (!((is_long >> row) & 1ull))
        __builtin_nontemporal_store(
            o, reinterpret_cast<i32x4*>(D.phi + (long long)M.shift[row] * k) + col);
      row += drow;
      col += dcol;
      if (col >= words) {
        col -= words;
        ++row;
      }
    }
  } else {
    for (int i = lane; i < nets * k; i += kWave) {
      const int row = i / k, col = i % k;
      if (!((is_long >> row) & 1ull))
        D.phi[(long long)M.shift[row] * k + col] =
            (int)((M.cnt[row * stride + (col >> 2)] >> (8 * (col & 3))) & 255u);
    }
  }
  wave_lds_sync();
  for (int i = lane; i < nets * stride; i += kWave) M.cnt[i] = 0;   // for the next nets
  for (unsigned long long left = is_long; left; left &= left - 1) {
    const int j = __ffsll((long long)left) - 1;
    const long long lb = __shfl(b, j);
    count_long_net(D, M, M.shift[j], lb, lb + __shfl(len, j), block);
    if (lane == j) {
      N.lambda = 0;
#pragma unroll
      for (int w = 0; w < WK; ++w) {
        N.lam[w] = N.one[w] = 0;
        for (int i = 0; i < 32 && w * 32 + i < k; ++i) {
          N.lam[w] |= (M.big[w * 32 + i] > 0 ? 1u : 0u) << i;
          N.one[w] |= (M.big[w * 32 + i] == 1 ? 1u : 0u) << i;
        }
        N.lambda += __popc(N.lam[w]);
      }
    }
    wave_lds_sync();
  }
}

// Phi rows can leave as 16-byte stores.
__device__ __forceinline__ bool aligned_rows(const InstDesc& D) {
  return (D.k & 3) == 0 && ((uintptr_t)D.phi & 15) == 0;
}

}  // namespace hg
