// hg_count.h -- pin counts of a wavefront's nets in LDS, shared by the pin-count
// sweep (consecutive nets) and the finalize (the nets that movers touched).
//
// The nets' pins are laid end to end as one run and counted 64 at a time, every
// lane a pin, into byte counters in LDS; then each lane builds its net's bitsets
// from its counters and the Phi rows leave as whole lines.  Where a net has more
// than 255 pins, so that a count might not fit a byte, the same places hold its 32-bit
// counters.  Nets of more than kWaveNet pins are left to a workgroup each
// (k_long_nets).
#pragma once

#include "hg_device.h"
#include "hg_internal.h"
#include "hg_netrec.h"

namespace hg {

constexpr int kCountFlight = 4;              // pins in flight per lane
constexpr int kCountStep = kCountFlight * kWave;
constexpr int kByteNet = 255;                // longest net whose counts surely fit a byte
constexpr int kWaveNet = 2048;               // longest net that a wavefront counts

// Most nets a wavefront counts at a time (64 nets' counters fill the LDS for
// k > 128).
__host__ __device__ inline int count_nets(int k) { return k > 128 ? 32 : 64; }
// Words of a net's byte counters in LDS: odd, so that lanes reading their own
// nets' word i use all banks.
__host__ __device__ inline int count_stride(int k) { return ((k + 3) / 4) | 1; }
// Words of a wavefront's counters: `nets` nets of bytes, or one of 32-bit counters.
__host__ __device__ inline int counter_words(int k, int nets) {
  const int bytes = nets * count_stride(k);
  return bytes > k ? bytes : k;
}
// LDS words of one wavefront that counts `nets` nets at a time: the counters, a
// flag byte per position in flight, one word a net.
__host__ __device__ inline int count_words(int k, int nets) {
  return counter_words(k, nets) + kCountStep / 4 + kWave;
}

// A run of pins is walked kCountStep places at a time.  It has fewer than 2^31
// places, but its last step may end beyond: places and steps are unsigned.
typedef unsigned RunPlace;
__host__ __device__ inline bool run_left(RunPlace s, int total) { return s < (RunPlace)total; }
// Place `first` within the step at s; kCountStep or more: not in it.
__host__ __device__ inline RunPlace in_step(int first, RunPlace s) { return (RunPlace)first - s; }

struct CountLds {
  unsigned* cnt;               // [nets][stride], zero between calls
  unsigned char* flag;         // [kCountStep], zero between calls
  int* shift;                  // [kWave]: first pin - place in the run, per net
  int stride;
  int words;                   // of cnt
};

// The wavefront's share of the LDS words at `base`, cleared.
__device__ __forceinline__ CountLds count_lds(unsigned* base, int k, int nets) {
  CountLds M;
  M.stride = count_stride(k);
  M.words = counter_words(k, nets);
  M.cnt = base;
  M.flag = reinterpret_cast<unsigned char*>(base + M.words);
  M.shift = reinterpret_cast<int*>(base + M.words + kCountStep / 4);
  for (int i = lane_id(); i < M.words; i += kWave) M.cnt[i] = 0;
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
//
// The blocks of N pins (v = -1: none, and then ~0) are read together: all loads
// first, in no branch of their own (a pin without a vertex reads vertex 0's place),
// and what has to be done to the values after them.  With a branch, a load and a
// shift per pin the compiler waited for each before the next, and through generic
// pointers for the LDS too (pin counts of 10M pins, k = 8 55 -> 52 us, k = 64 84 -> 75).
struct Blocks {
  const int* part;
  const unsigned char* part8;
  bool packed;
  int two;                     // 1: two vertices a byte
  template <int N>
  __device__ __forceinline__ void operator()(const int (&v)[N], unsigned (&id)[N]) const {
    if (packed) {
#pragma unroll
      for (int q = 0; q < N; ++q) id[q] = global_ptr(part8)[(unsigned)(v[q] < 0 ? 0 : v[q]) >> two];
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const unsigned half = (id[q] >> (4 * (v[q] & 1))) & 15u;
        id[q] = v[q] < 0 ? ~0u : two ? half : id[q];
      }
    } else {
#pragma unroll
      for (int q = 0; q < N; ++q) id[q] = (unsigned)global_ptr(part)[v[q] < 0 ? 0 : v[q]];
#pragma unroll
      for (int q = 0; q < N; ++q) id[q] = v[q] < 0 ? ~0u : id[q];
    }
  }
};

__device__ __forceinline__ Blocks blocks_of(const InstDesc& D, bool valid) {
  return Blocks{D.part, D.part8, valid && (*D.err_flags & kErrPart) == 0, D.k <= 16 ? 1 : 0};
}

// Makes pins eligible for the next round.
struct EligiblePins {
  unsigned char* eligible;
  __device__ __forceinline__ void operator()(const int (&v)[kCountFlight]) const {
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q)
      if (v[q] >= 0) global_out(eligible)[v[q]] = 1;
  }
};

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

// Words h and h + 1 of a net's sets from the ballots over its blocks 32 h .. 32 h + 63,
// where `mine`.
template <int WK>
__device__ __forceinline__ void set_words(NetSets<WK>& N, int h, unsigned long long nz,
                                          unsigned long long one, bool mine) {
  if (!mine) return;
  N.lam[h] = (unsigned)nz;
  N.one[h] = (unsigned)one;
  if (h + 1 < WK) {
    N.lam[h + 1] = (unsigned)(nz >> 32);
    N.one[h + 1] = (unsigned)(one >> 32);
  }
  N.lambda += __popcll(nz);
}

// The pins of the wavefront's nets -- lane's net is pins [b, b + len), len = 0:
// none -- laid end to end, kCountFlight per lane at a time: `load(v)` gets the
// pins of a step (-1 past the end), then `take(net, q)` is called for each with the
// rank of its net among those that are there.  So a step waits once for its pins and
// once for what load fetches.
// RUN: the nets are neighbours in the first lanes, their pins one run already.  A
// position's net is the count of net starts at or before it: a flag per position
// in LDS, one ballot.  Every lane calls.
template <bool RUN, typename LoadF, typename TakeF>
__device__ __forceinline__ void for_pins(const int* pin_array, const CountLds& M, long long b,
                                         int len, LoadF load, TakeF take) {
  auto pins = global_ptr(pin_array);
  const int lane = lane_id();
  const int incl = wave_incl_scan(len);
  const int total = last_lane(incl), first = incl - len;   // this net's place in the run
  if constexpr (RUN) pins += __shfl(b, 0);
  else if (const int at = lanes_below(__ballot(len > 0), 0); len > 0)
    M.shift[at] = (int)b - first;                          // pin positions are below 2^31
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
    load(v);
    if constexpr (RUN) nets_of();
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q) take(net[q], q);
    wave_lds_sync();
  }
}

// One add per run of equal keys in neighbouring lanes (pins of a net in one block
// are often neighbours).  `live` lanes' key is below 2^32 - 1; add(n) is called by
// the first lane of each run of n.  Every lane calls.
template <typename Add>
__device__ __forceinline__ void add_runs(bool live, unsigned key, Add add) {
  const int lane = lane_id();
  key = live ? key : ~0u;
  const unsigned prev = lane_before(key);
  const unsigned long long heads = __ballot(lane == 0 || key != prev);
  if (live && ((heads >> lane) & 1ull)) {
    const unsigned long long later = heads >> lane >> 1;
    add(later ? __ffsll((long long)later) : kWave - lane);
  }
}

// Counts of the nets of `in` lanes, each of at most kByteNet pins: byte counters, the
// nets' in the order of their lanes; N is set for every lane.
template <int WK, bool RUN, typename Block, typename Pin>
__device__ __forceinline__ void count_bytes(const InstDesc& D, const CountLds& M, long long e,
                                            long long b, int len, bool in, bool vec_phi,
                                            Block block, Pin pin, NetSets<WK>& N) {
  const int lane = lane_id(), k = D.k, stride = M.stride;
  const unsigned long long nets_in = __ballot(in);
  const int nets = __popcll(nets_in), mine = RUN ? lane : lanes_below(nets_in, 0);
  wave_lds_sync();
  unsigned id[kCountFlight];
  for_pins<RUN>(
      D.pins, M, b, in ? len : 0,
      [&](const int (&v)[kCountFlight]) {
        block(v, id);
        pin(v);
      },
      [&](int net, int q) {
        add_runs(id[q] < (unsigned)k, ((unsigned)net << 8) | id[q], [&](int n) {
          atomicAdd(&M.cnt[net * stride + (id[q] >> 2)], (unsigned)n << (8 * (id[q] & 3)));
        });
      });
  // lane's net: bitsets from its counters
  N.lambda = 0;
#pragma unroll
  for (int w = 0; w < WK; ++w) {
    N.lam[w] = N.one[w] = 0;
    if (in) {
      for (int j = 0; j < 8 && w * 32 + 4 * j < k; ++j) {
        unsigned nz, on;
        byte_bits(M.cnt[mine * stride + w * 8 + j], nz, on);
        N.lam[w] |= nz << (4 * j);
        N.one[w] |= on << (4 * j);
      }
    }
    N.lambda += __popc(N.lam[w]);
  }
  // Phi rows, 16 bytes (or one count) per lane and step; M.shift now holds the
  // nets' ids
  if (in) M.shift[mine] = (int)e;
  wave_lds_sync();
  if (vec_phi) {
    const int words = k >> 2, all = nets * words;
    int row = lane / words, col = lane % words;             // words <= 64
    const int drow = kWave / words, dcol = kWave % words;
    for (int i = lane; i < all; i += kWave) {
      const unsigned x = M.cnt[row * stride + col];
      const i32x4 o = {(int)(x & 255u), (int)((x >> 8) & 255u), (int)((x >> 16) & 255u),
                       (int)(x >> 24)};
      __builtin_nontemporal_store(
          o, global_out(reinterpret_cast<i32x4*>(D.phi + (long long)M.shift[row] * k)) + col);
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
      global_out(D.phi)[(long long)M.shift[row] * k + col] =
          (int)((M.cnt[row * stride + (col >> 2)] >> (8 * (col & 3))) & 255u);
    }
  }
  wave_lds_sync();
  for (int i = lane; i < nets * stride; i += kWave) M.cnt[i] = 0;   // for the next nets
}

// The same for the longer nets of lanes `left`, one net after the other: 32-bit
// counters, kCountStep pins a step, the next step's pins (or the next net's) on their
// way while this one's are counted; the sets and the Phi row by ballots.  N is set
// for those lanes.  (Pin counts of 2,000 nets of 1,500 pins, k = 8, per call, us: a
// lane group per net 45, 64 pins a step after a first walk past them 136, so 32.)
template <int WK, typename Block, typename Pin>
__device__ __forceinline__ void count_mid_nets(const InstDesc& D, const CountLds& M, long long e,
                                               long long b, int len, unsigned long long left,
                                               Block block, Pin pin, NetSets<WK>& N) {
  const int lane = lane_id(), k = D.k;
  int owner = 0, size = 0, s = 0;            // wave-uniform: this step's net and place
  long long at = 0;
  int next[kCountFlight];
  // the pins of the step after place s of the net, or of the next net's first
  auto advance = [&]() {
    s += kCountStep;
    if (s >= size) {
      owner = left ? __ffsll((long long)left) - 1 : -1;
      left &= left - 1;
      s = 0;
      size = owner < 0 ? 0 : __builtin_amdgcn_readlane(len, owner);
      at = owner < 0 ? 0 : lane_value(b, owner);
    }
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q) {
      const int p = s + q * kWave + lane;
      next[q] = p < size ? global_ptr(D.pins)[at + p] : -1;
    }
  };
  advance();
  while (owner >= 0) {
    const int net = owner;
    unsigned id[kCountFlight];
    block(next, id);
    pin(next);
    advance();
#pragma unroll
    for (int q = 0; q < kCountFlight; ++q)
      add_runs(id[q] < (unsigned)k, id[q], [&](int n) { atomicAdd(&M.cnt[id[q]], (unsigned)n); });
    if (s > 0) continue;                     // more of the same net
    wave_lds_sync();
    const long long phi_row = lane_value(e, net) * k;
    if (lane == net) N.lambda = 0;
#pragma unroll
    for (int h = 0; h < WK; h += 2) {
      const int i = h * 32 + lane;
      const int x = i < k ? (int)M.cnt[i] : 0;
      if (i < k) {
        M.cnt[i] = 0;                        // for the next net
        global_out(D.phi)[phi_row + i] = x;
      }
      set_words<WK>(N, h, __ballot(x != 0), __ballot(x == 1), lane == net);
    }
    wave_lds_sync();
  }
}

// Pin counts of the wavefront's nets: lane owns net e, pins [b, b + len), len = 0:
// none.  RUN: neighbouring nets in the first lanes.  block(v, id) gives the blocks of a
// lane's kCountFlight pins (-1: none), anything >= k where a pin counts nowhere;
// pin(v) gets the same pins, every pin of the nets once.
// Writes the Phi rows and leaves lane's sets in N.  Nets of more than kWaveNet
// pins are passed over: neither counted nor written.  vec_phi: rows are 16-byte
// aligned and leave as 16-byte streaming stores.  Every lane calls.
template <int WK, bool RUN, typename Block, typename Pin>
__device__ __forceinline__ void count_batch(const InstDesc& D, const CountLds& M, long long e,
                                            long long b, int len, bool vec_phi, Block block,
                                            Pin pin, NetSets<WK>& N) {
  const bool in = len > 0 && len <= kByteNet;
  if constexpr (RUN) {
    if (!__any(len > kByteNet)) {
      count_bytes<WK, true>(D, M, e, b, len, in, vec_phi, block, pin, N);
      return;
    }
  }
  count_bytes<WK, false>(D, M, e, b, len, in, vec_phi, block, pin, N);
  if (const unsigned long long rest = __ballot(len > kByteNet && len <= kWaveNet)) {
    wave_lds_sync();
    count_mid_nets<WK>(D, M, e, b, len, rest, block, pin, N);
  }
}

// Phi rows can leave as 16-byte stores.
__device__ __forceinline__ bool aligned_rows(const InstDesc& D) {
  return (D.k & 3) == 0 && ((uintptr_t)D.phi & 15) == 0;
}

}  // namespace hg
