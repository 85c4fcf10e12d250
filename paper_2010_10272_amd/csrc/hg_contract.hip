// hg_contract.hip -- contraction of a vertex clustering into a coarse
// hypergraph (section "Coarsening", subsection "Contraction"), as a second
// HBM-bound workload beside refinement.
//
//   1. used cluster ids are flagged and renumbered by a prefix sum (the
//      rank of the id among the used ones): map[v];
//   2. coarse vertex weights by integer atomics;
//   3. every net's pins are mapped, sorted and deduplicated in the net's own
//      slots of a scratch copy (tmp[eptr[e] ..]): nets of up to kSmallNet
//      pins up to 64 nets per wavefront in LDS (every pin counts the smaller ones of
//      its net), longer
//      nets one workgroup each (bitonic sort in LDS, or in place beyond the
//      LDS capacity, then a compaction by block scans); the same pass gives
//      the surviving size and the fingerprint;
//   4. nets left with fewer than two pins are dropped;
//   5. identical nets (parallel INRSRT): the fingerprint sum of v^2 and the
//      size of every net are hashed to a key of 16 to 32 bits; a stable sort by key
//      puts candidates for identity next to each other in net-id order, and
//      each net compares its pins with the nets before it in its run, from
//      the run's head, until the first identical one -- whose id is then the
//      lowest among them and becomes the representative; weights are summed
//      at the representative;
//   6. representatives are numbered in net-id order and written out as net
//      CSR with their sorted pins (prefix sums over kept nets and sizes).
// The order of every output is fixed by the definition (ranks, net ids,
// sorted pins), so the result is deterministic and equals the plain
// sequential contraction.
#include <string.h>

#include "hg_device.h"
#include "hg_internal.h"
#include "hg_scan.h"
#include "hg_sort.h"

namespace hg {
namespace {

struct Ct {
  // input
  int n, m;
  long long P;
  const long long* eptr;
  const int* pins;
  const int* vwgt;
  const int* ewgt;
  const int* cluster;
  // output
  int* map;
  int* cvwgt;
  long long* ceptr;
  int* cpins;
  int* cewgt;
  long long* sizes;      // n', m', P'
  // workspace
  unsigned char* used;   // [n]
  long long* rank;       // [n]
  unsigned long long* cw;// [n]
  int* tmp;              // [P]: net e's sorted distinct coarse pins at eptr[e] ..
  int* big;              // [m]: nets longer than kSmallNet
  int* big_count;        // [1]
  int* nsize;            // [m]: pins after deduplication
  unsigned long long* fp;// [m]
  int unit, emit_unit;   // nets per wavefront and turn: sorting, writing (ct_unit)
  int key_bits;          // 8 bits per sorting pass
  unsigned* nkey[2];     // [m]
  int* nval[2];          // [m]
  long long* hscan;      // [m]: run heads before a sorted position
  int* heads;            // [m]: sorted position of every run head
  int* rep;              // [m]: representative, -1 for dropped nets
  unsigned* wsum;        // [m]
  long long* nid;        // [m]: coarse id of a kept net
  long long* npos;       // [m]: first coarse pin of a kept net
  int* err;
};

__global__ __launch_bounds__(kBlock) void k_ct_mark(Ct C) {
  const long long v = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (v >= C.n) return;
  const int c = C.cluster[v];
  if ((unsigned)c >= (unsigned)C.n) {
    atomicOr(C.err, kErrCluster);
    return;
  }
  C.used[c] = 1;
}

struct UsedF {
  const unsigned char* used;
  __device__ long long operator()(long long i) const { return used[i]; }
};

__global__ __launch_bounds__(kBlock) void k_ct_map(Ct C) {
  const long long v = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (v >= C.n) return;
  const int c = C.cluster[v];
  if ((unsigned)c >= (unsigned)C.n) return;
  const int x = (int)C.rank[c];
  C.map[v] = x;
  atomicAdd(&C.cw[x], (unsigned long long)(C.vwgt ? C.vwgt[v] : 1));
}

__global__ __launch_bounds__(kBlock) void k_ct_vweights(Ct C) {
  const long long x = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (x >= C.sizes[0]) return;
  const unsigned long long w = C.cw[x];
  if (w > 0x7fffffffULL) atomicOr(C.err, kErrClusterWeight);
  C.cvwgt[x] = (int)w;
}

__device__ __forceinline__ unsigned ct_hash(unsigned long long fp, int size) {
  unsigned long long h = fp * 0x9E3779B97F4A7C15ULL + (unsigned long long)size * 0xC2B2AE3D27D4EB4FULL;
  h ^= h >> 29;
  h *= 0xBF58476D1CE4E5B9ULL;
  h ^= h >> 32;
  return (unsigned)h;
}

// The sort key of a net: the hash's first key_bits bits, but not the value of
// dropped nets, which all share one run.
__device__ __forceinline__ unsigned ct_dropped(int bits) { return 0xffffffffu >> (32 - bits); }
__device__ __forceinline__ unsigned ct_key(unsigned hash, int bits) {
  const unsigned x = hash >> (32 - bits);
  return x == ct_dropped(bits) ? x - 1 : x;
}

constexpr int kSmallNet = 128;      // nets up to this many pins go through the tiles
constexpr int kNetLdsCap = 8192;    // longer nets sort in LDS up to this many pins

__device__ __forceinline__ void ct_net_done(const Ct& C, long long e, int size,
                                            unsigned long long fp) {
  C.nsize[e] = size;
  C.fp[e] = fp;
  C.nkey[0][e] = size >= 2 ? ct_key(ct_hash(fp, size), C.key_bits) : ct_dropped(C.key_bits);
  C.nval[0][e] = (int)e;
  C.rep[e] = -1;
  C.wsum[e] = 0;
}

// Consecutive nets per wavefront and turn: 64, fewer where that leaves the chip idle
// and each still has 512 pins.  (Contraction of 10,000 nets of 128 pins, us, 64 a
// wavefront 532, so 148; 30,000 of 100 414, 172; 2,000 of 1,500 557, 200.)
int ct_unit(long long m, long long P) {
  int nets = kWave;
  while (nets > 1 && m < 8192LL * nets && nets / 2 * P >= 512 * m) nets >>= 1;
  return nets;
}

// Small nets: a wavefront takes `unit` consecutive nets, as many of them at a time as
// fit its kCtCap LDS places; no barrier, the wavefronts work on their own.  A net
// lies at a multiple of four places, filled up with a value above all others.
//   1. lane = place: the mapped pin goes to LDS (kCtFlight pins and map values on
//      their way; a place's net is the count of net starts at or before it).
//   2. lane = place: the number of smaller values in its net, read four at a time,
//      is its place in sorted order; equal pins write the same value to the same
//      place, so the places left empty are the duplicates'.
//   3. lane = place: the distinct pins leave side by side; prefix sums give
//      sizes and fingerprints.
// Long nets are listed for k_ct_big_nets, 64 at a time, the last ones of a workgroup
// together (one atomic each: one per wavefront, at 12 ns, took 59 us for 10,000 nets of
// 256, two a wavefront).
// What bounds it: the comparisons (a pin's net has 27 pins on average on the
// sparse matrix, whose nets have 10) and the gathers of the map.  Workgroups that
// went through a tile of 1,024 pins together, with a dozen barriers, binary
// searches for the nets and LDS atomics for the fingerprints, took 195 us for 10M
// pins; 128 so.
constexpr int kCtCap = 832;          // LDS places of a wavefront
constexpr int kCtFlight = 4;
constexpr int kCtGrid = 2048;        // persistent workgroups
constexpr int kCtBigGrid = 1024;     // as many as reside (a little over kNetLdsCap words each:
                                     // four a compute unit; with 1280, 256 had to wait for a
                                     // turn of their own)
constexpr int kCtLongEmit = 2048;    // longer nets leave by a workgroup each

struct alignas(16) CtLds {             // val is read four at a time
  int val[kCtCap];
  int sorted[kCtCap];
  unsigned char net[kCtCap];
  unsigned char flag[kCtFlight * kWave];
  int shift[kWave];                  // pin position - place, per net
  int start[kWave + 1];
  int len[kWave + 1];                // pins; then distinct pins before the net
  int big[2 * kWave];
  unsigned long long sum[kWave + 1]; // of squares before the net
};

__device__ __forceinline__ void ct_flush_big(const Ct& C, CtLds& M, int count) {
  const int lane = lane_id();
  unsigned at = 0;
  if (lane == 0) at = atomicAdd((unsigned*)C.big_count, (unsigned)count);
  at = __shfl(at, 0);
  if (lane < count) C.big[at + lane] = M.big[lane];
}

__global__ __launch_bounds__(kBlock) void k_ct_small_nets(Ct C) {
  __shared__ CtLds s_lds[kBlock / kWave];
  __shared__ int s_big[kBlock / kWave], s_at;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  CtLds& M = s_lds[wv];
  constexpr int kEmpty = -1, kAbove = 0x7fffffff;
  for (int i = lane; i < kCtFlight * kWave; i += kWave) M.flag[i] = 0;
  int big = 0;                                        // long nets queued
  for (long long e0 = ((long long)blockIdx.x * (kBlock / kWave) + wv) * C.unit; e0 < C.m;
       e0 += (long long)gridDim.x * (kBlock / kWave) * C.unit) {
    const long long e = e0 + lane;
    long long b = 0;
    int len = 0;
    if (lane < C.unit && e < C.m) {
      b = C.eptr[e];
      const long long size = C.eptr[e + 1] - b;
      len = size > kSmallNet ? kSmallNet + 1 : (int)size;
    }
    const unsigned long long longs = __ballot(len > kSmallNet);
    if (longs) {
      if (len > kSmallNet) {
        M.big[lanes_below(longs, big)] = (int)e;
        len = 0;
      }
      big += __popcll(longs);
      wave_lds_sync();
      if (big >= kWave) {
        ct_flush_big(C, M, kWave);
        wave_lds_sync();
        const int rest = M.big[kWave + lane];
        wave_lds_sync();
        M.big[lane] = rest;
        big -= kWave;
        wave_lds_sync();
      }
    }
    for (int from = 0; from < kWave;) {
      // lanes [from, to): the nets that fit
      const int room = lane >= from ? (len + 3) & ~3 : 0;
      const int incl = wave_incl_scan(room);
      const unsigned long long over = __ballot(incl > kCtCap);
      const int to = over ? __ffsll((long long)over) - 1 : kWave;
      const bool here = lane >= from && lane < to && len > 0;
      const int first = incl - room;
      const unsigned long long in = __ballot(here);
      from = to;
      if (!in) continue;
      const int total = __shfl(incl, 63 - __clzll((long long)in));
      const int at = lanes_below(in, 0), count = __popcll(in);
      if (here) {
        M.shift[at] = (int)b - first;                 // pin positions are below 2^31
        M.start[at] = first;
        M.len[at] = len;
      }
      if (lane == 0) M.start[count] = total;
      // 1. mapped pins
      int before = -1;
      for (int s = 0; s < total; s += kCtFlight * kWave) {
        if (here && first >= s && first < s + kCtFlight * kWave) M.flag[first - s] = 1;
        wave_lds_sync();
        int pin[kCtFlight], x[kCtFlight];
#pragma unroll
        for (int q = 0; q < kCtFlight; ++q) {
          const int p = s + q * kWave + lane;
          const int mark = M.flag[q * kWave + lane];
          M.flag[q * kWave + lane] = 0;
          const unsigned long long starts = __ballot(mark != 0);
          const int net = lanes_below(starts, before) + mark;
          before += __popcll(starts);
          pin[q] = -1;
          if (p < total) {
            M.net[p] = (unsigned char)net;
            if (p - M.start[net] < M.len[net]) pin[q] = C.pins[M.shift[net] + p];
          }
        }
#pragma unroll
        for (int q = 0; q < kCtFlight; ++q) x[q] = pin[q] >= 0 ? C.map[pin[q]] : kAbove;
#pragma unroll
        for (int q = 0; q < kCtFlight; ++q) {
          const int p = s + q * kWave + lane;
          if (p < total) {
            M.val[p] = x[q];
            M.sorted[p] = kEmpty;
          }
        }
        wave_lds_sync();
      }
      // 2. places in sorted order
      for (int p = lane; p < total; p += kWave) {
        const int net = M.net[p], x = M.val[p];
        const int f = M.start[net], t = M.start[net + 1];
        int rank = 0;
        for (int r = f; r < t; r += 4) {
          const int4 v = *reinterpret_cast<const int4*>(&M.val[r]);
          rank += (v.x < x) + (v.y < x) + (v.z < x) + (v.w < x);
        }
        if (p - f < M.len[net]) M.sorted[f + rank] = x;
      }
      wave_lds_sync();
      // 3. out, counted and summed up along the places: a net's size and
      // fingerprint are differences of the sums at its start and end
      int places = 0;
      unsigned long long sum = 0;
      for (int s = 0; s < total; s += kWave) {
        const int p = s + lane;
        const int net = p < total ? M.net[p] : 0, x = p < total ? M.sorted[p] : kEmpty;
        const bool distinct = x != kEmpty;
        const unsigned long long sq =
            distinct ? (unsigned long long)(unsigned)x * (unsigned)x : 0ull;
        const long long upto = wave_incl_scan64((long long)sq);
        const unsigned long long mask = __ballot(distinct);
        const int place = lanes_below(mask, places);
        const int f = M.start[net];
        if (p == f) {
          M.len[net] = place;
          M.sum[net] = sum + (unsigned long long)upto - sq;
        }
        wave_lds_sync();
        if (distinct) C.tmp[M.shift[net] + f + (place - M.len[net])] = x;
        places += __popcll(mask);
        sum += (unsigned long long)last_lane(upto);
      }
      if (lane == 0) {
        M.len[count] = places;
        M.sum[count] = sum;
      }
      wave_lds_sync();
      if (here) ct_net_done(C, e, M.len[at + 1] - M.len[at], M.sum[at + 1] - M.sum[at]);
      wave_lds_sync();
    }
  }
  if (lane == 0) s_big[wv] = big;
  __syncthreads();
  if (threadIdx.x == 0) {
    int all = 0;
    for (int w = 0; w < kBlock / kWave; ++w) {
      const int n = s_big[w];
      s_big[w] = all;
      all += n;
    }
    s_at = all ? (int)atomicAdd((unsigned*)C.big_count, (unsigned)all) : 0;
  }
  __syncthreads();
  if (lane < big) C.big[s_at + s_big[wv] + lane] = M.big[lane];
}

// One workgroup per listed net (workgroups stride over the list).  Up to kBlock
// pins, a thread each: sorted by counting the smaller ones, as the small nets
// (five barriers; a bitonic sort of 256 has 36: 38,000 nets of 129 to 205 pins 428
// us, 300 so).  Longer: map, bitonic sort (LDS when it fits), then keep first
// occurrences in order by block scans over chunks of the sorted row.
__global__ __launch_bounds__(kBlock) void k_ct_big_nets(Ct C) {
  __shared__ __attribute__((aligned(16))) int s_row[kNetLdsCap];
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ int s_prev;
  const int count = *C.big_count;
  for (int idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int e = C.big[idx];
    const long long b = C.eptr[e];
    const int len = (int)(C.eptr[e + 1] - b);
    int* row = C.tmp + b;
    if (len <= kBlock) {
      constexpr int kEmpty = -1;
      int* sorted = s_row + kBlock;
      const int i = threadIdx.x;
      const int x = i < len ? C.map[C.pins[b + i]] : 0x7fffffff;
      s_row[i] = x;
      sorted[i] = kEmpty;
      __syncthreads();
      int rank = 0;
      for (int r = 0; r < len; r += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&s_row[r]);
        rank += (v.x < x) + (v.y < x) + (v.z < x) + (v.w < x);
      }
      if (i < len) sorted[rank] = x;              // equal pins: the same place
      __syncthreads();
      const int y = sorted[i];
      const bool distinct = y != kEmpty;
      const unsigned long long sq = distinct ? (unsigned long long)(unsigned)y * (unsigned)y : 0ull;
      long long size;
      const long long at = block_excl_scan64(distinct, s_tmp, &size);
      if (distinct) row[at] = y;
      const unsigned long long f = (unsigned long long)block_sum64((long long)sq, s_tmp);
      if (i == 0) ct_net_done(C, e, (int)size, f);
      __syncthreads();
      continue;
    }
    int pow2 = 1;
    while (pow2 < len) pow2 <<= 1;
    if (pow2 <= kNetLdsCap) {
      for (int i = threadIdx.x; i < len; i += kBlock) s_row[i] = C.map[C.pins[b + i]];
      __syncthreads();
      bitonic_sort_block(len, pow2, [&](int i) { return s_row[i]; },
                         [&](int i, int x) { s_row[i] = x; });
      for (int i = threadIdx.x; i < len; i += kBlock) row[i] = s_row[i];
    } else {
      for (int i = threadIdx.x; i < len; i += kBlock) row[i] = C.map[C.pins[b + i]];
      __syncthreads();
      bitonic_sort_block(len, pow2, [&](int i) { return row[i]; },
                         [&](int i, int x) { row[i] = x; });
    }
    __syncthreads();
    // compaction in place: writes never pass the chunk being read
    long long kept = 0;
    unsigned long long fp = 0;
    if (threadIdx.x == 0) s_prev = -1;
    __syncthreads();
    for (int c0 = 0; c0 < len; c0 += kBlock) {
      const int i = c0 + threadIdx.x;
      const int x = i < len ? row[i] : 0;
      const int before = i == 0 ? -1 : (threadIdx.x == 0 ? s_prev : row[i - 1]);
      const bool first = i < len && (i == 0 || x != before);
      long long tot;
      const long long at = kept + block_excl_scan64(first ? 1 : 0, s_tmp, &tot);
      if (threadIdx.x == kBlock - 1 || i == len - 1) s_prev = x;
      __syncthreads();
      if (first) {
        row[at] = x;
        fp += (unsigned long long)(unsigned)x * (unsigned)x;
      }
      kept += tot;
      __syncthreads();
    }
    const unsigned long long f = (unsigned long long)block_sum64((long long)fp, s_tmp);
    if (threadIdx.x == 0) ct_net_done(C, e, (int)kept, f);
    __syncthreads();
  }
}

struct HeadF {
  const unsigned* key;
  __device__ long long operator()(long long j) const { return j == 0 || key[j] != key[j - 1]; }
};

__global__ __launch_bounds__(kBlock) void k_ct_heads(Ct C, const unsigned* key) {
  const long long j = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (j >= C.m) return;
  if (j == 0 || key[j] != key[j - 1]) C.heads[C.hscan[j]] = (int)j;
}

__device__ bool ct_same(const Ct& C, long long be, long long bf, int size) {
  for (int x = 0; x < size; ++x)
    if (C.tmp[be + x] != C.tmp[bf + x]) return false;
  return true;
}

// Sorted position j: the first net of j's run (from the head, in net-id
// order) with the same pins is the representative of j's net.  Nearly every run
// is one net, which then writes its weight itself: one atomic per net (20 G a
// second for the whole GPU) took 47 us for 1M nets, 26 with the few that
// are needed.
__global__ __launch_bounds__(kBlock) void k_ct_reps(Ct C, const unsigned* key, const int* val) {
  const long long j = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (j >= C.m) return;
  const unsigned x = key[j];
  if (x == ct_dropped(C.key_bits)) return;
  const int e = val[j];
  const unsigned w = (unsigned)(C.ewgt ? C.ewgt[e] : 1);
  const bool head = j == 0 || x != key[j - 1];
  if (head && (j + 1 == C.m || x != key[j + 1])) {
    C.rep[e] = e;
    C.wsum[e] = w;
    return;
  }
  const int size = C.nsize[e];
  const long long h = C.heads[C.hscan[j] + (head ? 1 : 0) - 1];
  const unsigned long long fe = C.fp[e];
  const long long be = C.eptr[e];
  int r = e;
  for (long long i = h; i < j; ++i) {
    const int f = val[i];
    if (C.nsize[f] != size || C.fp[f] != fe) continue;
    if (ct_same(C, be, C.eptr[f], size)) {
      r = f;
      break;
    }
  }
  C.rep[e] = r;
  atomicAdd(&C.wsum[r], w);
}

struct KeptF {
  const int* rep;
  __device__ long long operator()(long long e) const { return rep[e] == e; }
};

struct KeptSizeF {
  const int* rep;
  const int* nsize;
  __device__ long long operator()(long long e) const { return rep[e] == e ? nsize[e] : 0; }
};

// The pins of the kept nets.  A wavefront takes `unit` consecutive nets, their pins
// laid end to end, kCtFlight per lane at a time (a position's net is the count of
// net starts at or before it: a flag per position in LDS, one ballot).  Bound by its
// bytes; eight lanes a net took 55 us for 9M pins, 22 so.  Nets of more than
// kCtLongEmit pins are left to k_ct_emit_long.
__global__ __launch_bounds__(kBlock) void k_ct_emit(Ct C) {
  __shared__ unsigned char s_flag[kBlock / kWave][kCtFlight * kWave];
  __shared__ long long s_from[kBlock / kWave][kWave], s_to[kBlock / kWave][kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  unsigned char* flag = s_flag[wv];
  for (int i = lane; i < kCtFlight * kWave; i += kWave) flag[i] = 0;
  const long long e = ((long long)blockIdx.x * (kBlock / kWave) + wv) * C.emit_unit + lane;
  const bool kept = lane < C.emit_unit && e < C.m && C.rep[e] == e;
  long long pos = 0;
  int len = 0;
  if (kept) {
    const long long id = C.nid[e];
    pos = C.npos[e];
    len = C.nsize[e];
    C.ceptr[id] = pos;
    C.cewgt[id] = (int)C.wsum[e];
    if (len > kCtLongEmit) len = 0;
  }
  const int incl = wave_incl_scan(len), first = incl - len;
  const int total = last_lane(incl);                      // at most kWave * kCtLongEmit
  if (len > 0) {
    const int at = lanes_below(__ballot(len > 0), 0);
    s_from[wv][at] = C.eptr[e] - first;
    s_to[wv][at] = pos - first;
  }
  int before = -1;
  for (int s = 0; s < total; s += kCtFlight * kWave) {
    if (len > 0 && first >= s && first < s + kCtFlight * kWave) flag[first - s] = 1;
    wave_lds_sync();
    int x[kCtFlight];
    long long to[kCtFlight];
#pragma unroll
    for (int q = 0; q < kCtFlight; ++q) {
      const int p = s + q * kWave + lane;
      const int mark = flag[q * kWave + lane];
      flag[q * kWave + lane] = 0;
      const unsigned long long starts = __ballot(mark != 0);
      const int net = lanes_below(starts, before) + mark;
      before += __popcll(starts);
      if (p < total) {
        x[q] = C.tmp[s_from[wv][net] + p];
        to[q] = s_to[wv][net] + p;
      }
    }
#pragma unroll
    for (int q = 0; q < kCtFlight; ++q)
      if (s + q * kWave + lane < total) C.cpins[to[q]] = x[q];
    wave_lds_sync();
  }
}

// Kept nets of more than kCtLongEmit pins, a workgroup each (they are among the long
// nets that k_ct_small_nets listed; launched for hypergraphs that may have some).
__global__ __launch_bounds__(kBlock) void k_ct_emit_long(Ct C) {
  const int count = *C.big_count;
  for (int idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int e = C.big[idx], size = C.nsize[e];
    if (C.rep[e] != e || size <= kCtLongEmit) continue;
    const int* from = C.tmp + C.eptr[e];
    int* to = C.cpins + C.npos[e];
    for (long long i = threadIdx.x; i < size; i += kBlock * kCtFlight) {
      int x[kCtFlight];
#pragma unroll
      for (int q = 0; q < kCtFlight; ++q) x[q] = i + q * kBlock < size ? from[i + q * kBlock] : 0;
#pragma unroll
      for (int q = 0; q < kCtFlight; ++q)
        if (i + q * kBlock < size) to[i + q * kBlock] = x[q];
    }
  }
}

__global__ void k_ct_close(Ct C) {
  if (threadIdx.x == 0) C.ceptr[C.sizes[1]] = C.sizes[2];
}

}  // namespace

struct ContractLayout {
  size_t used, rank, cw, tmp, big, big_count, nsize, fp, nkey[2], nval[2], hscan, heads, rep, wsum,
      nid, npos, csum, coff, nhist, ndtot, total;
};

static ContractLayout contract_layout(long long n, long long m, long long P) {
  ContractLayout L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t at = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return at;
  };
  L.used = take((size_t)n);
  L.rank = take(8 * (size_t)n);
  L.cw = take(8 * (size_t)n);
  L.tmp = take(4 * (size_t)P);
  L.big = take(4 * (size_t)m);
  L.big_count = take(4);
  for (int i = 0; i < 2; ++i) {
    L.nkey[i] = take(4 * (size_t)m);
    L.nval[i] = take(4 * (size_t)m);
  }
  L.nsize = take(4 * (size_t)m);
  L.fp = take(8 * (size_t)m);
  L.hscan = take(8 * (size_t)m);
  L.heads = take(4 * (size_t)m);
  L.rep = take(4 * (size_t)m);
  L.wsum = take(4 * (size_t)m);
  L.nid = take(8 * (size_t)m);
  L.npos = take(8 * (size_t)m);
  const long long most = n > m ? n : m;
  L.csum = take(8 * (size_t)scan_chunks(most));
  L.coff = take(8 * (size_t)scan_chunks(most));
  L.nhist = take(4 * (size_t)kDigits * sort_tiles(m));
  L.ndtot = take(4 * (size_t)kDigits);
  L.total = off;
  return L;
}

size_t contract_workspace_size(long long n, long long m, long long P) {
  return contract_layout(n, m, P).total;
}

static unsigned blocks_of(long long items) {
  long long b = (items + kBlock - 1) / kBlock;
  return (unsigned)(b < 1 ? 1 : b);
}

static hipError_t launch_contract(hg_graph_s* g, const int* cluster, int* map, int* cvwgt,
                                  long long* ceptr, int* cpins, int* cewgt, long long* sizes,
                                  char* ws, hipStream_t s) {
  const ContractLayout L = contract_layout(g->n, g->m, g->P);
  Ct C;
  memset(&C, 0, sizeof(C));
  C.n = g->n;
  C.m = g->m;
  C.P = g->P;
  C.eptr = g->eptr;
  C.pins = g->pins;
  C.vwgt = g->vwgt;
  C.ewgt = g->ewgt;
  C.cluster = cluster;
  C.map = map;
  C.cvwgt = cvwgt;
  C.ceptr = ceptr;
  C.cpins = cpins;
  C.cewgt = cewgt;
  C.sizes = sizes;
  C.used = (unsigned char*)(ws + L.used);
  C.rank = (long long*)(ws + L.rank);
  C.cw = (unsigned long long*)(ws + L.cw);
  for (int i = 0; i < 2; ++i) {
    C.nkey[i] = (unsigned*)(ws + L.nkey[i]);
    C.nval[i] = (int*)(ws + L.nval[i]);
  }
  C.tmp = (int*)(ws + L.tmp);
  C.big = (int*)(ws + L.big);
  C.big_count = (int*)(ws + L.big_count);
  C.nsize = (int*)(ws + L.nsize);
  C.fp = (unsigned long long*)(ws + L.fp);
  C.hscan = (long long*)(ws + L.hscan);
  C.heads = (int*)(ws + L.heads);
  C.rep = (int*)(ws + L.rep);
  C.wsum = (unsigned*)(ws + L.wsum);
  C.nid = (long long*)(ws + L.nid);
  C.npos = (long long*)(ws + L.npos);
  C.err = (int*)(g->ws + g->lay.flags);
  ScanBufs B;
  B.csum = (long long*)(ws + L.csum);
  B.coff = (long long*)(ws + L.coff);
  const long long n = g->n, m = g->m;
  // one sorting pass (23 us for 1M nets) per 8 bits: at least 16 key values per net
  // up to 2^28 nets, so that few nets that differ share a run
  C.key_bits = m <= (1 << 12) ? 16 : m <= (1 << 20) ? 24 : 32;

  // 1-2. renumbering, map, coarse weights
  ZeroRanges Z;
  Z.add(C.used, n);
  Z.add((void*)C.cw, (long long)sizeof(long long) * n);
  Z.add(C.big_count, (long long)sizeof(int));
  hipError_t e = zero_ranges(Z, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ct_mark, dim3(blocks_of(n)), dim3(kBlock), 0, s, C);
  exclusive_scan(UsedF{C.used}, n, C.rank, &sizes[0], B, s);
  hipLaunchKernelGGL(k_ct_map, dim3(blocks_of(n)), dim3(kBlock), 0, s, C);
  hipLaunchKernelGGL(k_ct_vweights, dim3(blocks_of(n)), dim3(kBlock), 0, s, C);

  // 3-4. per net: mapped, sorted, deduplicated pins, size, fingerprint
  const long long small_pins = (long long)kSmallNet * m;   // at most: longer nets are listed
  C.unit = ct_unit(m, g->P < small_pins ? g->P : small_pins);
  C.emit_unit = ct_unit(m, g->P);
  const unsigned units = (unsigned)units_of(m, C.unit * (kBlock / kWave));
  const unsigned emits = (unsigned)units_of(m, C.emit_unit * (kBlock / kWave));
  const unsigned sg = units < kCtGrid ? units : kCtGrid;
  hipLaunchKernelGGL(k_ct_small_nets, dim3(sg), dim3(kBlock), 0, s, C);
  hipLaunchKernelGGL(k_ct_big_nets, dim3(kCtBigGrid), dim3(kBlock), 0, s, C);

  // 5. identical nets
  int ncur = 0;
  SortPass SN;
  SN.hist = (unsigned*)(ws + L.nhist);
  SN.dtot = (unsigned*)(ws + L.ndtot);
  SN.n = (int)m;
  SN.tiles = sort_tiles(m);
  for (int shift = 0; shift < C.key_bits; shift += 8) {
    SN.key_in = C.nkey[ncur];
    SN.val_in = C.nval[ncur];
    SN.key_out = C.nkey[ncur ^ 1];
    SN.val_out = C.nval[ncur ^ 1];
    SN.shift = shift;
    sort_pass(SN, s);
    ncur ^= 1;
  }
  exclusive_scan(HeadF{C.nkey[ncur]}, m, C.hscan, nullptr, B, s);
  hipLaunchKernelGGL(k_ct_heads, dim3(blocks_of(m)), dim3(kBlock), 0, s, C, C.nkey[ncur]);
  hipLaunchKernelGGL(k_ct_reps, dim3(blocks_of(m)), dim3(kBlock), 0, s, C, C.nkey[ncur],
                     C.nval[ncur]);

  // 6. coarse net CSR in representative order
  exclusive_scan(KeptF{C.rep}, m, C.nid, &sizes[1], B, s);
  exclusive_scan(KeptSizeF{C.rep, C.nsize}, m, C.npos, &sizes[2], B, s);
  hipLaunchKernelGGL(k_ct_emit, dim3(emits), dim3(kBlock), 0, s, C);
  if (g->info.max_net_size > kCtLongEmit)
    hipLaunchKernelGGL(k_ct_emit_long, dim3(kCtBigGrid), dim3(kBlock), 0, s, C);
  hipLaunchKernelGGL(k_ct_close, dim3(1), dim3(kWave), 0, s, C);
  return hipGetLastError();
}

}  // namespace hg

using hg::fail;

extern "C" {

size_t hg_contract_workspace_size(int32_t n, int32_t m, int64_t P) {
  if (n < 1 || m < 1 || P < 1 || P > 0x7fffffffLL) return 0;
  return hg::contract_workspace_size(n, m, P);
}

hg_status hg_contract(hg_graph g, const int32_t* cluster, int32_t* map, int32_t* cvwgt,
                      int64_t* ceptr, int32_t* cpins, int32_t* cewgt, int64_t* sizes,
                      void* workspace, size_t ws_bytes, void* stream) {
  if (!g) return fail(HG_ERR_INVALID, "graph handle is NULL");
  if (!cluster || !map || !cvwgt || !ceptr || !cpins || !cewgt || !sizes)
    return fail(HG_ERR_INVALID, "cluster, map, cvwgt, ceptr, cpins, cewgt and sizes must be "
                                "non-NULL");
  if (g->P > 0x7fffffffLL)
    return fail(HG_ERR_UNSUPPORTED, "contraction needs fewer than 2^31 pins");
  const size_t need = hg::contract_workspace_size(g->n, g->m, g->P);
  if (!workspace || ws_bytes < need)
    return fail(HG_ERR_WORKSPACE, "contraction workspace needs %zu bytes (got %zu)", need,
                ws_bytes);
  if (((uintptr_t)workspace & 255) != 0)
    return fail(HG_ERR_INVALID, "the contraction workspace must be 256-byte aligned");
  HG_TRY(hg::launch_contract(g, cluster, map, cvwgt, (long long*)ceptr, cpins, cewgt,
                             (long long*)sizes, (char*)workspace, (hipStream_t)stream),
         "contraction");
  return HG_OK;
}

}  // extern "C"
