// hg_lp.hip -- one synchronous label-propagation round (section "Label
// Propagation"), split into select / approve / apply / finalize kernels that
// all read the round-start state.
//
//   select     per eligible vertex: boundary test, best feasible target by
//              (gain desc, block weight asc, block id asc), move rule; writes
//              a candidate word per vertex and adds c(u) to a per-(target,
//              gain) weight histogram.
//   threshold  per target block: the highest gain g* at which the cumulative
//              candidate weight (from the top gain down) overflows
//              L_max - c(V_t); gains above g* are approved whole.
//   tilesum    per tile of 512 vertices: weight of gain-g* candidates per
//              target block (vertex id order is tile order).
//   tilescan   per target block: the tile where the budget runs out.
//   approve    per tile: decide every candidate; the one boundary tile per
//              block is resolved by a workgroup-wide prefix sum in vertex
//              order.  Approved moves are applied right away: part, block
//              weights, touched nets flagged.
//   finalize   per touched net (k_long_nets where it is long): Phi, Lambda, S and lambda counted from its
//              pins, the attributed km1 change summed from the blocks that
//              left and entered Lambda (subsection "Attributed Gains"), its
//              pins made eligible for the next round.
//   stats      one workgroup per instance sums the counter slots into the
//              round record.
//
// Every kernel takes a Launch: one instance by value, or a batch of
// instances with a per-workgroup work table (see hg_internal.h).
//
// Candidate word: (gain << 32) | target, or -1 for "no candidate".
#include <limits.h>

#include "hg_bits.h"
#include "hg_count.h"
#include "hg_device.h"
#include "hg_gain_deltas.h"
#include "hg_internal.h"
#include "hg_lp.h"
#include "hg_sweep.h"

namespace hg {

// Contiguous XCD-aware split: workgroup blockIdx < grid gets units
// [lb*per, (lb+1)*per).
__device__ __forceinline__ WorkItem xcd_block(long long units, unsigned grid) {
  const long long lb = xcd_remap(blockIdx.x, grid);
  const long long per = (units + grid - 1) / grid;
  long long end = (lb + 1) * per;
  if (end > units) end = units;
  WorkItem w;
  w.inst = 0;
  w.first = (int)(lb * per);
  w.stride = 1;
  w.count = lb * per < end ? (int)(end - lb * per) : 0;
  return w;
}

__device__ __forceinline__ WorkItem single_unit(int unit) {
  WorkItem w;
  w.inst = 0;
  w.first = unit;
  w.count = 1;
  w.stride = 1;
  return w;
}

// --------------------------------------------------------------- select

// Light vertices, one thread each.  Unit: a chunk of 256 vertices.  Single
// instance: persistent grid, XCD-aware sweep (each XCD walks one vertex
// range with its workgroups side by side, so neighbouring vertices' net
// records stay in that XCD's L2).  Candidate weights go to an LDS histogram
// (buckets [0, B) per target block, B = min(256, 2048/k)); higher gains and
// the final flush go to the histogram replica of this workgroup's XCD.
constexpr int kDenseWave = 3 * kWave / 4;   // eligible lanes that make a wave's slice dense

// The sweep's end: the workgroup's counts (each below 2^31, so two fit one
// 64-bit sum) to its counter slots, and `flush` once every thread is done.
template <typename F>
__device__ __forceinline__ void add_select_counts(const InstDesc& D, unsigned long long* s_sums,
                                                  int elig, int bnd, int cand, int apins,
                                                  F flush) {
  const long long eb = wave_sum((long long)elig | ((long long)bnd << 32));
  const long long ca = wave_sum((long long)cand | ((long long)apins << 32));
  if (lane_id() == 0) {
    atomicAdd(&s_sums[0], (unsigned long long)eb);
    atomicAdd(&s_sums[1], (unsigned long long)ca);
  }
  __syncthreads();
  flush();
  if (threadIdx.x < 4) {
    const int which[4] = {kCtrEligible, kCtrBoundary, kCtrCandidates, kCtrActivePins};
    const unsigned long long v = (s_sums[threadIdx.x / 2] >> (32 * (threadIdx.x % 2))) & 0xffffffffu;
    if (v) atomicAdd(&D.ctr->slot[which[threadIdx.x]][blockIdx.x % kSlots], v);
  }
}

template <int WK, int VIEW, int U>
__global__ __launch_bounds__(kBlock) void k_select_light(Launch L) {
  __shared__ long long s_W[HG_MAX_K];
  __shared__ unsigned s_open[WK];
  __shared__ unsigned long long s_hist[kLdsHistEntries];
  __shared__ unsigned long long s_sums[2];
  __shared__ int s_q[kBlock / kWave][2 * kWave];   // per-wave queues of eligible vertices
  const InstDesc D0 = L.one;
  const WorkItem wi = work_item(L, xcd_sweep(units_of(D0.n, kBlock)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, B = D.lds_buckets, n = D.n;
  const long long lmax = D.lmax;
  for (int i = threadIdx.x; i < WK; i += kBlock) s_open[i] = 0;
  if (threadIdx.x < 2) s_sums[threadIdx.x] = 0;
  for (int i = threadIdx.x; i < k * B; i += kBlock) s_hist[i] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < k; i += kBlock) {
    long long W = D.block_w[i];
    s_W[i] = W;
    if (W + D.cmax <= lmax) atomicOr(&s_open[i >> 5], 1u << (i & 31));
  }
  __syncthreads();
  unsigned long long* my_hist = D.hist + (size_t)(blockIdx.x % D.hist_reps) * D.hist_stride;
  // per thread: at most n vertices and P pins, both below 2^31
  int n_elig = 0, n_bnd = 0, n_cand = 0, n_apins = 0;
  // valid-block masks (only blocks < k; guards against stale caller state)
  unsigned valid[WK];
#pragma unroll
  for (int w = 0; w < WK; ++w) {
    const int lo = w * 32;
    valid[w] = k >= lo + 32 ? ~0u : (k > lo ? (1u << (k - lo)) - 1u : 0u);
  }
  const void* __restrict__ view =
      VIEW == kView8 || VIEW == kView4 ? (const void*)D.sview : (const void*)D.view_ptr;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  // Each wave queues the eligible vertices of its 64-vertex slices in LDS
  // and processes them 64 at a time, so that later rounds (few eligible
  // vertices) run full waves instead of mostly idle ones; slices that are
  // mostly eligible (every vertex in round 1) are processed in place.  No
  // workgroup barrier is involved, so waves keep sweeping independently.
  // Every vertex gets its moved flag cleared, and the non-eligible ones
  // their "no candidate" word, when its slice is read.
  //
  // One wavefront's vertices: lane's vertex u, if `act`.
  auto wave_vertices = [&](const long long u, const bool act) {
    int a = 0, deg = 0;
    long long b0 = 0, cu = 1;
    bool mine = false;
    if (act) {
      a = D.part[u];
      b0 = D.vptr[u];
      const long long len = D.vptr[u + 1] - b0;
      if (D.vwgt) cu = D.vwgt[u];
      if ((unsigned)a >= (unsigned)k) {
        atomicOr(D.err_flags, kErrPart);
        D.cand[u] = -1;
        D.eligible[u] = 0;
      } else if (len <= kLightLimit) {           // longer rows: the heavy kernel's
        mine = true;
        deg = (int)len;
      }
    }
    if (!mine) a = 0;
    RowSums<WK, VIEW> R;
    walk_row<WK, VIEW, U>(D, view, b0, deg, a, R);
    if (!mine || R.heavy) return;
    D.eligible[u] = 0;
    n_elig += 1;
    long long out = -1;
    const int aw = a >> 5;
    const unsigned abit = 1u << (a & 31);
    // blocks of u's nets beside its own: there is one iff u is on a cut net
    unsigned T[WK], anyT = 0;
    R.C.nonzero(T);
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      T[w] &= w == aw ? valid[w] & ~abit : valid[w];
      anyT |= T[w];
    }
    if (anyT) {
      n_bnd += 1;
      n_apins += deg;
      unsigned F[WK];
      unsigned anyF = 0;
#pragma unroll
      for (int w = 0; w < WK; ++w) {
        F[w] = T[w] & s_open[w];
        unsigned rest = T[w] & ~s_open[w];
        while (rest) {
          int b = __ffs(rest) - 1;
          rest &= rest - 1;
          if (s_W[w * 32 + b] + cu <= lmax) F[w] |= 1u << b;
        }
        anyF |= F[w];
      }
      if (anyF) {
        const int conn = (int)R.C.narrow_to_max(F);
        int t = -1;
        long long tw = 0;
#pragma unroll
        for (int w = 0; w < WK; ++w) {
          unsigned x = F[w];
          while (x) {
            int b = __ffs(x) - 1;
            x &= x - 1;
            int i = w * 32 + b;
            long long Wi = s_W[i];
            if (t < 0 || Wi < tw) {
              t = i;
              tw = Wi;
            }
          }
        }
        const int g = R.ben - R.tot + conn;
        if (g > 0 || (g == 0 && tw + cu < s_W[a])) {
          out = pack_cand(g, t);
          n_cand += 1;
          if (g < B)
            atomicAdd(&s_hist[t * B + g], (unsigned long long)cu);
          else
            atomicAdd(&my_hist[t * kBuckets + (g < kBuckets ? g : kBuckets - 1)],
                      (unsigned long long)cu);
        }
      }
    }
    D.cand[u] = out;
  };
  int* my_q = s_q[wv];
  int qn = 0;                                  // this wave's queue length (wave-uniform)
  // the next slice's flags are on their way while a slice is processed
  auto flag_of = [&](int it) {
    const long long u = ((long long)wi.first + (long long)it * wi.stride) * kBlock + threadIdx.x;
    return it < wi.count && u < n ? D.eligible[u] : (unsigned char)0;
  };
  unsigned char next_flag = flag_of(0);
  // one call site of wave_vertices (the select body is large): the extra last
  // iteration flushes the queue
  for (int it = 0; it <= wi.count; ++it) {
    long long u = 0;
    bool act = false, run = false;
    if (it < wi.count) {
      const long long c = (long long)wi.first + (long long)it * wi.stride;
      u = c * kBlock + threadIdx.x;
      const bool el = next_flag != 0;
      next_flag = flag_of(it + 1);
      if (u < n) {
        if (D.moved) D.moved[u] = 0;
        if (!el) D.cand[u] = -1;
      }
      const unsigned long long mask = __ballot(el);
      const int cnt = __popcll(mask);
      if (cnt >= kDenseWave) {                 // mostly eligible: in place
        act = el;
        run = true;
      } else {
        if (el) my_q[qn + __popcll(mask & ((1ull << lane) - 1))] = (int)u;
        qn += cnt;                             // < 2 * kWave
        wave_lds_sync();
        if (qn >= kWave) {
          u = my_q[lane];
          act = run = true;
          const int rest = qn - kWave;
          const int keep = lane < rest ? my_q[kWave + lane] : 0;
          wave_lds_sync();
          if (lane < rest) my_q[lane] = keep;
          qn = rest;
          wave_lds_sync();
        }
      }
    } else if (qn > 0) {
      run = true;
      act = lane < qn;
      u = act ? my_q[lane] : 0;
    }
    if (run) wave_vertices(u, act);
  }
  add_select_counts(D, s_sums, n_elig, n_bnd, n_cand, n_apins, [&] {
    for (int i = threadIdx.x; i < k * B; i += kBlock) {
      const unsigned long long v = s_hist[i];
      if (v) atomicAdd(&my_hist[(i / B) * kBuckets + (i % B)], v);
    }
  });
}

// One wavefront per heavy vertex (w(I(u)) > 255): per-block connection
// weights in LDS (int32, enough because w(E) < 2^31), lanes stride over I(u).
// Unit: 4 consecutive entries of the heavy list (one per wavefront).
__global__ __launch_bounds__(kBlock) void k_select_heavy(Launch L) {
  __shared__ long long s_W[HG_MAX_K];
  __shared__ int s_conn[kBlock / kWave][HG_MAX_K];
  const WorkItem wi = work_item(L, single_unit(blockIdx.x));
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k;
  for (int i = threadIdx.x; i < k; i += kBlock) s_W[i] = D.block_w[i];
  __syncthreads();
  const int wv = threadIdx.x / kWave, lane = lane_id();
  const long long idx = (long long)wi.first * (kBlock / kWave) + wv;
  if (idx >= D.heavy_count) return;
  const int sl = (int)(idx % kSlots);
  unsigned long long* my_hist = D.hist + (size_t)(blockIdx.x % D.hist_reps) * D.hist_stride;
  RoundCounters* ctr = D.ctr;
  const int u = D.heavy_list[idx];
  const int a = D.part[u];
  const unsigned char el = D.eligible[u];
  if (!el || (unsigned)a >= (unsigned)k) {
    if (lane == 0) {
      D.cand[u] = -1;
      if (el) {
        atomicOr(D.err_flags, kErrPart);
        D.eligible[u] = 0;
      }
    }
    return;
  }
  int* conn = s_conn[wv];
  for (int i = lane; i < k; i += kWave) conn[i] = 0;
  wave_lds_sync();
  const long long b0 = D.vptr[u], b1 = D.vptr[u + 1];
  const int wk = bit_words(k);
  int tot = 0, ben = 0;
  bool bnd = false;
  for (long long j = b0 + lane; j < b1; j += kWave) {
    const int e = D.vnets[j];
    const unsigned* r = D.netstate + (long long)e * D.rw;
    const int w = (int)r[0];
    tot += w;
    bnd |= r[1] > 1u;
    if ((r[2 + wk + (a >> 5)] >> (a & 31)) & 1u) ben += w;
    for (int q = 0; q < wk; ++q) {
      unsigned x = r[2 + q];
      while (x) {
        int b = __ffs(x) - 1;
        x &= x - 1;
        atomicAdd(&conn[q * 32 + b], w);
      }
    }
  }
  wave_lds_sync();
  tot = wave_sum(tot);
  ben = wave_sum(ben);
  bnd = __any(bnd);
  const long long cu = D.vwgt ? D.vwgt[u] : 1;
  // best feasible neighbouring block on this lane's share of the blocks
  int bc = -1, bi = -1;
  long long bw = 0;
  for (int i = lane; i < k; i += kWave) {
    int ci = conn[i];
    if (i == a || ci <= 0 || s_W[i] + cu > D.lmax) continue;
    long long Wi = s_W[i];
    if (bi < 0 || ci > bc || (ci == bc && (Wi < bw || (Wi == bw && i < bi)))) {
      bc = ci;
      bi = i;
      bw = Wi;
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    int oc = __shfl_xor(bc, o), oi = __shfl_xor(bi, o);
    long long ow = __shfl_xor(bw, o);
    bool take = oi >= 0 && (bi < 0 || oc > bc || (oc == bc && (ow < bw || (ow == bw && oi < bi))));
    if (take) {
      bc = oc;
      bi = oi;
      bw = ow;
    }
  }
  if (lane == 0) {
    D.eligible[u] = 0;
    atomicAdd(&ctr->slot[kCtrEligible][sl], 1ull);
    long long out = -1;
    if (bnd) {
      atomicAdd(&ctr->slot[kCtrBoundary][sl], 1ull);
      atomicAdd(&ctr->slot[kCtrActivePins][sl], (unsigned long long)(b1 - b0));
      if (bi >= 0) {
        const int g = ben - tot + bc;
        if (g > 0 || (g == 0 && bw + cu < s_W[a])) {
          out = pack_cand(g, bi);
          atomicAdd(&ctr->slot[kCtrCandidates][sl], 1ull);
          atomicAdd(&my_hist[bi * kBuckets + (g < kBuckets ? g : kBuckets - 1)],
                    (unsigned long long)cu);
          if (g > kBuckets - 1) atomicOr(&D.overflow[bi], 1);
        }
      }
    }
    D.cand[u] = out;
  }
}

// Select from a gain cache (subsection "Gain Caching"): the same decisions
// as k_select_light / k_select_heavy, read from b(u), w(I(u)) and the
// penalty row instead of the incident nets.  Block i neighbours u iff
// conn_i = w(I(u)) - p_i(u) > 0, and then g_i(u) = b(u) - w(I(u)) + conn_i.
// G lanes share a vertex, each reading 16-byte quads of its row, so one
// wavefront reads 64 / G consecutive rows.  Unit: a chunk of 256 vertices;
// every vertex, light or heavy, is handled here.
template <int G>
__global__ __launch_bounds__(kBlock) void k_select_cached(Launch L) {
  __shared__ long long s_W[HG_MAX_K];
  __shared__ unsigned long long s_hist[kLdsHistEntries];
  __shared__ unsigned long long s_sums[2];
  const InstDesc D0 = L.one;
  const WorkItem wi = work_item(L, xcd_sweep(units_of(D0.n, kBlock)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, B = D.lds_buckets, n = D.n;
  const long long lmax = D.lmax;
  for (int i = threadIdx.x; i < k * B; i += kBlock) s_hist[i] = 0;
  if (threadIdx.x < 2) s_sums[threadIdx.x] = 0;
  for (int i = threadIdx.x; i < k; i += kBlock) s_W[i] = D.block_w[i];
  __syncthreads();
  unsigned long long* my_hist = D.hist + (size_t)(blockIdx.x % D.hist_reps) * D.hist_stride;
  int n_elig = 0, n_bnd = 0, n_cand = 0, n_apins = 0;   // as in the light sweep
  const int gl = threadIdx.x % G;
  constexpr int kPer = kBlock / G;
  const int Q = cache_stride(k) / 4;
  const int* __restrict__ cb = D.cache;
  const int4* __restrict__ rows = (const int4*)(D.cache + cache_pbase(n));
  for (int it = 0; it < wi.count; ++it) {
    const long long c = (long long)wi.first + (long long)it * wi.stride;
    for (int sub = 0; sub < G; ++sub) {
      // every lane of a group has the same u, so control flow below is
      // uniform within the group
      const long long u = c * kBlock + sub * kPer + threadIdx.x / G;
      if (u >= n) continue;
      if (gl == 0 && D.moved) D.moved[u] = 0;
      const unsigned char el = D.eligible[u];
      if (!el) {
        if (gl == 0) D.cand[u] = -1;
        continue;
      }
      const int a = D.part[u];
      if ((unsigned)a >= (unsigned)k) {
        if (gl == 0) {
          atomicOr(D.err_flags, kErrPart);
          D.cand[u] = -1;
          D.eligible[u] = 0;
        }
        continue;
      }
      const int ben = cb[u], tot = cb[n + u];
      const long long cu = D.vwgt ? D.vwgt[u] : 1;
      bool bnd = false;
      int bc = -1, bi = -1;
      long long bw = 0;
      for (int q = gl; q < Q; q += G) {
        const int4 p4 = rows[u * Q + q];
        const int pv[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = q * 4 + j;
          const int ci = tot - pv[j];
          if (i >= k || i == a || ci <= 0) continue;
          bnd = true;
          const long long Wi = s_W[i];
          if (Wi + cu > lmax) continue;
          if (bi < 0 || ci > bc || (ci == bc && Wi < bw)) {
            bc = ci;
            bi = i;
            bw = Wi;
          }
        }
      }
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) {
        const int oc = __shfl_xor(bc, o, G), oi = __shfl_xor(bi, o, G);
        const long long ow = __shfl_xor(bw, o, G);
        bnd |= __shfl_xor((int)bnd, o, G) != 0;
        const bool take =
            oi >= 0 && (bi < 0 || oc > bc || (oc == bc && (ow < bw || (ow == bw && oi < bi))));
        if (take) {
          bc = oc;
          bi = oi;
          bw = ow;
        }
      }
      if (gl != 0) continue;
      D.eligible[u] = 0;
      n_elig += 1;
      long long out = -1;
      if (bnd) {
        n_bnd += 1;
        n_apins += (int)(D.vptr[u + 1] - D.vptr[u]);
        if (bi >= 0) {
          const int g = ben - tot + bc;
          if (g > 0 || (g == 0 && bw + cu < s_W[a])) {
            out = pack_cand(g, bi);
            n_cand += 1;
            if (g < B) {
              atomicAdd(&s_hist[bi * B + g], (unsigned long long)cu);
            } else {
              atomicAdd(&my_hist[bi * kBuckets + (g < kBuckets ? g : kBuckets - 1)],
                        (unsigned long long)cu);
              if (g > kBuckets - 1) atomicOr(&D.overflow[bi], 1);
            }
          }
        }
      }
      D.cand[u] = out;
    }
  }
  add_select_counts(D, s_sums, n_elig, n_bnd, n_cand, n_apins, [&] {
    for (int i = threadIdx.x; i < k * B; i += kBlock) {
      const unsigned long long v = s_hist[i];
      if (v) atomicAdd(&my_hist[(i / B) * kBuckets + (i % B)], v);
    }
  });
}

constexpr unsigned kMoversGrid = 1024;   // persistent workgroups

// b(u) of every vertex that moved this round, from the finalized net records
// (the nets where u is the only pin of its new block).  Each wavefront queues the
// moved vertices (few) of its slices and walks 64 rows at a time, four nets of
// each on their way (matrix, k = 8, per round: a thread per vertex 25 us, 12 so).
__global__ __launch_bounds__(kBlock) void k_cache_movers(Launch L) {
  __shared__ int s_q[kBlock / kWave][2 * kWave];
  const InstDesc D = L.one;
  const WorkItem run = xcd_sweep(units_of(D.n, kBlock));
  const int lane = lane_id(), wk = bit_words(D.k), rw = D.rw;
  int* my_q = s_q[threadIdx.x / kWave];
  auto wave_vertices = [&](int cnt) {
    if (lane >= cnt) return;
    const int u = my_q[lane], a = D.part[u];
    const unsigned* rec = D.netstate + 2 + wk + (a >> 5);
    const unsigned bit = 1u << (a & 31);
    const long long b0 = D.vptr[u], b1 = D.vptr[u + 1];
    int ben = 0;
    for (long long j = b0; j < b1; j += 4) {
      long long at[4];
      unsigned set[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) at[q] = (long long)D.vnets[j + q < b1 ? j + q : j] * rw;
#pragma unroll
      for (int q = 0; q < 4; ++q) set[q] = rec[at[q]];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (j + q < b1 && (set[q] & bit)) ben += D.unit_nets ? 1 : (int)D.netstate[at[q]];
    }
    D.cache[u] = ben;
  };
  int qn = 0;                                    // wave-uniform
  for (int it = 0; it <= run.count; ++it) {
    if (it < run.count) {
      const long long u = ((long long)run.first + (long long)it * run.stride) * kBlock +
                          threadIdx.x;
      const bool moved = u < D.n && D.moved[u];
      const unsigned long long mask = __ballot(moved);
      if (moved) my_q[lanes_below(mask, qn)] = (int)u;
      qn += __popcll(mask);                      // < 2 * kWave
      wave_lds_sync();
    }
    if (qn >= kWave || (it == run.count && qn > 0)) {
      const int cnt = qn < kWave ? qn : kWave;
      wave_vertices(cnt);
      const int rest = lane < qn - cnt ? my_q[kWave + lane] : 0;
      wave_lds_sync();
      my_q[lane] = rest;
      qn -= cnt;
      wave_lds_sync();
    }
  }
}

int cached_group(int k) {
  const int q = cache_stride(k) / 4;
  int G = 1;
  while (G < q && G < kWave) G <<= 1;
  return G;
}

SelectKernel select_cached_kernel(int k) {
  switch (cached_group(k)) {
    case 1: return k_select_cached<1>;
    case 2: return k_select_cached<2>;
    case 4: return k_select_cached<4>;
    case 8: return k_select_cached<8>;
    case 16: return k_select_cached<16>;
    case 32: return k_select_cached<32>;
    default: return k_select_cached<64>;
  }
}

// A single-instance round that reads and updates the gain cache d.cache:
// cached select in place of the light and heavy sweeps, the finalize that
// applies the net deltas, and the movers' b before the round record.
void cached_round_plan(const InstDesc& d, RoundPlan& plan) {
  single_round_plan(d, plan);
  plan.select[0].kernel = (void*)select_cached_kernel(d.k);
  plan.heavy.clear();   // any_heavy stays: heavy vertices can still overflow the buckets
}

hipError_t launch_cached_round(const RoundPlan& plan, int round, hipStream_t s,
                               hipEvent_t* marks) {
  hipError_t e = launch_round_front(plan, s, marks);
  if (e == hipSuccess) e = launch_round_finalize(plan, s, marks);
  if (e != hipSuccess) return e;
  const InstDesc& d = plan.stats.L.one;
  const unsigned chunks = (unsigned)units_of(d.n, kBlock);
  hipLaunchKernelGGL(k_cache_movers, dim3(chunks < kMoversGrid ? chunks : kMoversGrid),
                     dim3(kBlock), 0, s, plan.stats.L);
  return launch_round_stats(plan, round, s, marks);
}

// Block weights and round record (one workgroup each).  Fold the apply's
// block-weight slots into block_w; returns the heaviest of this thread's blocks.
template <int A>
__device__ __forceinline__ long long fold_block_weights(const InstDesc& D) {
  long long mx = LLONG_MIN;
  // slot cells A at a time are requested before the stores that clear them (not
  // one round trip per cell)
  for (int i = threadIdx.x; i < D.k; i += kBlock) {
    long long* col = D.bw_slots + i;
    const size_t ks = (size_t)D.k;
    long long d = D.block_w[i];
    for (int s0 = 0; s0 < kSlots; s0 += A) {
      long long cells[A];
#pragma unroll
      for (int q = 0; q < A; ++q) cells[q] = col[(s0 + q) * ks];
#pragma unroll
      for (int q = 0; q < A; ++q) d += cells[q];
#pragma unroll
      for (int q = 0; q < A; ++q) col[(s0 + q) * ks] = 0;
    }
    D.block_w[i] = d;
    mx = d > mx ? d : mx;
  }
  return mx;
}

// The largest of the workgroup's values, in two halves around a barrier.
__device__ __forceinline__ void block_max64_put(long long v, long long* s_max /*[kBlock/kWave]*/) {
  v = wave_max(v);
  if (lane_id() == 0) s_max[threadIdx.x / kWave] = v;
}
__device__ __forceinline__ long long block_max64_get(const long long* s_max) {   // after a barrier
  long long m = s_max[0];
  for (int i = 1; i < kBlock / kWave; ++i) m = s_max[i] > m ? s_max[i] : m;
  return m;
}

// A workgroup's view of the counter slots: wavefront w holds rows w, w + 4, ...
constexpr int kCounterRows = (kNumCounters + kBlock / kWave - 1) / (kBlock / kWave);
struct CounterRows {
  unsigned long long v[kCounterRows];
  __device__ __forceinline__ void load(const RoundCounters* ctr) {
#pragma unroll
    for (int r = 0; r < kCounterRows; ++r) {
      const int c = (int)threadIdx.x / kWave + r * (kBlock / kWave);
      v[r] = c < kNumCounters ? ctr->slot[c][lane_id()] : 0ull;
    }
  }
};

// Sum the counter slots, write the round record, move km1 by the attributed
// drop, reset the counters.  `mx`: the heaviest of the thread's blocks.
__device__ __forceinline__ void write_record(const InstDesc& D, RoundCounters* ctr,
                                             const CounterRows& rows, long long mx,
                                             hg_round_stats* out) {
  __shared__ long long s_sum[kNumCounters];
  __shared__ long long s_max[kBlock / kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
#pragma unroll
  for (int r = 0; r < kCounterRows; ++r) {
    const int c = wv + r * (kBlock / kWave);
    if (c < kNumCounters) {
      const long long sum = wave_sum((long long)rows.v[r]);
      if (lane == 0) s_sum[c] = sum;
      ctr->slot[c][lane] = 0;
    }
  }
  block_max64_put(mx, s_max);
  __syncthreads();
  if (threadIdx.x == 0) {
    hg_round_stats st;
    st.eligible = s_sum[kCtrEligible];
    st.boundary = s_sum[kCtrBoundary];
    st.candidates = s_sum[kCtrCandidates];
    st.approved = s_sum[kCtrApproved];
    st.moved_pins = s_sum[kCtrMovedPins];
    st.touched_nets = s_sum[kCtrTouched];
    st.km1_delta = s_sum[kCtrDeltaAttr];
    st.km1_delta_recomputed = s_sum[kCtrDeltaCheck];
    st.active_pins = s_sum[kCtrActivePins];
    st.touched_pins = s_sum[kCtrTouchedPins];
    st.km1_after = *D.km1 - st.km1_delta;
    st.max_block_weight = block_max64_get(s_max);
    *D.km1 = st.km1_after;
    *out = st;
    ctr->any_overflow = 0;
  }
}

// Late rounds: the last workgroup of the thresholds (or of the brief rounds' tile
// sums) writes the record of the round before.  (A launch of its own for five
// microseconds of work each round: n = 10,000 k = 2, five rounds, 154 us per call,
// 138 so; matrix, ten rounds, k = 8 1434 -> 1382, k = 64 2025 -> 1984; netlist step
// 4376 -> 4320.)
__device__ __forceinline__ bool records_previous(const InstDesc& D) {
  if (!D.prev || blockIdx.x + 1 != gridDim.x) return false;
  CounterRows rows;
  rows.load(D.prev);
  write_record(D, D.prev, rows, D.prev->max_block_w, D.stats - 1);
  return true;
}

// --------------------------------------------------------------- threshold

// Unit: one target block t.  Thread j looks at gain bucket 255 - j (summed
// over the XCD replicas, which it also clears for the next round).
__global__ __launch_bounds__(kBlock) void k_threshold(Launch L) {
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ int s_first;
  const WorkItem wi = work_item(L, single_unit(blockIdx.x));
  const InstDesc D = inst_desc(L, wi.inst);
  if (records_previous(D)) return;
  const int t = wi.first;
  const int bucket = kBuckets - 1 - threadIdx.x;
  long long h = 0;
  unsigned long long* col = D.hist + (size_t)t * kBuckets + bucket;
  unsigned long long rv[kHistReplicas];
  // all replicas' cells requested before the stores that clear them
#pragma unroll
  for (int rep = 0; rep < kHistReplicas; ++rep)
    rv[rep] = rep < D.hist_reps ? col[(size_t)rep * D.hist_stride] : 0ull;
#pragma unroll
  for (int rep = 0; rep < kHistReplicas; ++rep) {
    h += (long long)rv[rep];
    if (rep < D.hist_reps) col[(size_t)rep * D.hist_stride] = 0;
  }
  const long long budget = D.lmax - D.block_w[t];
  if (threadIdx.x == 0) s_first = kBlock;
  long long total;
  const long long above = block_excl_scan64(h, s_tmp, &total);   // weight of higher gains
  if (h > 0 && above + h > budget) atomicMin(&s_first, (int)threadIdx.x);
  __syncthreads();
  const int f = s_first;
  if ((int)threadIdx.x == (f < kBlock ? f : 0)) {
    Threshold r;
    r.tau = 0;
    r.rem_tile = 0;
    if (f < kBlock) {
      r.gstar = bucket;
      r.rem = budget - above;
    } else {
      r.gstar = -1;
      r.rem = 0;
    }
    D.thr[t] = r;
    if (f < kBlock && bucket == kBuckets - 1 && D.overflow[t]) {
      atomicOr(&D.ctr->any_overflow, 1u);
    } else {
      D.overflow[t] = 0;
    }
  }
}

// Only for graphs with heavy vertices: the ">= 255" bucket of block t holds
// several gain values and its budget ran out inside it.  Find the exact
// threshold gain by bisection over all candidates (a slow but rare path).
// Unit: one target block.
__global__ __launch_bounds__(kBlock) void k_overflow_resolve(Launch L) {
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ long long s_max[kBlock / kWave];
  const WorkItem wi = work_item(L, single_unit(blockIdx.x));
  const InstDesc D = inst_desc(L, wi.inst);
  const int t = wi.first;
  if (!D.ctr->any_overflow) return;
  if (!D.overflow[t]) return;
  const long long rem = D.thr[t].rem;
  const int n = D.n;
  const long long* cand = D.cand;
  long long gmax = 0;
  for (long long u = threadIdx.x; u < n; u += kBlock) {
    long long x = cand[u];
    if (x >= 0 && cand_target(x) == t && cand_gain(x) > gmax) gmax = cand_gain(x);
  }
  {
    long long v = wave_max(gmax);
    if (lane_id() == 0) s_max[threadIdx.x / kWave] = v;
    __syncthreads();
    gmax = 0;
    for (int i = 0; i < kBlock / kWave; ++i) gmax = s_max[i] > gmax ? s_max[i] : gmax;
    __syncthreads();
  }
  long long lo = kBuckets - 1, hi = gmax + 1, w_hi = 0;   // weight(>= lo) > rem >= weight(>= hi)
  while (hi - lo > 1) {
    long long mid = (lo + hi) / 2;
    long long s = 0;
    for (long long u = threadIdx.x; u < n; u += kBlock) {
      long long x = cand[u];
      if (x >= 0 && cand_target(x) == t && cand_gain(x) >= mid) s += D.vwgt ? D.vwgt[u] : 1;
    }
    s = block_sum64(s, s_tmp);
    if (s > rem) {
      lo = mid;
    } else {
      hi = mid;
      w_hi = s;
    }
  }
  if (threadIdx.x == 0) {
    D.thr[t].gstar = (int)lo;
    D.thr[t].rem = rem - w_hi;
    D.overflow[t] = 0;
  }
}

// --------------------------------------------------------------- tiles

// Brief rounds: gstar of every block into s_g, and with `publish` into D.thr for
// the approve.  A wavefront per block, lane i its buckets 255 - 4 i and the three
// below.
__device__ __forceinline__ void brief_thresholds(const InstDesc& D, int* s_g, bool publish) {
  constexpr int kAhead = 4, kWaves = kBlock / kWave;
  const int lane = lane_id(), k = D.k;
  for (int t0 = threadIdx.x / kWave; t0 < k; t0 += kAhead * kWaves) {
    ulonglong2 lo[kAhead], hi[kAhead];
    long long bw[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int t = t0 + q * kWaves;
      lo[q] = hi[q] = ulonglong2{0, 0};
      bw[q] = 0;
      if (t < k) {
        const ulonglong2* col = reinterpret_cast<const ulonglong2*>(
            D.hist + (size_t)t * kBuckets + (kBuckets - 4) - 4 * lane);
        lo[q] = col[0];
        hi[q] = col[1];
        bw[q] = D.block_w[t];
      }
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int t = t0 + q * kWaves;
      if (t >= k) break;
      const long long h[4] = {(long long)hi[q].y, (long long)hi[q].x, (long long)lo[q].y,
                              (long long)lo[q].x};
      const long long mine = h[0] + h[1] + h[2] + h[3];
      const long long budget = D.lmax - bw[q];
      long long above = wave_incl_scan64(mine) - mine;        // weight of higher gains
      int at = -1;
      long long rem = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (at < 0 && h[x] > 0 && above + h[x] > budget) {
          at = kBuckets - 1 - 4 * lane - x;
          rem = budget - above;
        }
        above += h[x];
      }
      const unsigned long long hits = __ballot(at >= 0);
      const int first = hits ? __ffsll((long long)hits) - 1 : 0;
      if (lane == first) {
        s_g[t] = at;
        if (publish) D.thr[t] = Threshold{at, D.num_tiles, rem, 0};
      }
    }
  }
}

// Brief rounds: gstar of every block, the tile where each block that is cut runs
// out of budget, and what is left of it there, from the tile sums (as
// k_tilescan).  A wavefront per block, lane i tiles 4 i .. 4 i + 3.
__device__ __forceinline__ void brief_tiles(const InstDesc& D, int* s_g, int* s_tau,
                                            long long* s_remt) {
  constexpr int kAhead = 4, kWaves = kBlock / kWave;
  static_assert(kBriefTiles == 4 * kWave, "four tiles a lane");
  const int lane = lane_id(), k = D.k, num_tiles = D.num_tiles;
  for (int t0 = threadIdx.x / kWave; t0 < k; t0 += kAhead * kWaves) {
    long long v[kAhead][4], rem[kAhead];
    int g[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int t = t0 + q * kWaves;
      const bool in = t < k;
      g[q] = in ? D.thr[t].gstar : -1;
      rem[q] = in ? D.thr[t].rem : 0;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        v[q][x] = in && 4 * lane + x < num_tiles
                      ? D.tilesum[(long long)t * num_tiles + 4 * lane + x]
                      : 0;
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int t = t0 + q * kWaves;
      if (t >= k) break;
      const long long mine = v[q][0] + v[q][1] + v[q][2] + v[q][3];
      long long run = wave_incl_scan64(mine) - mine;
      int at = num_tiles;
      long long left = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (at == num_tiles && v[q][x] > 0 && run + v[q][x] > rem[q]) {
          at = 4 * lane + x;
          left = rem[q] - run;
        }
        run += v[q][x];
      }
      // (a block that is not cut has no tile sums: nothing has its gain -1)
      const unsigned long long hits = __ballot(at < num_tiles);
      const int first = hits ? __ffsll((long long)hits) - 1 : 0;
      if (lane == first) {
        s_g[t] = g[q];
        s_tau[t] = at;
        s_remt[t] = left;
      }
    }
  }
}

// Unit: one tile of kTile vertices.  BRIEF: a brief round (RoundPlan::brief).
template <bool BRIEF>
__global__ __launch_bounds__(kBlock) void k_tilesum(Launch L) {
  __shared__ unsigned long long s_sum[HG_MAX_K];
  __shared__ int s_g[HG_MAX_K];
  const WorkItem wi = work_item(L, single_unit(blockIdx.x));
  const InstDesc D = inst_desc(L, wi.inst);
  if constexpr (BRIEF) {
    if (records_previous(D)) return;
  }
  const int k = D.k;
  const int tile = wi.first;
  const long long base = (long long)tile * kTile;
  // every candidate word and weight of this thread requested before the first wait
  long long x[kPerThreadTile];
  int cw[kPerThreadTile];
#pragma unroll
  for (int j = 0; j < kPerThreadTile; ++j) {
    const long long u = base + (long long)j * kBlock + threadIdx.x;
    x[j] = u < D.n ? D.cand[u] : -1;
    cw[j] = u < D.n && D.vwgt ? D.vwgt[u] : 1;
  }
  if constexpr (BRIEF) brief_thresholds(D, s_g, tile == 0);
  for (int i = threadIdx.x; i < k; i += kBlock) {
    s_sum[i] = 0;
    if constexpr (!BRIEF) s_g[i] = D.thr[i].gstar;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPerThreadTile; ++j) {
    if (x[j] >= 0) {
      const int t = cand_target(x[j]);
      if (cand_gain(x[j]) == s_g[t]) atomicAdd(&s_sum[t], (unsigned long long)cw[j]);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < k; i += kBlock)
    D.tilesum[(long long)i * D.num_tiles + tile] = (long long)s_sum[i];
}

// Unit: one target block.  Thread i takes kScanPerThread consecutive tiles
// of each span of kBlock * kScanPerThread tiles (one span covers 2048 tiles,
// about a million vertices): one workgroup scan per span.
constexpr int kScanPerThread = 8;

__global__ __launch_bounds__(kBlock) void k_tilescan(Launch L) {
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ int s_tau;
  __shared__ long long s_remt;
  const WorkItem wi = work_item(L, single_unit(blockIdx.x));
  const InstDesc D = inst_desc(L, wi.inst);
  const int t = wi.first;
  const int num_tiles = D.num_tiles;
  const Threshold r = D.thr[t];
  if (r.gstar < 0) {
    if (threadIdx.x == 0) D.thr[t].tau = num_tiles;
    return;
  }
  if (threadIdx.x == 0) {
    s_tau = num_tiles;
    s_remt = 0;
  }
  const long long* row = D.tilesum + (long long)t * num_tiles;
  long long carry = 0;
  for (int base = 0; base < num_tiles; base += kBlock * kScanPerThread) {
    const int first = base + threadIdx.x * kScanPerThread;
    long long v[kScanPerThread];
    long long mine = 0;
#pragma unroll
    for (int q = 0; q < kScanPerThread; ++q) {
      v[q] = first + q < num_tiles ? row[first + q] : 0;
      mine += v[q];
    }
    long long tot;
    long long run = carry + block_excl_scan64(mine, s_tmp, &tot);
    // this thread's first tile whose gain-g* weight overflows the budget,
    // and the weight before it
    int hit = -1;
    long long hit_before = 0;
#pragma unroll
    for (int q = 0; q < kScanPerThread; ++q) {
      if (hit < 0 && v[q] > 0 && run + v[q] > r.rem) {
        hit = first + q;
        hit_before = run;
      }
      run += v[q];
    }
    if (hit >= 0) atomicMin(&s_tau, hit);
    __syncthreads();
    const int f = s_tau;
    if (f < num_tiles) {
      if (hit == f) s_remt = r.rem - hit_before;   // budget left at tile f's start
      break;
    }
    carry += tot;
    __syncthreads();
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    D.thr[t].tau = s_tau;
    D.thr[t].rem_tile = s_remt;
  }
}

// --------------------------------------------------------------- approve + apply

// Apply the moves held in s_list[0..count) (vertex ids; targets in s_tgt):
// part, moved flags and block-weight deltas per mover, then the movers'
// incident nets as one flattened range split over all 256 threads (so a tile
// with few movers still keeps four wavefronts busy, and a high-degree mover is
// spread over the workgroup): every incident net gets its touched flag (a plain
// byte store: all writers store the same value).  Phi is left to the finalize,
// which counts the touched nets' pins anew: it visits those pins anyway to make
// them eligible, where two atomics per mover and net, 20 G a second for the
// whole GPU, were two thirds of this kernel's time.
// The mover owning flattened incidence j: the largest i < count with
// s_off[i] <= j.
__device__ __forceinline__ int list_owner(const int* s_off, int count, long long j) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_off[mid] <= j) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ void apply_list(const InstDesc& D, const int* s_list, const int* s_tgt, int count,
                           long long* s_beg, int* s_off, long long* s_tmp,
                           unsigned long long* s_dW, long long& moved_pins,
                           long long& approved) {
  // per mover: move it, record where its incident nets start
  long long my_len = 0;
  int lens[kPerThreadTile];
  const int first = threadIdx.x * kPerThreadTile;   // entries [first, first + kPerThreadTile)
#pragma unroll
  for (int q = 0; q < kPerThreadTile; ++q) {
    const int i = first + q;
    lens[q] = 0;
    if (i < count) {
      const int u = s_list[i], t = s_tgt[i];
      const int a = D.part[u];
      const long long b = D.vptr[u];
      const int len = (int)(D.vptr[u + 1] - b);
      const long long cu = D.vwgt ? D.vwgt[u] : 1;
      D.part[u] = t;
      if (D.kept) move_packed(D, u, a, t);
      if (D.moved) D.moved[u] = 1;
      atomicAdd(&s_dW[t], (unsigned long long)cu);
      atomicAdd(&s_dW[a], (unsigned long long)(-cu));
      s_beg[i] = b;
      lens[q] = len;
      my_len += len;
      moved_pins += len;
      approved += 1;
    }
  }
  long long total;
  long long off = block_excl_scan64(my_len, s_tmp, &total);
#pragma unroll
  for (int q = 0; q < kPerThreadTile; ++q) {
    if (first + q < count) s_off[first + q] = (int)off;
    off += lens[q];
  }
  __syncthreads();
  for (long long j = threadIdx.x; j < total; j += kBlock) {
    const int lo = list_owner(s_off, count, j);
    D.touched[D.vnets[s_beg[lo] + (j - s_off[lo])]] = 1;
  }
}

// Monotone rounds: mark the approved moves, and set the cells (e, source) and
// (e, target) of their incident nets empty for the exact-gain kernels that
// follow (out_max 0, in_min "none", out_cnt 0); the incidences are spread
// over the workgroup as in apply_list.
__device__ void mark_list(const InstDesc& D, const int* s_list, const int* s_tgt, int count,
                          int* s_from, long long* s_beg, int* s_off, long long* s_tmp) {
  long long my_len = 0;
  int lens[kPerThreadTile];
  const int first = threadIdx.x * kPerThreadTile;
#pragma unroll
  for (int q = 0; q < kPerThreadTile; ++q) {
    const int i = first + q;
    lens[q] = 0;
    if (i < count) {
      const int u = s_list[i];
      const long long b = D.vptr[u];
      D.appr[u] = 1;
      s_from[i] = D.part[u];
      s_beg[i] = b;
      lens[q] = (int)(D.vptr[u + 1] - b);
      my_len += lens[q];
    }
  }
  long long total;
  long long off = block_excl_scan64(my_len, s_tmp, &total);
#pragma unroll
  for (int q = 0; q < kPerThreadTile; ++q) {
    if (first + q < count) s_off[first + q] = (int)off;
    off += lens[q];
  }
  __syncthreads();
  const int k = D.k;
  const int4 empty = make_int4(0, 0x7fffffff, 0, 0);
  for (long long j = threadIdx.x; j < total; j += kBlock) {
    const int lo = list_owner(s_off, count, j);
    const long long e = D.vnets[s_beg[lo] + (j - s_off[lo])];
    D.seq_cell[e * k + s_from[lo]] = empty;
    D.seq_cell[e * k + s_tgt[lo]] = empty;
  }
}

// Unit: a tile of kTile vertices (count = 1), or -- boundary workgroups --
// the tile of target block `first` where its budget runs out (count = -1).
// Single instance: workgroups [0, num_tiles) are tiles (XCD-remapped), the
// k after them the boundary workgroups.  BRIEF: a brief round.
template <bool BRIEF>
__global__ __launch_bounds__(kBlock) void k_approve_apply(Launch L) {
  __shared__ int s_list[kTile];
  __shared__ int s_tgt[kTile];
  __shared__ int s_from[kTile];
  __shared__ int s_off[kTile];
  __shared__ long long s_beg[kTile];
  __shared__ int s_g[HG_MAX_K];
  __shared__ int s_tau[HG_MAX_K];
  __shared__ long long s_remt[BRIEF ? kBriefMaxK : 1];
  __shared__ unsigned long long s_dW[HG_MAX_K];
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ unsigned s_count;
  WorkItem fb;
  {
    const int nt = L.one.num_tiles;
    fb = (int)blockIdx.x < nt ? single_unit((int)xcd_remap(blockIdx.x, nt))
                              : single_unit((int)blockIdx.x - nt);
    if ((int)blockIdx.x >= nt) fb.count = -1;
  }
  const WorkItem wi = work_item(L, fb);
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, n = D.n, num_tiles = D.num_tiles;
  const long long* __restrict__ cand = D.cand;
  const int tile = wi.first;        // (count >= 0)
  long long xs[kPerThreadTile];     // requested before the first wait
  if (wi.count >= 0) {
#pragma unroll
    for (int j = 0; j < kPerThreadTile; ++j) {
      const long long u = (long long)tile * kTile + (long long)j * kBlock + threadIdx.x;
      xs[j] = u < n ? cand[u] : -1;
    }
  }
  if constexpr (BRIEF) {
    brief_tiles(D, s_g, s_tau, s_remt);
    if (wi.count < 0)               // for the next round
      D.hist[(size_t)wi.first * kBuckets + threadIdx.x] = 0;
  }
  for (int i = threadIdx.x; i < k; i += kBlock) {
    if constexpr (!BRIEF) {
      s_g[i] = D.thr[i].gstar;
      s_tau[i] = D.thr[i].tau;
    }
    s_dW[i] = 0;
  }
  if (threadIdx.x == 0) s_count = 0;
  __syncthreads();
  if (wi.count >= 0) {
    const long long base = (long long)tile * kTile;
#pragma unroll
    for (int j = 0; j < kPerThreadTile; ++j) {
      const long long u = base + (long long)j * kBlock + threadIdx.x;
      bool ok = false;
      int t = 0;
      const long long x = xs[j];
      if (x >= 0) {
        t = cand_target(x);
        const int g = cand_gain(x), gs = s_g[t];
        ok = g > gs || (g == gs && tile < s_tau[t]);
      }
      const int slot = wave_append(&s_count, ok);   // LDS counter, one atomic per wave
      if (ok) {
        s_list[slot] = (int)u;
        s_tgt[slot] = t;
      }
    }
  } else {
    // the tile where block t's budget runs out: prefix sums in vertex order
    const int t = wi.first;
    Threshold r = D.thr[t];
    if constexpr (BRIEF) {
      r.tau = s_tau[t];
      r.rem_tile = s_remt[t];
    }
    if (r.gstar < 0 || r.tau >= num_tiles) return;   // whole workgroup leaves together
    const long long base = (long long)r.tau * kTile + (long long)threadIdx.x * kPerThreadTile;
    long long mine = 0;
    for (int j = 0; j < kPerThreadTile; ++j) {
      const long long u = base + j;
      if (u < n) {
        const long long x = cand[u];
        if (x >= 0 && cand_target(x) == t && cand_gain(x) == r.gstar)
          mine += D.vwgt ? D.vwgt[u] : 1;
      }
    }
    long long tot;
    long long run = block_excl_scan64(mine, s_tmp, &tot);
    for (int j = 0; j < kPerThreadTile; ++j) {
      const long long u = base + j;
      bool ok = false;
      if (u < n) {
        const long long x = cand[u];
        if (x >= 0 && cand_target(x) == t && cand_gain(x) == r.gstar) {
          const long long cu = D.vwgt ? D.vwgt[u] : 1;
          ok = run + cu <= r.rem_tile;
          run += cu;
        }
      }
      const int slot = wave_append(&s_count, ok);
      if (ok) {
        s_list[slot] = (int)u;
        s_tgt[slot] = t;
      }
    }
  }
  __syncthreads();
  const int count = (int)s_count;
  long long moved_pins = 0, approved = 0;
  if (count > 0 && D.appr) {
    // monotone round: only mark; the moves are ordered, re-gained and cut later
    mark_list(D, s_list, s_tgt, count, s_from, s_beg, s_off, s_tmp);
    if (threadIdx.x == 0)
      atomicAdd(&D.ctr->slot[kCtrMarked][blockIdx.x % kSlots], (unsigned long long)count);
  } else if (count > 0) {
    apply_list(D, s_list, s_tgt, count, s_beg, s_off, s_tmp, s_dW, moved_pins, approved);
  }
  __syncthreads();
  // block-weight deltas go to one of kSlots partial rows (a single row
  // would serialize one atomic per tile on each of the k addresses); the
  // round record folds them into block_w
  long long* my_dw = D.bw_slots + (size_t)(blockIdx.x % kSlots) * k;
  for (int i = threadIdx.x; i < k; i += kBlock)
    if (s_dW[i]) atomicAdd((unsigned long long*)&my_dw[i], s_dW[i]);
  // both below 2^31: one sum
  const long long both = block_sum64(moved_pins | (approved << 32), s_tmp);
  moved_pins = both & 0xffffffffLL;
  approved = both >> 32;
  if (threadIdx.x == 0) {
    const int sl = blockIdx.x % kSlots;
    RoundCounters* ctr = D.ctr;
    if (moved_pins) atomicAdd(&ctr->slot[kCtrMovedPins][sl], (unsigned long long)moved_pins);
    if (approved) atomicAdd(&ctr->slot[kCtrApproved][sl], (unsigned long long)approved);
  }
}

// --------------------------------------------------------------- finalize

// Unit: a block of kFinalChunk (256) nets, a quarter of it per wavefront.  The
// wavefronts work on their own (no barrier): each reads its quarter's touched
// flags, queues the touched nets in LDS and takes them as many at a time as it
// can count (64, or 32 for k > 128): their pins are made
// eligible and counted by block (count_batch), every lane rewrites the record of
// its net.  The record's old Lambda gives the attributed km1 change, w(e) for
// every block that left it and -w(e) for every one that entered; the drop
// (lambda_old - lambda_new) * w(e) checks it.  Because everything is counted from
// the final partition, nothing depends on the order of the moves (the paper
// needs a spin-lock per net for this).
// What bounds it is the chain flags -> offsets, records -> pins -> blocks and the
// scattered eligible stores.  Counting anew costs more here than rereading Phi
// rows that the approve had updated by atomics, but less than those atomics
// (approve + finalize per round, us: netlist 66 + 63 -> 23 + 82, matrix k = 8
// 41 + 39 -> 14 + 52, k = 64 49 + 61 -> 13 + 68, 64 small hypergraphs 50 + 127
// -> 22 + 87; with the gain cache, which then needs no second variant of the
// walk, 41 + 147 -> 14 + 104).  Blocks from part8 instead of part: matrix k = 8
// 71 -> 54, k = 64 86 -> 73.  A wavefront's life is a few such chains, so small
// units in many resident workgroups even them out (1024 nets, 2048 workgroups:
// netlist 96, k = 8 54, k = 64 74, weighted 12.0 against 8.7).
// Single instance: contiguous XCD-aware runs of blocks.
constexpr int kFinalQueue = 2 * kWave;   // touched nets waiting

// Gain-cache deltas of a batch of nets (subsection "Gain Caching"): the four
// update rules, summed over all moves of the round, for every pin of a net
// (pin_deltas).  Moved vertices get b recomputed after the round.  Only nets
// whose sets changed are walked: `nets` of them, lane i < nets holding pins
// [b, b + len), their changes in the LDS words `chg`, [word][count_nets]: changed
// and old Lambda, changed and new S, w(e), b, len.
constexpr __host__ __device__ int cache_nets(int wk) { return wk == 8 ? 32 : kWave; }
constexpr __host__ __device__ int cache_words(int wk) { return (4 * wk + 3) * cache_nets(wk); }

template <int WK>
__device__ __forceinline__ void cache_deltas(const InstDesc& D, const CountLds& M,
                                             const unsigned* chg, long long b, int len) {
  constexpr int CN = cache_nets(WK);
  int v[kCountFlight];
  for_pins<false>(
      D.pins, M, b, len,
      [&](const int (&pins)[kCountFlight]) {
#pragma unroll
        for (int q = 0; q < kCountFlight; ++q) v[q] = pins[q];
      },
      [&](int net, int q) {
        if (v[q] >= 0)
          pin_deltas<WK>(D, v[q], (int)chg[4 * WK * CN + net],
                         [&](int x) { return chg[x * CN + net]; });
      });
}

template <int WK, bool CACHE>
__global__ __launch_bounds__(kBlock, !CACHE && WK <= 2 ? 8 : 4) void k_finalize(Launch L) {
  extern __shared__ unsigned s_final[];   // per wavefront: count_words, the queue, cache_words
  __shared__ unsigned long long s_sums[3];
  // late rounds: one workgroup more, for the block weights
  // (refine calls have no gain cache)
  if constexpr (!CACHE) {
    if (!L.items && L.one.late && blockIdx.x + 1 == gridDim.x) {
      __shared__ long long s_max[kBlock / kWave];
      block_max64_put(fold_block_weights<8>(L.one), s_max);   // (16: spills)
      __syncthreads();
      if (threadIdx.x == 0) L.one.ctr->max_block_w = block_max64_get(s_max);
      return;
    }
  }
  const WorkItem wi = work_item(L, xcd_block(units_of(L.one.m, kFinalChunk),
                                             gridDim.x - (!CACHE && L.one.late ? 1 : 0)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  if (threadIdx.x < 3) s_sums[threadIdx.x] = 0;
  __syncthreads();
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int k = D.k, NW = count_nets(k);
  const int words = count_words(k, NW) + kFinalQueue + (CACHE ? cache_words(WK) : 0);
  const CountLds M = count_lds(s_final + (size_t)wv * words, k, NW);
  int* queue = reinterpret_cast<int*>(s_final + (size_t)wv * words + count_words(k, NW));
  unsigned* chg = reinterpret_cast<unsigned*>(queue + kFinalQueue);
  const Blocks block = blocks_of(D, D.kept != 0);
  const bool vec_phi = aligned_rows(D);
  long long attr = 0, drop = 0;
  int ntouched = 0, tpins = 0;               // nets and pins: below 2^31
  auto batch = [&](const int* q, int cnt) {
    int len = 0, w = 0, lambda = 0;
    bool mine = lane < cnt;
    long long e = 0, b = 0;
    unsigned lam[WK], one[WK];
#pragma unroll
    for (int x = 0; x < WK; ++x) lam[x] = one[x] = 0;
    if (lane < cnt) {
      e = q[lane];
      b = global_ptr(D.eptr)[e];
      len = (int)(global_ptr(D.eptr)[e + 1] - b);
      read_record<WK>(D, e, w, lambda, lam, one);
      mine = len <= kWaveNet;
      if (mine) global_out(D.touched)[e] = 0;   // the others: k_long_nets
    }
    NetSets<WK> N;
    count_batch<WK, false>(D, M, e, b, len, vec_phi, block, EligiblePins{D.eligible}, N);
    bool changed = false;
    if (mine) {
      write_record<WK, false>(D, e, w, N.lambda, N.lam, N.one);
      int left = 0;
#pragma unroll
      for (int x = 0; x < WK; ++x) {
        left += __popc(lam[x] & ~N.lam[x]) - __popc(N.lam[x] & ~lam[x]);
        changed |= lam[x] != N.lam[x] || one[x] != N.one[x];
      }
      attr += (long long)left * w;
      drop += (long long)(lambda - N.lambda) * w;
      ntouched += 1;
      tpins += len;
    }
    if constexpr (CACHE) {
      // the changed nets to the first lanes
      constexpr int CN = cache_nets(WK);
      const unsigned long long mask = __ballot(changed);
      const int at = lanes_below(mask, 0), nets = __popcll(mask);
      if (changed) {
#pragma unroll
        for (int x = 0; x < WK; ++x) {
          chg[x * CN + at] = lam[x] ^ N.lam[x];
          chg[(WK + x) * CN + at] = lam[x];
          chg[(2 * WK + x) * CN + at] = one[x] ^ N.one[x];
          chg[(3 * WK + x) * CN + at] = N.one[x];
        }
        chg[4 * WK * CN + at] = (unsigned)w;
        chg[(4 * WK + 1) * CN + at] = (unsigned)b;      // pin positions are below 2^31
        chg[(4 * WK + 2) * CN + at] = (unsigned)len;
      }
      wave_lds_sync();
      const long long cb = lane < nets ? (long long)chg[(4 * WK + 1) * CN + lane] : 0;
      const int cl = lane < nets ? (int)chg[(4 * WK + 2) * CN + lane] : 0;
      cache_deltas<WK>(D, M, chg, cb, cl);
      wave_lds_sync();
    }
  };
  // the next block's flags are loaded while this block is finalized (flags past
  // m are zero up to a whole block)
  auto flag_at = [&](int it) {
    const long long c = (long long)wi.first + (long long)it * wi.stride;
    return it < wi.count ? global_ptr(D.touched)[c * kFinalChunk + threadIdx.x] : (unsigned char)0;
  };
  unsigned char next = flag_at(0);
  int qn = 0;                                              // nets queued (wave-uniform)
  // one call site of batch: the extra last iteration empties the queue
  for (int it = 0; it <= wi.count; ++it) {
    if (it < wi.count) {
      const bool mine = next != 0;
      next = flag_at(it + 1);
      const unsigned long long mask = __ballot(mine);
      if (mine)
        queue[lanes_below(mask, qn)] =
            (int)(((long long)wi.first + (long long)it * wi.stride) * kFinalChunk) + threadIdx.x;
      qn += __popcll(mask);
      wave_lds_sync();
    }
    while (qn >= NW || (it == wi.count && qn > 0)) {
      const int cnt = qn < NW ? qn : NW;
      batch(queue + (qn - cnt), cnt);                      // the last ones: nothing moves
      qn -= cnt;
    }
  }
  const long long np = wave_sum((long long)ntouched | ((long long)tpins << 32));
  attr = wave_sum(attr);
  drop = wave_sum(drop);
  if (lane == 0) {
    atomicAdd(&s_sums[0], (unsigned long long)np);
    atomicAdd(&s_sums[1], (unsigned long long)attr);
    atomicAdd(&s_sums[2], (unsigned long long)drop);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int sl = blockIdx.x % kSlots;
    const unsigned long long nt = s_sums[0] & 0xffffffffu, tp = s_sums[0] >> 32;
    if (s_sums[1]) atomicAdd(&D.ctr->slot[kCtrDeltaAttr][sl], s_sums[1]);
    if (s_sums[2]) atomicAdd(&D.ctr->slot[kCtrDeltaCheck][sl], s_sums[2]);
    if (nt) atomicAdd(&D.ctr->slot[kCtrTouched][sl], nt);
    if (tp) atomicAdd(&D.ctr->slot[kCtrTouchedPins][sl], tp);
  }
}

// Unit: one instance.  Late rounds: the finalize has folded the block weights.
__global__ __launch_bounds__(kBlock) void k_round_stats(Launch L) {
  const WorkItem wi = work_item(L, single_unit(0));
  const InstDesc D = inst_desc(L, wi.inst);
  CounterRows rows;              // on their way before the fold waits
  rows.load(D.ctr);
  const long long mx = D.late ? D.ctr->max_block_w : fold_block_weights<16>(D);
  write_record(D, D.ctr, rows, mx, D.stats + (L.round - D.round_base));
}

// --------------------------------------------------------------- launch

// Kernel selection per instance shape (shared with the batch planner).
// Entries in flight per vertex: eight where the average degree is 12 or more
// and an entry is at most two words (half the dependent load steps for the
// typical vertex: netlist 162 -> 148 us), four elsewhere (eight would mostly
// load padding slots: matrix 46.9 against 48.8 us; wider entries cost
// registers).
SelectKernel select_kernel(int k, int view, long long P, int n) {
  const bool wide = P >= 12LL * n;
  switch (view) {
    case kView16: return wide ? k_select_light<1, kView16, 8> : k_select_light<1, kView16, 4>;
    case kView32: return wide ? k_select_light<1, kView32, 8> : k_select_light<1, kView32, 4>;
    case kView8: return wide ? k_select_light<1, kView8, 8> : k_select_light<1, kView8, 4>;
    case kView4: return wide ? k_select_light<1, kView4, 8> : k_select_light<1, kView4, 4>;
    case kView64: return k_select_light<2, kView64, 4>;
    case kViewUnit:
      return bit_words(k) == 4 ? k_select_light<4, kViewUnit, 4> : k_select_light<8, kViewUnit, 4>;
    default: break;
  }
  switch (bit_words(k)) {
    case 1: return k_select_light<1, kViewFull, 4>;
    case 2: return k_select_light<2, kViewFull, 4>;
    case 4: return k_select_light<4, kViewFull, 4>;
    default: return k_select_light<8, kViewFull, 4>;
  }
}

// The gain-cache update lives in its own instantiation: the plain one then
// needs far fewer registers (more workgroups per compute unit).
FinalizeKernel finalize_kernel(int k, bool cache) {
  switch (bit_words(k)) {
    case 1: return cache ? k_finalize<1, true> : k_finalize<1, false>;
    case 2: return cache ? k_finalize<2, true> : k_finalize<2, false>;
    case 4: return cache ? k_finalize<4, true> : k_finalize<4, false>;
    default: return cache ? k_finalize<8, true> : k_finalize<8, false>;
  }
}

size_t finalize_lds(int k, bool cache) {
  return sizeof(unsigned) * (size_t)(kBlock / kWave) *
         (count_words(k, count_nets(k)) + kFinalQueue + (cache ? cache_words(bit_words(k)) : 0));
}

// Launch one round of every kernel for a batch (items per kernel kind) or a
// single instance (L.descs == nullptr).
hipError_t launch_round(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks) {
  hipError_t e = launch_round_front(plan, s, marks);
  if (e != hipSuccess) return e;
  return launch_round_back(plan, round, s, marks);
}

// Select, thresholds, tiles and approve (+ apply unless the descriptor asks
// for marks only).
hipError_t launch_round_front(const RoundPlan& plan, hipStream_t s, hipEvent_t* marks) {
  // a null start mark: the previous round's end mark starts this round
  if (marks && marks[0]) (void)hipEventRecord(marks[0], s);
  for (const PlanLaunch& pl : plan.select)
    hipLaunchKernelGGL((SelectKernel)pl.kernel, dim3(pl.grid), dim3(kBlock), 0, s, pl.L);
  for (const PlanLaunch& pl : plan.heavy)
    hipLaunchKernelGGL(k_select_heavy, dim3(pl.grid), dim3(kBlock), 0, s, pl.L);
  if (marks) (void)hipEventRecord(marks[1], s);
  const unsigned extra = plan.tiles.L.one.prev ? 1 : 0;   // the record of the round before
  if (plan.brief) {
    hipLaunchKernelGGL(k_tilesum<true>, dim3(plan.tiles.grid + extra), dim3(kBlock), 0, s, plan.tiles.L);
    hipLaunchKernelGGL(k_approve_apply<true>, dim3(plan.approve.grid), dim3(kBlock), 0, s,
                       plan.approve.L);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_threshold, dim3(plan.blocks.grid + extra), dim3(kBlock), 0, s, plan.blocks.L);
  if (plan.any_heavy)
    hipLaunchKernelGGL(k_overflow_resolve, dim3(plan.blocks.grid), dim3(kBlock), 0, s,
                       plan.blocks.L);
  hipLaunchKernelGGL(k_tilesum<false>, dim3(plan.tiles.grid), dim3(kBlock), 0, s, plan.tiles.L);
  hipLaunchKernelGGL(k_tilescan, dim3(plan.blocks.grid), dim3(kBlock), 0, s, plan.blocks.L);
  hipLaunchKernelGGL(k_approve_apply<false>, dim3(plan.approve.grid), dim3(kBlock), 0, s,
                     plan.approve.L);
  return hipGetLastError();
}

// Finalize (touched nets, next eligible set) and the round record.
hipError_t launch_round_back(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks) {
  hipError_t e = launch_round_finalize(plan, s, marks);
  if (e != hipSuccess) return e;
  return plan.record ? launch_round_stats(plan, round, s, marks) : hipSuccess;
}

hipError_t launch_round_finalize(const RoundPlan& plan, hipStream_t s, hipEvent_t* marks) {
  if (marks) (void)hipEventRecord(marks[2], s);
  for (const PlanLaunch& pl : plan.finalize)
    hipLaunchKernelGGL((FinalizeKernel)pl.kernel, dim3(pl.grid), dim3(kBlock), pl.lds, s, pl.L);
  launch_long(plan.longs, s);
  return hipGetLastError();
}

hipError_t launch_round_stats(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks) {
  Launch ls = plan.stats.L;
  ls.round = round;
  hipLaunchKernelGGL(k_round_stats, dim3(plan.stats.grid), dim3(kBlock), 0, s, ls);
  if (marks) (void)hipEventRecord(marks[3], s);
  return hipGetLastError();
}

// Plan for one instance (no work tables; kernels derive units from blockIdx).
void single_round_plan(const InstDesc& d, RoundPlan& plan) {
  plan = RoundPlan();
  const Launch L = single_launch(d);
  const int chunks = units_of(d.n, kBlock);
  PlanLaunch sel;
  sel.kernel = (void*)select_kernel(d.k, d.sweep, d.P, d.n);
  sel.grid = (unsigned)(chunks < kSelectGrid ? chunks : kSelectGrid);
  sel.L = L;
  plan.select.push_back(sel);
  if (d.heavy_count > 0) {
    PlanLaunch hv;
    hv.grid = (unsigned)(units_of(d.heavy_count, kBlock / kWave));
    hv.L = L;
    plan.heavy.push_back(hv);
    plan.any_heavy = true;
  }
  plan.brief = brief_rounds(d.n, d.k, d.heavy_count);
  plan.blocks.grid = (unsigned)d.k;
  plan.blocks.L = L;
  plan.tiles.grid = (unsigned)d.num_tiles;
  plan.tiles.L = L;
  plan.approve.grid = (unsigned)(d.num_tiles + d.k);
  plan.approve.L = L;
  PlanLaunch fin;
  fin.kernel = (void*)finalize_kernel(d.k, d.cache != nullptr);
  fin.lds = finalize_lds(d.k, d.cache != nullptr);
  const int fchunks = units_of(d.m, kFinalChunk);
  fin.grid = (unsigned)(fchunks < kFinalizeGrid ? fchunks : kFinalizeGrid) + (d.late ? 1 : 0);
  fin.L = L;
  plan.finalize.push_back(fin);
  plan_long(d, long_round_kernel(d.k, d.cache != nullptr), plan.longs);
  plan.stats.grid = 1;
  plan.stats.L = L;
}

}  // namespace hg
