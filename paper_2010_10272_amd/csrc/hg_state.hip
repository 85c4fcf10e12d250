// hg_state.hip -- pin counts Phi(e,i), connectivity sets Lambda(e), the
// singleton sets S(e) = {i : Phi(e,i) = 1}, block weights c(V_i) and km1.
//
// Section "Preliminaries" defines Phi, Lambda, lambda and km1; subsection
// "Data Structures for Gain Calculation" keeps Phi and a bitset Lambda per
// net.  Here a wavefront owns 64 consecutive nets at a time: their pins are one
// run of the pin array, counted 64 at a time into byte counters in LDS; then
// each lane builds its net's bitsets from its counters, and the rows leave as
// whole lines.  Nets of 64 pins and more on average get eight lanes each, nets of
// more than kWaveNet pins a workgroup.  No global atomics touch Phi, so the result is deterministic by
// construction.
#include <climits>

#include "hg_count.h"
#include "hg_device.h"
#include "hg_internal.h"
#include "hg_lp.h"

namespace hg {

constexpr int kStateGrid = 4096;   // persistent workgroups of the single-instance net sweep
constexpr int kKm1Chunk = kBlock * 8;

__device__ __forceinline__ WorkItem contiguous_units(long long units) {
  const long long lb = xcd_remap(blockIdx.x, gridDim.x);
  const long long per = (units + gridDim.x - 1) / gridDim.x;
  long long end = (lb + 1) * per;
  if (end > units) end = units;
  WorkItem w;
  w.inst = 0;
  w.first = (int)(lb * per);
  w.stride = 1;
  w.count = lb * per < end ? (int)(end - lb * per) : 0;
  return w;
}

// Block ids are gathered from a packed copy of the partition that the
// block-weight sweep writes just before: four bits a vertex for k <= 16, a byte
// beyond (2 and 4 MB on a 4M-vertex netlist, where an XCD's L2 has 4 MB, instead
// of 16 MB).  If that sweep met an id outside [0, k), the ids come from the
// partition itself, so that such vertices are skipped.
//
// Unit: count_unit consecutive nets.  What bounds it: the block ids' gathers
// (lines outstanding per compute unit).  A lane group per net (8 lanes, four
// slots each) left two thirds of the gather slots empty on nets of ten pins and
// half the lanes idle; here every lane has a pin.  (Four consecutive pins per
// lane need a third fewer operations, but their gathers touch more lines at a
// time: netlist 370 -> 404 us.)  Per launch, lane groups and now: netlist 56.5M pins,
// k = 16 523 -> 306 us, matrix 10M pins k = 8 82 -> 43 (38 repeated, 51 after other
// work), k = 64 128 -> 71 (61, 90).
template <int WK>
__global__ __launch_bounds__(kBlock) void k_pincounts(Launch L) {
  extern __shared__ unsigned s_count[];   // count_words per wavefront
  __shared__ long long s_km1;
  const WorkItem wi = work_item(L, contiguous_units(units_of(L.one.m, count_unit(L.one.k, L.one.m, L.one.P))));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, m = D.m;
  const int unit_nets = count_unit(k, m, D.P), NW = unit_nets / (kBlock / kWave);
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const CountLds M = count_lds(s_count + (size_t)wv * count_words(k, NW), k, NW);
  const Blocks block = blocks_of(D, true);
  const bool vec_phi = aligned_rows(D);
  if (threadIdx.x == 0) s_km1 = 0;
  __syncthreads();
  long long km1_local = 0;
  // first net of turn `it`, and lane's pin range in it (the next turn's is
  // loaded while this one's pins are counted)
  auto first_net = [&](int it) {
    return it < wi.count
               ? ((long long)wi.first + (long long)it * wi.stride) * unit_nets + wv * NW
               : (long long)m;
  };
  long long nb = 0, nt = 0;
  auto load_range = [&](long long e0) {
    nb = nt = 0;
    if (lane < NW && e0 + lane < m) {
      nb = global_ptr(D.eptr)[e0 + lane];
      nt = global_ptr(D.eptr)[e0 + lane + 1];
    }
  };
  load_range(first_net(0));
  for (int it = 0; it < wi.count; ++it) {
    const long long e0 = first_net(it);
    const long long b = nb;
    const int len = (int)(nt - nb);
    load_range(first_net(it + 1));
    if (e0 >= m) continue;                                  // the same for the whole wave
    const long long e = e0 + lane;
    NetSets<WK> N;
    count_batch<WK, true>(D, M, e, b, len, vec_phi, block,
                          [](const int (&)[kCountFlight]) {}, N);
    if (len > 0 && len <= kWaveNet) {                       // longer: k_long_nets
      const int w = D.ewgt ? global_ptr(D.ewgt)[e] : 1;
      write_record<WK, true>(D, e, w, N.lambda, N.lam, N.one);
      km1_local += (long long)(N.lambda - 1) * w;
    }
  }
  km1_local = wave_sum(km1_local);
  if (lane == 0 && km1_local) atomicAdd((unsigned long long*)&s_km1, (unsigned long long)km1_local);
  __syncthreads();
  if (threadIdx.x == 0 && s_km1)
    atomicAdd(&D.red[blockIdx.x % kSlots], (unsigned long long)s_km1);
}

// The same where nets are long on average (group_counts): kGroupLanes lanes a net,
// eight nets a wavefront, 32-bit counters.  A net's pins are consecutive, so no
// place has to look for its net, and few registers keep many wavefronts in flight;
// short nets would leave most lanes idle.  The Phi rows pass the caches by (400,000 nets
// of 100, k = 64: 100 -> 76 us).
// Unit: kGroupUnit consecutive nets.
constexpr int kGroupLanes = 8;
constexpr int kGroupNets = kWave / kGroupLanes;
constexpr int kGroupUnit = kBlock / kGroupLanes;

template <int WK>
__global__ __launch_bounds__(kBlock) void k_pincounts_groups(Launch L) {
  extern __shared__ unsigned s_count[];   // kGroupUnit * (k | 1)
  __shared__ long long s_km1;
  const WorkItem wi = work_item(L, contiguous_units(units_of(L.one.m, kGroupUnit)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, ks = k | 1, m = D.m;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int grp = lane / kGroupLanes, gl = lane % kGroupLanes;
  unsigned* cnt = s_count + wv * kGroupNets * ks;         // the wavefront's
  for (int i = lane; i < kGroupNets * ks; i += kWave) cnt[i] = 0;
  const Blocks block = blocks_of(D, true);
  const auto pins = global_ptr(D.pins);
  if (threadIdx.x == 0) s_km1 = 0;
  __syncthreads();
  long long km1_local = 0, b = 0, t = 0;
  // the next net's range is loaded while this one's pins are counted
  auto net_at = [&](int it) {
    return ((long long)wi.first + (long long)it * wi.stride) * kGroupUnit + wv * kGroupNets + grp;
  };
  auto load_range = [&](int it) {
    b = t = 0;
    if (it < wi.count && net_at(it) < m) {
      b = global_ptr(D.eptr)[net_at(it)];
      t = global_ptr(D.eptr)[net_at(it) + 1];
    }
  };
  load_range(0);
  for (int it = 0; it < wi.count; ++it) {
    const long long e = net_at(it), at = b;
    const int len = t - b <= kWaveNet ? (int)(t - b) : 0;  // longer: k_long_nets
    load_range(it + 1);
    for (int s = gl; s < len; s += kCountFlight * kGroupLanes) {
      int v[kCountFlight];
      unsigned id[kCountFlight];
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const int p = s + q * kGroupLanes;
        v[q] = pins[at + (p < len ? p : s)];
      }
      block(v, id);
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q)
        if (s + q * kGroupLanes < len && id[q] < (unsigned)k)
          atomicAdd(&cnt[grp * ks + (int)id[q]], 1u);
    }
    wave_lds_sync();
    NetSets<WK> N;
    N.lambda = 0;
#pragma unroll
    for (int w = 0; w < WK; ++w) N.lam[w] = N.one[w] = 0;
    const unsigned long long there = __ballot(len > 0);
#pragma unroll
    for (int r = 0; r < kGroupNets; ++r) {
      const int owner = r * kGroupLanes;
      if (!((there >> owner) & 1ull)) continue;
      const long long phi_row = lane_value(e, owner) * k;
#pragma unroll
      for (int h = 0; h < WK; h += 2) {
        const int i = h * 32 + lane;
        int x = 0;
        if (i < k) {
          x = (int)cnt[r * ks + i];
          cnt[r * ks + i] = 0;             // for the next nets
          __builtin_nontemporal_store(x, global_out(D.phi) + phi_row + i);
        }
        set_words<WK>(N, h, __ballot(x != 0), __ballot(x == 1), lane == owner);
      }
    }
    wave_lds_sync();
    if (gl == 0 && len > 0) {
      const int w = D.ewgt ? global_ptr(D.ewgt)[e] : 1;
      write_record<WK, true>(D, e, w, N.lambda, N.lam, N.one);
      km1_local += (long long)(N.lambda - 1) * w;
    }
  }
  km1_local = wave_sum(km1_local);
  if (lane == 0 && km1_local) atomicAdd((unsigned long long*)&s_km1, (unsigned long long)km1_local);
  __syncthreads();
  if (threadIdx.x == 0 && s_km1)
    atomicAdd(&D.red[blockIdx.x % kSlots], (unsigned long long)s_km1);
}

// Unit: one instance.  Sum its km1 slots into *km1 (or just clear them) and
// fold the block-weight slot rows of the sweep before into block_w (clearing
// them for the rounds).
__global__ __launch_bounds__(kBlock) void k_count_epilogue(Launch L, int want_km1) {
  const WorkItem wi = work_item(L, WorkItem{0, 0, 1, 1});
  const InstDesc D = inst_desc(L, wi.inst);
  if (threadIdx.x < kWave) {
    const int lane = lane_id();
    long long v = (long long)D.red[lane];
    D.red[lane] = 0;
    v = wave_sum(v);
    if (lane == 0 && want_km1) *D.km1 = v;
  }
  const size_t ks = (size_t)D.k;
  for (int i = threadIdx.x; i < D.k; i += kBlock) {
    long long* col = D.bw_slots + i;
    long long w = 0;
    for (int s0 = 0; s0 < kSlots; s0 += 16) {      // 16 loads in flight, then the clears
      long long cells[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) cells[q] = col[(s0 + q) * ks];
#pragma unroll
      for (int q = 0; q < 16; ++q) w += cells[q];
#pragma unroll
      for (int q = 0; q < 16; ++q) col[(s0 + q) * ks] = 0;
    }
    D.block_w[i] = w;
  }
}

// Unit: kBwChunk consecutive vertices, eight per thread and step.  LDS partial
// sums per workgroup, then one atomic per block into the workgroup's slot row
// (the epilogue folds the rows into block_w).  Every vertex's block also goes to
// part8, packed as the pin counts read it.  With mark_eligible every vertex is
// also made eligible (the start of a refinement).
__global__ __launch_bounds__(kBlock) void k_block_weights(Launch L, int mark_eligible) {
  __shared__ unsigned long long s_w[HG_MAX_K];
  const WorkItem wi = work_item(L, contiguous_units(units_of(L.one.n, kBwChunk)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, n = D.n;
  for (int i = threadIdx.x; i < k; i += kBlock) s_w[i] = 0;
  __syncthreads();
  int err = 0;
  constexpr int kRow = 8;                               // consecutive vertices per thread
  constexpr int kPer = kBwChunk / (kBlock * kRow);
  // eligible flags eight at a time where the caller's array allows it
  const bool wide_flags = ((uintptr_t)D.eligible & 7) == 0;
  const bool nibbles = k <= 16;
  for (int it = 0; it < wi.count; ++it) {
    const long long base = ((long long)wi.first + (long long)it * wi.stride) * kBwChunk;
    // every vertex's block and weight requested before the first wait
    int blk[kPer][kRow], cw[kPer][kRow];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const long long v = base + ((long long)j * kBlock + threadIdx.x) * kRow;
      if (v + kRow <= n) {
#pragma unroll
        for (int h = 0; h < kRow; h += 4) {
          const i32x4u x = load4_unaligned(D.part + v + h);
#pragma unroll
          for (int q = 0; q < 4; ++q) blk[j][h + q] = x[q];
        }
        if (D.vwgt) {
#pragma unroll
          for (int h = 0; h < kRow; h += 4) {
            const i32x4u x = load4_unaligned(D.vwgt + v + h);
#pragma unroll
            for (int q = 0; q < 4; ++q) cw[j][h + q] = x[q];
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < kRow; ++q) {
          blk[j][q] = v + q < n ? D.part[v + q] : 0;
          cw[j][q] = v + q < n && D.vwgt ? D.vwgt[v + q] : 1;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const long long v = base + ((long long)j * kBlock + threadIdx.x) * kRow;
      if (v >= n) continue;
      const int have = n - v < kRow ? (int)(n - v) : kRow;
      unsigned long long packed = 0;
#pragma unroll
      for (int q = 0; q < kRow; ++q) {
        if (q < have) {
          if ((unsigned)blk[j][q] < (unsigned)k)
            atomicAdd(&s_w[blk[j][q]], (unsigned long long)(D.vwgt ? cw[j][q] : 1));
          else
            err = kErrPart;
          packed |= nibbles ? (unsigned long long)(blk[j][q] & 15) << (4 * q)
                            : (unsigned long long)(blk[j][q] & 255) << (8 * q);
        }
      }
      // part8 holds whole groups of eight past n (see ws_layout)
      if (nibbles)
        *reinterpret_cast<unsigned*>(D.part8 + v / 2) = (unsigned)packed;
      else
        *reinterpret_cast<unsigned long long*>(D.part8 + v) = packed;
      if (mark_eligible) {
        if (wide_flags && have == kRow)
          *reinterpret_cast<unsigned long long*>(D.eligible + v) = 0x0101010101010101ull;
        else
          for (int q = 0; q < have; ++q) D.eligible[v + q] = 1;
      }
    }
  }
  if (err) atomicOr(D.err_flags, err);
  __syncthreads();
  long long* my_w = D.bw_slots + (size_t)(blockIdx.x % kSlots) * k;
  for (int i = threadIdx.x; i < k; i += kBlock)
    if (s_w[i]) atomicAdd((unsigned long long*)&my_w[i], s_w[i]);
}

// km1 partial sums from the net-state records (single instance only).
__global__ __launch_bounds__(kBlock) void k_km1(int m, int rw, const unsigned* netstate,
                                                unsigned long long* km1_slots) {
  __shared__ long long s_tmp[kBlock / kWave];
  long long stride = (long long)gridDim.x * kBlock;
  long long acc = 0;
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < m; e += stride) {
    const unsigned* r = netstate + e * rw;
    acc += (long long)((int)r[1] - 1) * (int)r[0];
  }
  acc = block_sum64(acc, s_tmp);
  if (threadIdx.x == 0 && acc) atomicAdd(&km1_slots[blockIdx.x % kSlots], (unsigned long long)acc);
}

// Sum the kSlots partials into *out and clear them (one wavefront).
__global__ void k_sum_slots(unsigned long long* slots, long long* out) {
  const int lane = lane_id();
  long long v = (long long)slots[lane];
  slots[lane] = 0;
  v = wave_sum(v);
  if (lane == 0) *out = v;
}

static unsigned grid_cap(long long items, int per_block, int cap) {
  long long b = (items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

// Lane groups for up to 64 blocks and nets of 64 pins and more on average; but not for
// a few thousand nets, which then get a wavefront each.  Us, k_pincounts and lane
// groups, n = 131,072, whole calls: 100,000 nets of 200 from one window k = 8 57 / 38,
// k = 64 56 / 41, from anywhere 83 / 82, 94 / 95; 600,000 of 64 k = 8 97 / 79, k = 64
// 85 / 81; n = 100,000, kernels: 100,000 of 300 k = 8 86 / 52, k = 64 109 / 73; but
// 300,000 of 100 k = 200 144 / 248; 2,100 of 300 k = 8 9.6 / 12.3.
// A batch gives a workgroup 256 nets whatever their length (16 members of 200 nets of
// 300, k = 8, 93 / 38).
static bool group_counts(int k, long long m, long long P, bool batch) {
  return k <= 64 && P >= 64 * m && (batch || m >= 4096);
}

int pincount_unit(int k, long long m, long long P, bool batch) {
  return group_counts(k, m, P, batch) ? kGroupUnit : count_unit(k, m, P);
}

size_t pincount_lds(int k, long long m, long long P, bool batch) {
  if (group_counts(k, m, P, batch)) return sizeof(unsigned) * kGroupUnit * (size_t)(k | 1);
  const int nets = count_unit(k, m, P) / (kBlock / kWave);
  return sizeof(unsigned) * (size_t)(kBlock / kWave) * count_words(k, nets);
}

GroupKernel pincount_kernel(int k, long long m, long long P, bool batch) {
  if (group_counts(k, m, P, batch)) {
    return bit_words(k) == 1 ? k_pincounts_groups<1> : k_pincounts_groups<2>;
  }
  switch (bit_words(k)) {
    case 1: return k_pincounts<1>;
    case 2: return k_pincounts<2>;
    case 4: return k_pincounts<4>;
    default: return k_pincounts<8>;
  }
}

void single_count_plan(const InstDesc& d, CountPlan& plan) {
  plan = CountPlan();
  const Launch L = single_launch(d);
  PlanLaunch pc;
  pc.kernel = (void*)pincount_kernel(d.k, d.m, d.P, false);
  // lane groups: a unit a workgroup, however many (a second turn of a few units of
  // 131,072 + i nets cost 40%: 160,000 of 200, k = 8, 70 -> 51 us)
  pc.grid = grid_cap(d.m, pincount_unit(d.k, d.m, d.P, false),
                     group_counts(d.k, d.m, d.P, false) ? INT_MAX : kStateGrid);
  pc.lds = pincount_lds(d.k, d.m, d.P, false);
  pc.L = L;
  plan.pincounts.push_back(pc);
  plan_long(d, long_counts_kernel(d.k), plan.longs);
  plan.instances.grid = 1;
  plan.instances.L = L;
  plan.vertices.grid = grid_cap(d.n, kBwChunk, 4096);
  plan.vertices.L = L;
}

// Block weights (and the byte partition), then pin counts, then km1 and the
// block-weight fold.
hipError_t launch_counts(const CountPlan& plan, bool want_km1, bool mark_eligible, hipStream_t s) {
  hipLaunchKernelGGL(k_block_weights, dim3(plan.vertices.grid), dim3(kBlock), 0, s,
                     plan.vertices.L, mark_eligible ? 1 : 0);
  for (const PlanLaunch& pl : plan.pincounts)
    hipLaunchKernelGGL((GroupKernel)pl.kernel, dim3(pl.grid), dim3(kBlock), pl.lds, s, pl.L);
  launch_long(plan.longs, s);
  hipLaunchKernelGGL(k_count_epilogue, dim3(plan.instances.grid), dim3(kBlock), 0, s,
                     plan.instances.L, want_km1 ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_km1(hg_graph_s* g, int k, const unsigned* netstate, long long* km1,
                      hipStream_t s) {
  unsigned long long* slots = (unsigned long long*)(g->ws + g->lay.red);
  hipLaunchKernelGGL(k_km1, dim3(grid_cap(g->m, kKm1Chunk, kStateGrid)), dim3(kBlock), 0, s,
                     g->m, net_words(k), netstate, slots);
  hipLaunchKernelGGL(k_sum_slots, dim3(1), dim3(kWave), 0, s, slots, km1);
  return hipGetLastError();
}

}  // namespace hg
