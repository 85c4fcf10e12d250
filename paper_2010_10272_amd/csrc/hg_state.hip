// hg_state.hip -- pin counts Phi(e,i), connectivity sets Lambda(e), the
// singleton sets S(e) = {i : Phi(e,i) = 1}, block weights c(V_i) and km1.
//
// Section "Preliminaries" defines Phi, Lambda, lambda and km1; subsection
// "Data Structures for Gain Calculation" keeps Phi and a bitset Lambda per
// net.  Here a wavefront owns 64 consecutive nets at a time: their pins are one
// run of the pin array, counted 64 at a time into byte counters in LDS; then
// each lane builds its net's bitsets from its counters, and the rows leave as
// whole lines.  No global atomics touch Phi, so the result is deterministic by
// construction.
#include "hg_device.h"
#include "hg_internal.h"
#include "hg_lp.h"
#include "hg_netrec.h"

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
constexpr int kCountFlight = 4;              // pins in flight per lane
constexpr int kByteNet = 255;                // longest net whose counts surely fit a byte

// Words of a net's byte counters in LDS: odd, so that lanes reading their own
// nets' word i use all banks.
__host__ __device__ __forceinline__ int count_stride(int k) { return ((k + 3) / 4) | 1; }

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

// Counts of one net longer than kByteNet by the whole wavefront, in 32-bit
// words (`cnt`, k of them): Phi row, and its bits into the lane that owns it.
template <typename Block>
__device__ void count_long_net(const InstDesc& D, long long e, long long b, long long t, int* cnt,
                               Block block) {
  const int lane = lane_id(), k = D.k;
  for (int i = lane; i < k; i += kWave) cnt[i] = 0;
  wave_lds_sync();
  for (long long p = b + lane; p < t; p += kWave) {
    const unsigned v = block(D.pins[p]);
    if (v < (unsigned)k) atomicAdd(&cnt[v], 1);
  }
  wave_lds_sync();
  for (int i = lane; i < k; i += kWave) D.phi[e * k + i] = cnt[i];
}

// Unit: count_unit consecutive nets.  What bounds it: the block ids' gathers
// (lines outstanding per compute unit).  A lane group per net (8 lanes, four
// slots each) left two thirds of the gather slots empty on nets of ten pins and
// half the lanes idle; here every lane has a pin.  Pins of a net in one block
// are often neighbours, so each run of equal (net, block) adds once.  (Four
// consecutive pins per lane need a third fewer operations, but their gathers
// touch more lines at a time: netlist 370 -> 404 us.)  Per call, before and
// now: netlist 56.5M pins, k = 16 523 -> 367 us (gathers 135 of them, Phi
// stores 65), matrix 10M pins k = 8 82 -> 48, k = 64 128 -> 95.
template <int WK>
__global__ __launch_bounds__(kBlock) void k_pincounts(Launch L) {
  extern __shared__ unsigned s_count[];   // per wave: NW x stride byte counters, k words
  __shared__ unsigned char s_flag[kBlock / kWave][kCountFlight * kWave];
  __shared__ long long s_km1;
  const WorkItem wi = work_item(L, contiguous_units((L.one.m + count_unit(L.one.k, L.one.m) - 1) /
                                                     count_unit(L.one.k, L.one.m)));
  if (wi.count == 0) return;
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, m = D.m;
  const int unit_nets = count_unit(k, m), NW = unit_nets / (kBlock / kWave);
  const int stride = count_stride(k);
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  unsigned* cnt = s_count + (size_t)wv * (NW * stride + k);
  int* big = reinterpret_cast<int*>(cnt + NW * stride);
  unsigned char* flag = s_flag[wv];
  const bool checked = (*D.err_flags & kErrPart) == 0;
  const bool nibbles = k <= 16;
  auto block = [&](int v) -> unsigned {
    if (!checked) return (unsigned)D.part[v];
    if (!nibbles) return D.part8[v];
    return (D.part8[(unsigned)v >> 1] >> (4 * (v & 1))) & 15u;
  };
  // Phi rows leave as 16-byte streaming stores when rows are 16-byte aligned
  const bool vec_phi = (k & 3) == 0 && ((uintptr_t)D.phi & 15) == 0;
  if (threadIdx.x == 0) s_km1 = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kCountFlight; ++q) flag[q * kWave + lane] = 0;
  for (int i = lane; i < NW * stride; i += kWave) cnt[i] = 0;
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
      nb = D.eptr[e0 + lane];
      nt = D.eptr[e0 + lane + 1];
    }
  };
  load_range(first_net(0));
  for (int it = 0; it < wi.count; ++it) {
    const long long e0 = first_net(it);
    const long long b = nb;
    const int len = (int)(nt - nb);
    load_range(first_net(it + 1));
    if (e0 >= m) continue;                                  // the same for the whole wave
    const int nets = m - e0 < NW ? (int)(m - e0) : NW;
    const long long e = e0 + lane;
    const unsigned long long is_long = __ballot(len > kByteNet);
    const int incl = wave_incl_scan(len);
    const int total = last_lane(incl), first = incl - len;  // this net's place in the run
    const long long run = __shfl(b, 0);
    const int* pins = D.pins + run;
    wave_lds_sync();
    int before = -1;                                        // last net starting before this step
    for (int s = 0; s < total; s += kCountFlight * kWave) {
      int v[kCountFlight];
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const int p = s + q * kWave + lane;
        v[q] = p < total ? pins[p] : -1;
      }
      if (len > 0 && first >= s && first < s + kCountFlight * kWave) flag[first - s] = 1;
      unsigned id[kCountFlight];
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) id[q] = v[q] >= 0 ? block(v[q]) : ~0u;
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const unsigned here = flag[q * kWave + lane];
        flag[q * kWave + lane] = 0;
        const unsigned long long starts = __ballot(here != 0);
        const int net = lanes_below(starts, before) + (int)here;
        before += __popcll(starts);
        bool live = id[q] < (unsigned)k;
        if (is_long) live = live && !((is_long >> (net & 63)) & 1ull);
        // one add per run of equal (net, block) in neighbouring lanes
        const unsigned key = live ? ((unsigned)net << 8) | id[q] : ~0u;
        const unsigned prev = lane_before(key);
        const unsigned long long heads = __ballot(lane == 0 || key != prev);
        if (live && ((heads >> lane) & 1ull)) {
          const unsigned long long later = heads >> lane >> 1;
          const int run_len = later ? __ffsll((long long)later) : kWave - lane;
          atomicAdd(&cnt[net * stride + (id[q] >> 2)], (unsigned)run_len << (8 * (id[q] & 3)));
        }
      }
      wave_lds_sync();
    }
    // lane's net: bitsets from its counters
    unsigned lam[WK], one[WK];
    int lambda = 0;
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      lam[w] = one[w] = 0;
      if (lane < nets) {
        for (int j = 0; j < 8 && w * 32 + 4 * j < k; ++j) {
          unsigned nz, on;
          byte_bits(cnt[lane * stride + w * 8 + j], nz, on);
          lam[w] |= nz << (4 * j);
          one[w] |= on << (4 * j);
        }
      }
      lambda += __popc(lam[w]);
    }
    // Phi rows: the run of rows, 16 bytes (or one count) per lane and step
    if (vec_phi) {
      const int words = k >> 2, all = nets * words;
      int row = lane / words, col = lane % words;           // words <= 64
      const int drow = kWave / words, dcol = kWave % words;
      for (int i = lane; i < all; i += kWave) {
        const unsigned x = cnt[row * stride + col];
        const i32x4 o = {(int)(x & 255u), (int)((x >> 8) & 255u), (int)((x >> 16) & 255u),
                         (int)(x >> 24)};
        if (!((is_long >> row) & 1ull))
          __builtin_nontemporal_store(o, reinterpret_cast<i32x4*>(D.phi + e0 * k) + i);
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
          D.phi[e0 * k + i] = (int)((cnt[row * stride + (col >> 2)] >> (8 * (col & 3))) & 255u);
      }
    }
    wave_lds_sync();
    for (int i = lane; i < nets * stride; i += kWave) cnt[i] = 0;   // for the next nets
    for (unsigned long long left = is_long; left; left &= left - 1) {
      const int j = __ffsll((long long)left) - 1;
      const long long lb = __shfl(b, j);
      count_long_net(D, e0 + j, lb, lb + __shfl(len, j), big, block);
      if (lane == j) {
        lambda = 0;
#pragma unroll
        for (int w = 0; w < WK; ++w) {
          lam[w] = one[w] = 0;
          for (int i = 0; i < 32 && w * 32 + i < k; ++i) {
            lam[w] |= (big[w * 32 + i] > 0 ? 1u : 0u) << i;
            one[w] |= (big[w * 32 + i] == 1 ? 1u : 0u) << i;
          }
          lambda += __popc(lam[w]);
        }
      }
      wave_lds_sync();
    }
    if (lane < nets) {
      const int w = D.ewgt ? D.ewgt[e] : 1;
      write_record<WK>(D, e, w, lambda, lam, one);
      km1_local += (long long)(lambda - 1) * w;
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
  const WorkItem wi = work_item(L, contiguous_units((L.one.n + kBwChunk - 1) / kBwChunk));
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

// Lanes per net for the finalize: enough lanes to hold every word of the net
// record (2 + 2 * bit_words(k), padded), and no more than that (but 8 for
// 4 < k <= 64): most nets have only a handful of pins, so narrower groups put
// more nets' loads in flight per wavefront.
int group_lanes(int k) {
  if (k <= 4) return 4;
  return net_words(k) > 8 ? net_words(k) : 8;
}

size_t pincount_lds(int k, long long m) {
  return sizeof(unsigned) *
         ((size_t)count_unit(k, m) * count_stride(k) + (size_t)(kBlock / kWave) * k);
}

GroupKernel pincount_kernel(int k) {
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
  pc.kernel = (void*)pincount_kernel(d.k);
  pc.grid = grid_cap(d.m, count_unit(d.k, d.m), kStateGrid);
  pc.lds = pincount_lds(d.k, d.m);
  pc.L = L;
  plan.pincounts.push_back(pc);
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
