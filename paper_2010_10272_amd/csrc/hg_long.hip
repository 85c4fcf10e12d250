// hg_long.hip -- pin counts and finalize of nets too long for a wavefront (more
// than kWaveNet pins), a workgroup each.  The sweeps over all nets (k_pincounts,
// k_finalize) pass these nets over; a graph that has any lists them once, when it
// is loaded, and its rounds and pin counts get one launch more.
//
// What bounds it: steps of pins, then their blocks, then LDS adds, kLongStep
// pins at a time.  A wavefront walks 256 a step, and every other net of its
// batch waits: one net of 300,000 pins among 50,000 of four, k = 8, pin counts and
// five rounds 14.7 ms by wavefronts, 0.87 so; 20 of 20,000 19.6 and 0.37.
#include "hg_count.h"
#include "hg_device.h"
#include "hg_gain_deltas.h"
#include "hg_internal.h"
#include "hg_lp.h"

namespace hg {
namespace {

constexpr int kLongBlock = 1024;                       // threads
constexpr int kLongStep = kLongBlock * kCountFlight;   // pins in flight
constexpr int kLongGrid = 1024;                        // workgroups striding over the list
constexpr int kLongPieces = 64;                        // the same for a member of a batch

// Every graph's long nets, in any order.
__global__ __launch_bounds__(kBlock) void k_list_long(int m, const long long* eptr, int* list,
                                                      LoadInfo* info) {
  const long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
  const bool is_long = e < m && eptr[e + 1] - eptr[e] > kWaveNet;
  const int at = wave_append(&info->long_count, is_long);
  if (is_long) list[at] = (int)e;
}

enum LongMode { kLongCounts, kLongRound, kLongCached };

// Unit: one listed net.
template <int WK, int MODE>
__global__ __launch_bounds__(kLongBlock) void k_long_nets(Launch L) {
  __shared__ int s_cnt[HG_MAX_K];
  __shared__ unsigned s_lam[8], s_one[8];
  __shared__ unsigned s_chg[4 * WK];   // changed and old Lambda, changed and new S
  __shared__ int s_w;
  WorkItem fb;
  fb.inst = 0;
  fb.first = (int)blockIdx.x;
  fb.stride = (int)gridDim.x;
  fb.count = ((int)L.one.long_count - fb.first + fb.stride - 1) / fb.stride;
  const WorkItem wi = work_item(L, fb);
  const InstDesc D = inst_desc(L, wi.inst);
  const int k = D.k, tid = threadIdx.x;
  const Blocks block = blocks_of(D, MODE == kLongCounts || D.kept != 0);
  for (int it = 0; it < wi.count; ++it) {
    const long long e = D.long_list[wi.first + it * wi.stride];
    if (MODE != kLongCounts && !D.touched[e]) continue;   // the whole workgroup
    const long long b = D.eptr[e], t = D.eptr[e + 1];
    if (tid < k) s_cnt[tid] = 0;
    __syncthreads();
    for (long long p = b; p < t; p += kLongStep) {
      int v[kCountFlight];
      unsigned id[kCountFlight];
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q) {
        const long long i = p + q * kLongBlock + tid;
        v[q] = i < t ? global_ptr(D.pins)[i] : -1;
      }
      block(v, id);
      if constexpr (MODE != kLongCounts) EligiblePins{D.eligible}(v);
#pragma unroll
      for (int q = 0; q < kCountFlight; ++q)
        add_runs(id[q] < (unsigned)k, id[q], [&](int n) { atomicAdd(&s_cnt[id[q]], n); });
    }
    __syncthreads();
    if (tid < HG_MAX_K) {                                  // whole wavefronts
      const int x = tid < k ? s_cnt[tid] : 0;
      if (tid < k) D.phi[e * k + tid] = x;
      const unsigned long long nz = __ballot(x != 0), one = __ballot(x == 1);
      if (lane_id() == 0) {
        const int w = tid / kWave * 2;
        s_lam[w] = (unsigned)nz;
        s_lam[w + 1] = (unsigned)(nz >> 32);
        s_one[w] = (unsigned)one;
        s_one[w + 1] = (unsigned)(one >> 32);
      }
    }
    __syncthreads();
    if (tid == 0) {
      unsigned lam[WK], one[WK];
      int lambda = 0;
#pragma unroll
      for (int x = 0; x < WK; ++x) {
        lam[x] = s_lam[x];
        one[x] = s_one[x];
        lambda += __popc(lam[x]);
      }
      const int sl = (int)(blockIdx.x % kSlots);
      if constexpr (MODE == kLongCounts) {
        const int w = D.ewgt ? D.ewgt[e] : 1;
        write_record<WK, true>(D, e, w, lambda, lam, one);
        if (lambda > 1) atomicAdd(&D.red[sl], (unsigned long long)((long long)(lambda - 1) * w));
      } else {
        int w, lambda_old, left = 0;
        unsigned lam_old[WK], one_old[WK];
        read_record<WK>(D, e, w, lambda_old, lam_old, one_old);
        write_record<WK, false>(D, e, w, lambda, lam, one);
        D.touched[e] = 0;
#pragma unroll
        for (int x = 0; x < WK; ++x) {
          left += __popc(lam_old[x] & ~lam[x]) - __popc(lam[x] & ~lam_old[x]);
          s_chg[x] = lam_old[x] ^ lam[x];
          s_chg[WK + x] = lam_old[x];
          s_chg[2 * WK + x] = one_old[x] ^ one[x];
          s_chg[3 * WK + x] = one[x];
        }
        s_w = w;
        RoundCounters* ctr = D.ctr;
        atomicAdd(&ctr->slot[kCtrDeltaAttr][sl], (unsigned long long)((long long)left * w));
        atomicAdd(&ctr->slot[kCtrDeltaCheck][sl],
                  (unsigned long long)((long long)(lambda_old - lambda) * w));
        atomicAdd(&ctr->slot[kCtrTouched][sl], 1ull);
        atomicAdd(&ctr->slot[kCtrTouchedPins][sl], (unsigned long long)(t - b));
      }
    }
    __syncthreads();
    if constexpr (MODE == kLongCached) {
      unsigned any = 0;
#pragma unroll
      for (int x = 0; x < WK; ++x) any |= s_chg[x] | s_chg[2 * WK + x];
      if (any)
        for (long long p = b + tid; p < t; p += kLongBlock)
          pin_deltas<WK>(D, D.pins[p], s_w, [&](int x) { return s_chg[x]; });
      __syncthreads();                                     // before the next net's sets
    }
  }
}

template <int MODE>
void* long_kernel(int k) {
  switch (bit_words(k)) {
    case 1: return (void*)k_long_nets<1, MODE>;
    case 2: return (void*)k_long_nets<2, MODE>;
    case 4: return (void*)k_long_nets<4, MODE>;
    default: return (void*)k_long_nets<8, MODE>;
  }
}

}  // namespace

void* long_counts_kernel(int k) { return long_kernel<kLongCounts>(k); }
void* long_round_kernel(int k, bool cache) {
  return cache ? long_kernel<kLongCached>(k) : long_kernel<kLongRound>(k);
}
int long_pieces(int long_count) { return long_count < kLongPieces ? long_count : kLongPieces; }

void plan_long(const InstDesc& d, void* kernel, std::vector<PlanLaunch>& out) {
  if (d.long_count == 0) return;
  PlanLaunch pl;
  pl.kernel = kernel;
  pl.grid = (unsigned)(d.long_count < kLongGrid ? d.long_count : kLongGrid);
  pl.L = single_launch(d);
  out.push_back(pl);
}

void launch_long(const std::vector<PlanLaunch>& plan, hipStream_t s) {
  for (const PlanLaunch& pl : plan)
    hipLaunchKernelGGL((FinalizeKernel)pl.kernel, dim3(pl.grid), dim3(kLongBlock), 0, s, pl.L);
}

hipError_t list_long_nets(hg_graph_s* g, hipStream_t s) {
  if (g->info.max_net_size <= kWaveNet) return hipSuccess;
  hipLaunchKernelGGL(k_list_long, dim3((unsigned)units_of(g->m, kBlock)), dim3(kBlock), 0, s, g->m,
                     g->eptr, (int*)(g->ws + g->lay.longs), (LoadInfo*)(g->ws + g->lay.info));
  return hipGetLastError();
}

}  // namespace hg
