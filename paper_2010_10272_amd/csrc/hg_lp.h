// hg_lp.h -- launch plans: which kernels a round (or a pin-count pass) runs,
// with which grid and arguments, for one instance or a batch.
#pragma once

#include <vector>

#include "hg_count.h"
#include "hg_internal.h"

namespace hg {

constexpr int kFinalChunk = kBlock;   // nets per unit of the finalize sweep

typedef void (*SelectKernel)(Launch);
typedef void (*FinalizeKernel)(Launch);
typedef void (*GroupKernel)(Launch);
typedef void (*GainsKernel)(Launch);

struct PlanLaunch {
  void* kernel = nullptr;   // for templated kernels: which instantiation
  void* kept_kernel = nullptr;   // batched select: the same where the private views are kept
  unsigned grid = 0;
  size_t lds = 0;           // dynamic LDS bytes (pin counts, finalize)
  Launch L{};
};

// One LP round: select launches (one per kernel variant in a batch), heavy
// select, per-block kernels (threshold, overflow, tilescan), tiles, approve,
// finalize launches (one per bitset width; likewise for long nets), stats.
struct RoundPlan {
  std::vector<PlanLaunch> select, heavy, finalize, longs;
  PlanLaunch blocks, tiles, approve, stats;
  bool any_heavy = false;
  bool brief = false;       // no threshold, no tile scan (brief_rounds)
  bool record = true;       // false: the next round's launches write the record
};

// The plan of calls that count the pins and run the rounds (InstDesc::kept), from
// a batch's plan.
RoundPlan kept_plan(const RoundPlan& plan);

// Pin counts (one launch per bitset width; likewise for long nets), then the
// per-instance km1 slot sums, the block-weight reset and sweep.
struct CountPlan {
  std::vector<PlanLaunch> pincounts, longs;
  PlanLaunch instances;     // one workgroup per instance
  PlanLaunch vertices;      // block weights: units of kBwChunk vertices
};

// Nets per unit of the pin counts: as many as a wavefront counts at a time,
// fewer where that leaves under eight wavefronts per compute unit (1,510 nets
// at k = 100: pin counts and gains 50 us with 64, 45 with 8); of long nets fewer
// still, up to 32 wavefronts while each has 512 pins (200 nets of 300, k = 8: 11.4 us
// with 1,024 pins, 8.6 so, 6.8 with 256; 10,000 of 300 14.8, 14.2, 17.1).
__host__ __device__ inline int count_unit(int k, long long m, long long P) {
  int nets = count_nets(k);
  while (nets > 8 && m < 2048LL * nets) nets >>= 1;
  while (nets > 1 && m < 8192LL * nets && nets / 2 * P >= 512 * m) nets >>= 1;
  return nets * (kBlock / kWave);
}

constexpr int kBwChunk = kBlock * 16;   // vertices per unit of the block-weight sweep

SelectKernel select_kernel(int k, int view, long long P, int n);
// cache: the variant that also applies the gain-cache deltas (it must be used
// exactly when the descriptor has a cache)
FinalizeKernel finalize_kernel(int k, bool cache);
size_t finalize_lds(int k, bool cache);      // its dynamic LDS bytes
// The pin-count kernel, the nets of its units (at most kBlock), its dynamic LDS bytes.
GroupKernel pincount_kernel(int k, long long m, long long P, bool batch);
int pincount_unit(int k, long long m, long long P, bool batch);
size_t pincount_lds(int k, long long m, long long P, bool batch);
GainsKernel gains_kernel(int k, int view);
// Nets of more than kWaveNet pins (InstDesc::long_list): the kernels of their pin
// counts and rounds, a single instance's launch (none without such nets), the
// work items of a batch member, the launches.
void* long_counts_kernel(int k);
void* long_round_kernel(int k, bool cache);
void plan_long(const InstDesc& d, void* kernel, std::vector<PlanLaunch>& out);
int long_pieces(int long_count);
void launch_long(const std::vector<PlanLaunch>& plan, hipStream_t s);

// Enqueue one round; the round record goes to stats[round] of every instance.
hipError_t launch_round(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks);
// Its two halves: select .. approve (+ apply), then finalize and the record.
hipError_t launch_round_front(const RoundPlan& plan, hipStream_t s, hipEvent_t* marks);
hipError_t launch_round_back(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks);
// launch_round_back in two steps: finalize, then the round record.
hipError_t launch_round_finalize(const RoundPlan& plan, hipStream_t s, hipEvent_t* marks);
hipError_t launch_round_stats(const RoundPlan& plan, int round, hipStream_t s, hipEvent_t* marks);
void single_round_plan(const InstDesc& d, RoundPlan& plan);
// Gain-cache rounds (single instance, d.cache and d.moved set): the plan and
// its launch (front, finalize with cache deltas, movers' b, record).
SelectKernel select_cached_kernel(int k);
void cached_round_plan(const InstDesc& d, RoundPlan& plan);
hipError_t launch_cached_round(const RoundPlan& plan, int round, hipStream_t s,
                               hipEvent_t* marks);

// Pin counts, block weights and (want_km1) km1 of every instance; with
// mark_eligible every vertex is made eligible as well.
hipError_t launch_counts(const CountPlan& plan, bool want_km1, bool mark_eligible, hipStream_t s);
void single_count_plan(const InstDesc& d, CountPlan& plan);

// All gains (or, with `cache`, a gain cache: b, w(I), p rows; see hgref.h).
hipError_t launch_gains(hg_graph_s* g, const InstDesc& d, long long* gains, long long* benefit,
                        hipStream_t s, int* cache = nullptr);
// The gain cache's entries of the heavy vertices in blocks heavier than d.lmax.
hipError_t launch_over_rows(const InstDesc& d, int* cache, hipStream_t s);
hipError_t launch_km1(hg_graph_s* g, int k, const unsigned* netstate, long long* km1,
                      hipStream_t s);

}  // namespace hg
