// hg_internal.h -- shared definitions of the HIP implementation behind hgref.h.
//
// Data layout in device memory (all caller-owned):
//   net CSR          eptr int64[m+1], pins int32[P]
//   incidence CSR    vptr int64[n+1], vnets int32[P] (rows sorted by net id)
//   partition state  part int32[n], phi int32[m*k] (row-major by net),
//                    netstate uint32[m*RW] (RW = hg_net_words(k)), block_w int64[k]
//   workspace        carved by WsLayout below
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hgref.h"

namespace hg {

constexpr int kWave = 64;
constexpr int kBlock = 256;            // threads per workgroup in every kernel
constexpr int kTile = 512;             // vertices per approval tile (256 threads x 2)
constexpr int kPerThreadTile = kTile / kBlock;
constexpr int kBuckets = 256;          // gain buckets per target block (0..254 exact, 255 = ">=255")
constexpr int kLightLimit = 255;       // w(I(v)) <= 255: bit-sliced register path
constexpr int kPlanes = 8;             // bit planes for counters <= 255
constexpr int kSmallRow = 64;          // incidence rows up to this length sort in-thread
constexpr int kNumXcd = 8;             // MI355X: 8 XCDs, each with its own L2
constexpr int kLdsHistEntries = 2048;  // per-workgroup LDS gain histogram (k * buckets)
constexpr int kSelectGrid = 2048;      // persistent workgroups of the select sweep
constexpr int kFinalizeGrid = 4096;    // persistent workgroups of the finalize sweep

// Validation bits raised on the device.
enum : int {
  kErrCsr = 1,         // eptr not increasing / wrong ends
  kErrPin = 2,         // pin outside [0,n)
  kErrWeight = 4,      // non-positive weight
  kErrDuplicate = 8,   // a vertex twice in one net
  kErrPart = 16,       // partition id outside [0,k)
  kErrNetWeight = 32,  // total net weight >= 2^31
  kErrMoves = 64,      // a move sequence names a vertex twice, a bad target or its own block
  kErrCluster = 128,   // cluster id outside [0,n)
  kErrClusterWeight = 256,  // a cluster weighs 2^31 or more
};

// Same-address global atomics serialize (tens of ns each), so every
// accumulator that many workgroups add to is split into kSlots partial sums
// (workgroup b adds to slot b % kSlots) and the partials are summed once by a
// single small kernel.  Histograms get one replica per XCD.
constexpr int kSlots = 64;
constexpr int kHistReplicas = kNumXcd;

enum CounterId : int {
  kCtrEligible = 0,
  kCtrBoundary,
  kCtrCandidates,
  kCtrApproved,
  kCtrMovedPins,
  kCtrDeltaAttr,    // two's complement int64 sums
  kCtrDeltaCheck,
  kCtrActivePins,
  kCtrTouched,
  kCtrMarked,       // approved moves marked for a monotone round (before the prefix cut)
  kCtrTouchedPins,  // sum of |e| over touched nets
  kNumCounters
};

// Per-round counters kept in the workspace.  Zero between rounds.
struct RoundCounters {
  unsigned long long slot[kNumCounters][kSlots];
  unsigned int any_overflow;       // some block's threshold fell into the ">=255" bucket
  unsigned int pad;
  long long max_block_w;           // late rounds: the finalize's, for the record
  unsigned int pad2[60];
};

// Units of `per` items that cover `items` items (counts may lie just below 2^31, so
// no sum of them is made in 32 bits).
__host__ __device__ inline int units_of(long long items, int per) {
  return (int)((items + per - 1) / per);
}

// Approval threshold of one target block.
struct Threshold {
  int gstar;          // gains > gstar approved; == gstar decided by vertex order; -1: all approved
  int tau;            // tile holding the last approved vertex of gain gstar (numTiles: none)
  long long rem;      // budget left for gain-gstar candidates after all higher gains
  long long rem_tile; // budget left inside tile tau
};

// Rounds of one small graph leave out two launches that have next to nothing to
// do: every tile-sum workgroup finds the thresholds of all k blocks itself, every
// approve workgroup scans their tile sums (one wavefront covers kBriefTiles in one
// step).  Both grow with n and k, the launches do not.  Five rounds, us, with the
// launches and without: a recorded refinement of n = 65,536 k = 2 180 / 167, k = 16 194
// / 191; n = 98,304 k = 8 199 / 194, k = 16 205 / 207; n = 131,072 k = 2 199 / 197,
// k = 8 210 / 212, but k = 16 214 / 226; single rounds, which the host launches,
// n = 131,072 k = 2 237 / 223, k = 8 243 / 237, k = 16 247 / 248.  Heavy vertices need
// the separate threshold (k_overflow_resolve).
constexpr int kBriefTiles = 256;
constexpr int kBriefMaxK = 16;
inline int brief_max_n(int k) { return k <= 8 ? 131072 : k <= kBriefMaxK ? 98304 : 0; }
static_assert(131072 <= kBriefTiles * kTile, "one step");
inline bool brief_rounds(int n, int k, int heavy_count) {
  return n <= brief_max_n(k) && heavy_count == 0;
}

// Facts gathered at load time (device side, copied to the host once).
struct LoadInfo {
  int err;
  int max_degree;
  int max_net_size;
  int max_incident_weight;
  int max_vertex_weight;
  int heavy_count;
  unsigned long long total_vertex_weight;
  unsigned long long total_net_weight;
  int big_rows;       // incidence rows longer than kSmallRow
  unsigned max_bucket;  // most pins in one vertex range of the transpose (LoadSplit)
  unsigned long_count;  // nets of more than kWaveNet pins
  int pad[3];
};

// One load workgroup's share of the LoadInfo maxima and sums; the load folds
// them into LoadInfo with one small kernel instead of one atomic per
// workgroup on the same words.
constexpr int kLoadGrid = 1024;   // workgroups of the load's sweeps
struct LoadPart {
  unsigned long long total_net_weight, total_vertex_weight;
  int max_net_size, max_vertex_weight, max_degree, max_incident_weight;
};

// Everything a kernel needs about one instance: a loaded hypergraph, its
// workspace, and one k-way partition state.  Single-instance entry points pass
// one by value inside the kernel arguments; batched launches pass a device
// array and a per-workgroup work table.
struct InstDesc {
  int n, m;
  int k, rw, view, unit_nets;
  int cmax, lds_buckets, heavy_count, num_tiles;
  int hist_stride;               // k_max * kBuckets: distance between histogram replicas
  int hist_reps;                 // histogram replicas in use (workgroup b adds to b % hist_reps)
  int sweep;                     // NetView that the select reads: view, or sview's kind
  int kept;                      // part8 follows part: this call counted the pins and runs the rounds
  int round_base;                // round r's record goes to stats[r - round_base]
  int long_count;                // nets of more than kWaveNet pins, in long_list
  long long P, lmax;
  const long long* eptr;
  const int* pins;
  const int* vwgt;
  const int* ewgt;
  const long long* vptr;
  const int* vnets;
  const int* heavy_list;
  const int* long_list;
  int* part;
  int* phi;
  unsigned* netstate;
  unsigned* view_ptr;            // compact Lambda/S copy (behind the records)
  unsigned char* sview;          // narrower copy kept by refine calls in the workspace; null: none
  long long* block_w;
  unsigned char* eligible;
  unsigned char* moved;          // may be null
  long long* km1;
  hg_round_stats* stats;
  long long* cand;
  unsigned char* touched;
  unsigned long long* hist;
  int* overflow;
  Threshold* thr;
  long long* tilesum;
  RoundCounters* ctr;
  // Late rounds (refine calls): the finalize folds the block weights, and round
  // r's record is written beside round r + 1's thresholds instead of by a launch
  // of its own, from the other of two sets of counters.
  int late;
  RoundCounters* prev;           // the round before's counters, to be recorded; null: none
  int* err_flags;
  unsigned long long* red;
  long long* bw_slots;           // kSlots x k block-weight deltas of a round's moves
  unsigned char* part8;          // packed copy of part: 4 bits a vertex for k <= 16, else 8
  unsigned char* appr;           // monotone rounds: approve marks moves here instead of applying
  int4* seq_cell;                // monotone rounds: per (net, block) cells the marking sets empty
  int* cache;                    // gain cache (b[n], w(I)[n], p[n*k]); null: none
};

// One workgroup's share of a batched launch: instance, and the units it
// handles: first, first + stride, ... (count of them).  What a unit is
// depends on the kernel (a 256-vertex chunk, a target block, a tile, ...).
struct WorkItem {
  int inst, first, count, stride;
};

// Kernel argument: a batch (descs + items, both device arrays) or one
// instance by value (descs == nullptr; each kernel then derives its units
// from blockIdx as documented with it).
//
// In a batch the items are either one per workgroup (split == 0) or grouped
// by XCD (split == 1): workgroup b runs on XCD b % 8 and takes item
// b / 8 of that XCD's queue items[xoff[x] .. xoff[x+1]), or nothing once the
// queue is used up.  Grouping keeps an instance's sweep on the XCD (and L2)
// it was placed on.
struct Launch {
  const InstDesc* descs;
  const WorkItem* items;
  int round;                     // round record index: stats + round (k_round_stats)
  int split;
  int xoff[kNumXcd + 1];
  int kept;                      // batch: InstDesc::kept of every member (0: nor is sview)
  InstDesc one;
};

// This workgroup's work item; `fallback` in single-instance mode.  An empty
// item (count == 0) means: nothing to do.
__device__ __forceinline__ WorkItem work_item(const Launch& L, WorkItem fallback) {
  if (!L.items) return fallback;
  if (!L.split) return L.items[blockIdx.x];
  const int x = (int)(blockIdx.x % kNumXcd);
  const int o = L.xoff[x] + (int)(blockIdx.x / kNumXcd);
  if (o >= L.xoff[x + 1]) {
    WorkItem w;
    w.inst = 0;
    w.first = 0;
    w.count = 0;
    w.stride = 1;
    return w;
  }
  return L.items[o];
}

__device__ __forceinline__ InstDesc inst_desc(const Launch& L, int inst) {
  if (!L.descs) return L.one;
  InstDesc d = L.descs[inst];
  d.kept = L.kept;
  if (!L.kept) d.sweep = d.view;
  return d;
}

// XCD-aware strided split of `units` over `grid` workgroups: XCD x owns the
// contiguous range [x*per_xcd, (x+1)*per_xcd) and its workgroups take
// neighbouring units side by side.
__device__ __forceinline__ WorkItem xcd_sweep(long long units) {
  const int xcd = blockIdx.x % kNumXcd;
  const int wg_on_xcd = (gridDim.x - xcd + kNumXcd - 1) / kNumXcd;
  const int li = blockIdx.x / kNumXcd;
  const long long per_xcd = (units + kNumXcd - 1) / kNumXcd;
  const long long c_begin = xcd * per_xcd;
  long long c_end = c_begin + per_xcd;
  if (c_end > units) c_end = units;
  WorkItem w;
  w.inst = 0;
  w.first = (int)(c_begin + li);
  w.stride = wg_on_xcd;
  w.count = c_begin + li < c_end ? (int)((c_end - (c_begin + li) + wg_on_xcd - 1) / wg_on_xcd) : 0;
  return w;
}

// Launch argument for one instance (kernels take their units from blockIdx).
inline Launch single_launch(const InstDesc& d) {
  Launch L;
  L.descs = nullptr;
  L.items = nullptr;
  L.round = 0;
  L.split = 0;
  for (int x = 0; x <= kNumXcd; ++x) L.xoff[x] = 0;
  L.kept = d.kept;
  L.one = d;
  return L;
}

// The transpose by vertex ranges (hg_load.hip): the pins are split into
// `coarse` ranges of 64 buckets, these into buckets of 2^shift vertices, and
// one workgroup turns a bucket into finished incidence rows in LDS.
constexpr int kPartTile = 8192;      // pins per tile of the two splits
constexpr int kPartGrid = 512;       // persistent workgroups of the first split
constexpr int kMaxBuckets = 8192;
constexpr int kFinePer = 64;         // buckets per coarse range
constexpr int kMaxCoarse = kMaxBuckets / kFinePer;
constexpr int kMaxShift = 10;        // a bucket holds at most 2^10 vertices
constexpr int kBucketCap = 10240;    // pins that a bucket's LDS rows hold
struct LoadSplit {
  int shift;      // vertices per bucket = 1 << shift; -1: sort by radix passes
  int buckets, coarse, tiles, grid;
};
LoadSplit load_split(int n, long long P);

struct WsLayout {
  size_t cand, touched, heavy, big, hist, overflow, thr, tilesum, ctr, info, scan, flags;
  size_t red;   // kSlots partial sums for whole-array reductions (km1)
  size_t bw_slots;   // kSlots x k_max block-weight deltas (apply), folded in by the round record
  size_t part8;      // up to n bytes: the partition in 4 or 8 bits a vertex (pin-count gathers)
  size_t lkey[2], lval, lhist, ldtot;   // load only: radix-sort buffers of the transpose
  size_t lpart;      // load only: per-workgroup partial facts (LoadPart[kLoadGrid])
  // inside others (see ws_layout)
  size_t lbase;      // load only: bucket starts and write cursors (LoadSplit)
  size_t ctr2;       // late rounds: the second set of counters
  size_t longs;      // the nets of more than kWaveNet pins
  size_t total;
  int num_tiles;
  int scan_blocks;
};

WsLayout ws_layout(int n, int m, long long P, int k_max);

// Touched-net flags: one byte per net, zero past m up to whole chunks of
// 1024 nets, so that the sweep reads its chunks of 256 without bounds tests.
inline size_t touched_bytes(int m) { return (((size_t)m + 1023) / 1024) * 1024; }

// 32-bit words per block bitset in a net record: ceil(k/32) rounded up to a
// power of two (1, 2, 4 or 8), so that word offsets are compile-time friendly.
__host__ __device__ inline int bit_words(int k) {
  int w = 1;
  while (w * 32 < k) w *= 2;
  return w;
}

// Compact per-net view read by the select and gain sweeps when every net
// weight is 1 and k <= 64: only the Lambda and S bitsets, packed into 4, 8 or
// 16 bytes (w(e) = 1 is implied and lambda(e) = popcount(Lambda)).  With k <=
// 16 a million nets take 4 MB, one XCD's L2.  kViewFull means the sweeps read
// the full net record instead.
// kViewUnit: full records (k > 64), every net weight 1.  kView8 and kView4
// (k <= 8 and k <= 4: 2 and 1 bytes a net) are never part of a net-state array:
// a call that counts the pins itself and then runs rounds keeps them in the
// workspace (see sweep_view).
enum NetView : int {
  kViewFull = 0, kView16 = 1, kView32 = 2, kView64 = 3, kViewUnit = 4, kView8 = 5, kView4 = 6
};

__host__ __device__ inline int net_view(int k, bool unit_nets) {
  if (!unit_nets) return kViewFull;
  if (k <= 16) return kView16;
  if (k <= 32) return kView32;
  if (k <= 64) return kView64;
  return kViewUnit;
}

// The copy that a refine call keeps for its select sweeps, or `view` itself.
inline int sweep_view(int view, int k, bool batch) {
  return view != kView16 ? view : k <= 4 && !batch ? kView4 : k <= 8 ? kView8 : kView16;
}

__host__ __device__ inline int view_bytes(int view) {
  return view == kView16 ? 4 : view == kView32 ? 8 : view == kView64 ? 16 : 0;
}

// 32-bit words per net reserved for the compact view in a net-state array
// (present for every k <= 64; maintained only for unit net weights).
__host__ __device__ inline int view_words(int k) {
  return k <= 16 ? 1 : k <= 32 ? 2 : k <= 64 ? 4 : 0;
}

// Words per net record: 2 + 2 * bit_words(k) rounded up to a power of two.
__host__ __device__ inline int net_words(int k) {
  if (k < 2 || k > HG_MAX_K) return 0;
  int need = 2 + 2 * bit_words(k);
  int rw = 4;
  while (rw < need) rw *= 2;
  return rw;
}

}  // namespace hg

struct hg_graph_s {
  int n, m;
  long long P;
  const long long* eptr;
  const int* pins;
  const int* vwgt;   // may be null (unit)
  const int* ewgt;   // may be null (unit)
  long long* vptr;
  int* vnets;
  char* ws;
  size_t ws_bytes;
  int k_max;
  bool unit_nets;    // every net weight is 1 (the compact net view is maintained)
  hg::WsLayout lay;
  hg::LoadInfo info;
  // recorded refinement graph (hipGraphExec_t) and the private stream it is
  // captured on (the caller's stream may be the legacy null stream)
  void* graph_exec;
  void* cap_stream;
  unsigned long long graph_key[12];
  // optional per-phase timing of label-propagation rounds (see hg_timing_*)
  int timing;
  void* timing_state;
};

namespace hg {

// ---- error reporting (hg_last_error) ----
hg_status fail(hg_status code, const char* fmt, ...);
size_t moves_workspace_size(long long n, long long m, int k);
size_t rebalance_workspace_size(long long n, int k);
size_t contract_workspace_size(long long n, long long m, long long P);
hg_status hip_fail(hipError_t e, const char* what);
hg_status check_k(hg_graph_s* g, int k);

#define HG_TRY(expr, what)                               \
  do {                                                   \
    hipError_t _e = (expr);                              \
    if (_e != hipSuccess) return hg::hip_fail(_e, what); \
  } while (0)

// ---- launch helpers implemented in the .hip files (return hipError_t) ----
// Up to kZeroRanges byte ranges of device memory, cleared by one launch of
// zero_ranges (add() ignores empty ranges; more than kZeroRanges is a bug).
constexpr int kZeroRanges = 8;
struct ZeroRanges {
  unsigned char* p[kZeroRanges];
  long long bytes[kZeroRanges];
  int count = 0;
  void add(void* ptr, long long nbytes);
};
hipError_t zero_ranges(const ZeroRanges& R, hipStream_t s);

hipError_t fill_i64(long long* p, long long v, long long count, hipStream_t s);
hipError_t fill_u8(unsigned char* p, unsigned char v, long long count, hipStream_t s);
hipError_t fill_i32(int* p, int v, long long count, hipStream_t s);

hipError_t load_check(hg_graph_s* g, hipStream_t s);
hipError_t load_build(hg_graph_s* g, hipStream_t s);
hipError_t list_long_nets(hg_graph_s* g, hipStream_t s);   // after load_build

// Gain cache (int32): b(u) at [u], w(I(u)) at [n + u], and the penalty row
// p_0(u) .. p_{k-1}(u) at [cache_pbase(n) + u * cache_stride(k)], rows padded
// to whole 16-byte quads.
__host__ __device__ inline long long cache_pbase(long long n) { return (2 * n + 3) & ~3LL; }
__host__ __device__ inline int cache_stride(int k) { return (k + 3) & ~3; }

// Gain-histogram buckets kept in LDS per target block by the select sweep.
inline int lds_buckets(int k) {
  int b = kBuckets;
  while (b > 1 && b * k > kLdsHistEntries) b >>= 1;
  return b;
}

// Descriptor of one instance: graph g, its workspace, and the caller's state.
InstDesc make_desc(hg_graph_s* g, int k, long long lmax, int* part, int* phi,
                   unsigned* netstate, long long* block_w, unsigned char* eligible,
                   unsigned char* moved, long long* km1, hg_round_stats* stats);
void keep_private_copies(hg_graph_s* g, InstDesc& d, bool batch);

}  // namespace hg
