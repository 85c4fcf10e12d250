// hg_load.hip -- input checks, incidence CSR (transpose of the net CSR) and
// static per-vertex facts.  Runs once per loaded hypergraph.
//
// The paper stores a hypergraph as two adjacency arrays, the pins of each net
// and the incident nets of each vertex (section "Coarsening", subsection
// "Contraction").  Here the second array is built on the device, I(v) listing
// nets in increasing id: the (pin, net) pairs are split by vertex range in two
// passes and finished in LDS, or, where a range would not fit, stably
// radix-sorted by pin.
#include "hg_device.h"
#include "hg_internal.h"
#include "hg_sort.h"

namespace hg {

// ------------------------------------------------------------------ fills
__global__ void k_fill_i64(long long* p, long long v, long long count) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long stride = (long long)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}
__global__ void k_fill_i32(int* p, int v, long long count) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long stride = (long long)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}
__global__ void k_fill_u8(unsigned char* p, unsigned char v, long long count) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long stride = (long long)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}

// Byte ranges cleared by one launch: each range's unaligned head and tail
// byte by byte, its middle in 16-byte stores.  One launch instead of one per
// range matters where a call clears many small arrays (a few microseconds
// of launch each).
__global__ void k_zero_ranges(ZeroRanges R) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (int r = 0; r < R.count; ++r) {
    unsigned char* p = R.p[r];
    const long long bytes = R.bytes[r];
    long long head = (long long)((16 - ((uintptr_t)p & 15)) & 15);
    if (head > bytes) head = bytes;
    const long long words = (bytes - head) / 16;
    const long long tail = head + words * 16;
    for (long long i = tid; i < head; i += stride) p[i] = 0;
    int4* w = reinterpret_cast<int4*>(p + head);
    for (long long i = tid; i < words; i += stride) w[i] = make_int4(0, 0, 0, 0);
    for (long long i = tail + tid; i < bytes; i += stride) p[i] = 0;
  }
}

static unsigned grid_for(long long count, int per_thread = 1) {
  long long blocks = (count + (long long)kBlock * per_thread - 1) / ((long long)kBlock * per_thread);
  if (blocks < 1) blocks = 1;
  if (blocks > 65536) blocks = 65536;
  return (unsigned)blocks;
}

hipError_t fill_i64(long long* p, long long v, long long count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(count)), dim3(kBlock), 0, s, p, v, count);
  return hipGetLastError();
}
hipError_t fill_i32(int* p, int v, long long count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(count)), dim3(kBlock), 0, s, p, v, count);
  return hipGetLastError();
}
void ZeroRanges::add(void* ptr, long long nbytes) {
  if (nbytes <= 0) return;
  if (count == kZeroRanges) __builtin_trap();   // a caller listed too many ranges
  p[count] = (unsigned char*)ptr;
  bytes[count] = nbytes;
  ++count;
}

hipError_t zero_ranges(const ZeroRanges& R, hipStream_t s) {
  long long most = 0;
  for (int r = 0; r < R.count; ++r) most = R.bytes[r] > most ? R.bytes[r] : most;
  if (most == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_ranges, dim3(grid_for(most, 16)), dim3(kBlock), 0, s, R);
  return hipGetLastError();
}

hipError_t fill_u8(unsigned char* p, unsigned char v, long long count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u8, dim3(grid_for(count)), dim3(kBlock), 0, s, p, v, count);
  return hipGetLastError();
}

// ------------------------------------------------------------------ checks
// Load-time checks run on a capped grid (kLoadGrid) and reduce per
// workgroup into that workgroup's LoadPart; k_fold_load folds the parts.

__device__ __forceinline__ int block_max_int(int v, int* s_tmp) {
  v = wave_max(v);
  __syncthreads();
  if (lane_id() == 0) s_tmp[threadIdx.x / kWave] = v;
  __syncthreads();
  int r = s_tmp[0];
  for (int i = 1; i < kBlock / kWave; ++i) r = s_tmp[i] > r ? s_tmp[i] : r;
  return r;
}

// Nets: increasing offsets with fixed ends (no empty net), positive weights.  The net
// holding the first pin of every tile of kPartTile pins goes to tile_first
// (tile_first[tiles] = m - 1).  Vertices: positive weights.  (One launch: the second
// took longer to start than to run on small hypergraphs.)
__global__ __launch_bounds__(kBlock) void k_check(int m, long long P, const long long* eptr,
                                                  const int* ewgt, int n, const int* vwgt,
                                                  LoadInfo* info, LoadPart* part,
                                                  int* tile_first, int tiles) {
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ int s_imax[kBlock / kWave];
  int err = 0, size = 0, cmax = 0;
  long long wsum = 0, csum = 0;
  const long long stride = (long long)gridDim.x * kBlock;
  const long long at = (long long)blockIdx.x * kBlock + threadIdx.x;
  for (long long e = at; e < m; e += stride) {
    const long long s = eptr[e], t = eptr[e + 1];
    if (e == 0 && s != 0) err |= kErrCsr;
    if (e == m - 1 && t != P) err |= kErrCsr;
    if (t <= s || s < 0 || t > P) err |= kErrCsr;
    else {
      if (t - s > size) size = (int)((t - s) > 0x7fffffffLL ? 0x7fffffff : (t - s));
      // tiles whose first pin lies in [s, t), all below `tiles` as t <= P
      for (long long x = (s + kPartTile - 1) / kPartTile; x * kPartTile < t; ++x)
        tile_first[x] = (int)e;
      if (e == m - 1) tile_first[tiles] = m - 1;
    }
    const long long w = ewgt ? ewgt[e] : 1;
    if (w <= 0) err |= kErrWeight;
    else wsum += w;
  }
  for (long long v = at; v < n; v += stride) {
    const long long c = vwgt ? vwgt[v] : 1;
    if (c <= 0) {
      err |= kErrWeight;
    } else {
      csum += c;
      if (c > cmax) cmax = (int)c;
    }
  }
  if (err) atomicOr(&info->err, err);
  size = block_max_int(size, s_imax);
  cmax = block_max_int(cmax, s_imax);
  wsum = block_sum64(wsum, s_tmp);
  csum = block_sum64(csum, s_tmp);
  if (threadIdx.x == 0) {
    LoadPart& mine = part[blockIdx.x];
    mine.max_net_size = size;
    mine.total_net_weight = (unsigned long long)wsum;
    mine.total_vertex_weight = (unsigned long long)csum;
    mine.max_vertex_weight = cmax;
  }
}

// LoadInfo's maxima and sums from the workgroups' parts (one workgroup).  With
// `cbase` set it holds the pin count of every coarse range of the split and
// `cmost` their fullest buckets': the counts become the ranges' starts
// (cbase[coarse] = their sum) and the fullest bucket goes to LoadInfo.
__global__ __launch_bounds__(kBlock) void k_fold_load(const LoadPart* part, LoadInfo* info,
                                                      unsigned* cbase, const unsigned* cmost,
                                                      int coarse) {
  __shared__ long long s_tmp[kBlock / kWave];
  __shared__ int s_imax[kBlock / kWave];
  unsigned long long tnw = 0, tvw = 0;
  int mns = 0, mvw = 0, md = 0, miw = 0;
  for (int b = threadIdx.x; b < kLoadGrid; b += kBlock) {
    const LoadPart p = part[b];
    tnw += p.total_net_weight;
    tvw += p.total_vertex_weight;
    mns = p.max_net_size > mns ? p.max_net_size : mns;
    mvw = p.max_vertex_weight > mvw ? p.max_vertex_weight : mvw;
    md = p.max_degree > md ? p.max_degree : md;
    miw = p.max_incident_weight > miw ? p.max_incident_weight : miw;
  }
  tnw = (unsigned long long)block_sum64((long long)tnw, s_tmp);
  tvw = (unsigned long long)block_sum64((long long)tvw, s_tmp);
  mns = block_max_int(mns, s_imax);
  mvw = block_max_int(mvw, s_imax);
  md = block_max_int(md, s_imax);
  miw = block_max_int(miw, s_imax);
  if (cbase) {
    const int c = threadIdx.x;                          // coarse <= kMaxCoarse < kBlock
    const long long mine = c < coarse ? cbase[c] : 0;
    long long tot;
    const long long at = block_excl_scan64(mine, s_tmp, &tot);
    if (c <= coarse) cbase[c] = (unsigned)at;
    const int most = block_max_int(c < coarse ? (int)cmost[c] : 0, s_imax);
    if (c == 0) info->max_bucket = (unsigned)most;
  }
  if (threadIdx.x == 0) {
    info->total_net_weight = tnw;
    info->total_vertex_weight = tvw;
    info->max_net_size = mns;
    info->max_vertex_weight = mvw;
    info->max_degree = md;
    info->max_incident_weight = miw;
  }
}

static unsigned grid_cap_load(long long items) {
  long long b = (items + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > kLoadGrid) b = kLoadGrid;
  return (unsigned)b;
}

// The transpose's radix sort: long sorts in 8192-item tiles (fuller digit
// runs per tile; the netlist's 56.5M pairs sort 11% faster), shorter ones in
// 4096-item tiles (more workgroups: 7% faster on 10M pairs).
static bool long_load_sort(long long P) { return P >= (1LL << 24); }

static int pin_tiles(long long P) { return (int)((P + kPartTile - 1) / kPartTile); }
static_assert(kPartTile == kNetTile, "tiles of the sort's nets mode");

// The sort's first pass: the keys are the caller's pins, read in place.
static SortPass first_load_pass(hg_graph_s* g) {
  SortPass SP;
  SP.hist = (unsigned*)(g->ws + g->lay.lhist);
  SP.dtot = (unsigned*)(g->ws + g->lay.ldtot);
  SP.n = (int)g->P;
  SP.tiles = long_load_sort(g->P) ? sort_tiles<kSortPerLong>(g->P) : sort_tiles(g->P);
  SP.key_in = (const unsigned*)g->pins;
  SP.shift = 0;
  return SP;
}

// ------------------------------------------------------------------ vertex ranges
// The transpose by vertex ranges.  A pass of the radix sort moves 8-byte pairs
// in runs of about 32 and needs its own digit count; three of them, the pair
// expansion and the row starts took 1.36 ms on a netlist of 4M cells and 56.5M
// pins, for the 0.5 GB that the transpose has to read and write.  Here
//   1. one count of the pins per bucket (a range of 2^shift vertices) and
//      workgroup, which is also the pins' range check,
//   2. a split into coarse ranges of 64 buckets, the nets found on the way,
//   3. a split of every coarse range into its buckets; what is left of a pin
//      fits 16 bits,
//   4. per bucket one workgroup that places the nets in their rows in LDS,
//      sorts every row and writes row starts and rows.
// The splits need not be stable (rows are sorted last), so a pin's place in
// its tile is one LDS atomic, and the workgroups of the second split reserve
// their output by one global atomic per bucket and tile.  Rows are sets
// sorted by net id, so nothing depends on the order of arrival.
// Measured (all kernels of one load, radix passes and now): netlist 4M cells, 56.5M
// pins 1420 -> 590 to 695 us (count 64 to 78, coarse split 155 to 199, fine split 169
// to 207, rows 130, checks and facts 70; the 2.1 GB they move take 410 us at a large
// copy's 5.1 TB/s), matrix 1M x 1M, 10M pins 287 -> 152 us.

constexpr int kPartBlock = 1024;                       // threads of the split kernels
constexpr int kPartPer = kPartTile / kPartBlock;       // pins per thread and tile
constexpr int kRowsBlock = 512;                        // threads of a bucket's workgroup
constexpr int kRowsWaves = kRowsBlock / kWave;

// Buckets of at most 8192 pins on average (the LDS rows take kBucketCap, so
// even ranges fit; the count decides), as long as the ranges stay few enough
// for the tables: n > 8192 * 1024, or more than 8192 pins on average in the
// smallest allowed range, go to the radix sort, and so do hypergraphs whose
// count table would not fit the scratch of one word per pin (far fewer pins
// than vertices).
LoadSplit load_split(int n, long long P) {
  LoadSplit L;
  L.shift = -1;
  L.buckets = L.coarse = L.tiles = L.grid = 0;
  int shift = 0;
  while (shift < kMaxShift && (((long long)n - 1) >> shift) + 1 > kMaxBuckets) ++shift;
  if ((((long long)n - 1) >> shift) + 1 > kMaxBuckets) return L;
  if ((P << shift) / n > kPartTile) return L;
  // wider ranges while they stay light and either leave two workgroups per
  // compute unit or are not worth a workgroup yet
  while (shift < 9 && (P << (shift + 1)) / n <= kPartTile &&
         ((n >> (shift + 1)) >= 512 || (P << shift) / n < 512))
    ++shift;
  const int buckets = ((n - 1) >> shift) + 1;
  const int tiles = pin_tiles(P);
  const int grid = tiles < kPartGrid ? tiles : kPartGrid;
  if ((long long)grid * buckets > P) return L;
  L.shift = shift;
  L.buckets = buckets;
  L.coarse = (buckets + kFinePer - 1) / kFinePer;
  L.tiles = tiles;
  L.grid = grid;
  return L;
}

struct Split {
  int n, m, P;
  LoadSplit L;
  const int* pins;
  const long long* eptr;
  int* tile_first;        // [tiles + 1]
  unsigned* counts;       // [grid][buckets]
  unsigned* ccounts;      // [grid][coarse]: pins per range; then, of the workgroups before
  unsigned* cbase;        // [coarse + 1]: first pin of every range
  unsigned* cmost;        // [coarse]: pins of the range's fullest bucket
  unsigned* rel;          // [buckets]: first pin of every bucket in its range
  unsigned* cursor;       // [buckets]: write positions of the second split, likewise
  unsigned* cpin;         // [P]: pins by coarse range
  int* cnet;              // [P]
  unsigned short* low;    // [P]: pin & (2^shift - 1) by bucket
  int* val;               // [P]: the nets, by bucket (in the rows' own array)
  LoadInfo* info;
  long long* vptr;
};

// Tiles [first, last) of persistent workgroup w.
__device__ __forceinline__ void split_tiles(const Split& S, int w, int& first, int& last) {
  const int per = S.L.tiles / S.L.grid, rem = S.L.tiles % S.L.grid;
  first = w * per + (w < rem ? w : rem);
  last = first + per + (w < rem ? 1 : 0);
}

// Pins per bucket of this workgroup's tiles, and the range check.
__global__ __launch_bounds__(kPartBlock) void k_split_count(Split S) {
  __shared__ unsigned s_cnt[kMaxBuckets];
  for (int i = threadIdx.x; i < S.L.buckets; i += kPartBlock) s_cnt[i] = 0;
  __syncthreads();
  int first, last;
  split_tiles(S, blockIdx.x, first, last);
  bool bad = false;
  for (int t = first; t < last; ++t) {
    const long long base = (long long)t * kPartTile;
    unsigned v[kPartPer];
#pragma unroll
    for (int r = 0; r < kPartPer; ++r) {
      const long long i = base + r * kPartBlock + threadIdx.x;
      v[r] = i < S.P ? (unsigned)S.pins[i] : 0xffffffffu;
    }
#pragma unroll
    for (int r = 0; r < kPartPer; ++r) {
      if (v[r] < (unsigned)S.n)
        atomicAdd(&s_cnt[v[r] >> S.L.shift], 1u);
      else
        bad |= base + r * kPartBlock + threadIdx.x < S.P;
    }
  }
  if (bad) atomicOr(&S.info->err, kErrPin);
  __syncthreads();
  unsigned* row = S.counts + (size_t)blockIdx.x * S.L.buckets;
  for (int i = threadIdx.x; i < S.L.buckets; i += kPartBlock) row[i] = s_cnt[i];
  const int lane = lane_id();
  for (int c = threadIdx.x / kWave; c < S.L.coarse; c += kPartBlock / kWave) {
    const int i = c * kFinePer + lane;                 // kFinePer == kWave
    const unsigned all = wave_sum(i < S.L.buckets ? s_cnt[i] : 0u);
    if (lane == 0) S.ccounts[(size_t)blockIdx.x * S.L.coarse + c] = all;
  }
}
static_assert(kFinePer == kWave, "a wavefront sums a range's buckets");

// One workgroup per coarse range: its buckets' starts, the range's total (to
// cbase, which k_fold_load turns into starts), and for every counting
// workgroup the pins of the range that the ones before it hold.
constexpr int kSplitScanBlock = 1024;

__global__ __launch_bounds__(kSplitScanBlock) void k_split_scan(Split S) {
  constexpr int kRowsAt = kSplitScanBlock / kWave;     // table rows read at a time
  constexpr int kRows = kPartGrid / kRowsAt;
  __shared__ unsigned s_col[kRowsAt][kWave];
  const int wv = threadIdx.x / kWave, lane = lane_id();
  const int col = blockIdx.x * kFinePer + lane;
  const bool in = col < S.L.buckets;
  unsigned c[kRows];                                   // every row requested before the first wait
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int w = wv + q * kRowsAt;
    c[q] = in && w < S.L.grid ? S.counts[(size_t)w * S.L.buckets + col] : 0u;
  }
  unsigned sum = 0;
#pragma unroll
  for (int q = 0; q < kRows; ++q) sum += c[q];
  s_col[wv][lane] = sum;
  __syncthreads();
  if (wv == 0) {
    unsigned tot = 0;
    for (int q = 0; q < kRowsAt; ++q) tot += s_col[q][lane];
    const unsigned before = (unsigned)wave_incl_scan((int)tot) - tot;
    if (in) S.rel[col] = S.cursor[col] = before;
    const unsigned most = (unsigned)wave_max((int)tot);
    if (lane == kWave - 1) {
      S.cbase[blockIdx.x] = before + tot;
      S.cmost[blockIdx.x] = most;
    }
  } else if (wv == 1) {
    unsigned x[kPartGrid / kWave];
#pragma unroll
    for (int q = 0; q < kPartGrid / kWave; ++q) {
      const int w = q * kWave + lane;
      x[q] = w < S.L.grid ? S.ccounts[(size_t)w * S.L.coarse + blockIdx.x] : 0u;
    }
    unsigned carry = 0;
#pragma unroll
    for (int q = 0; q < kPartGrid / kWave; ++q) {
      const int w = q * kWave + lane;
      const unsigned incl = (unsigned)wave_incl_scan((int)x[q]);
      if (w < S.L.grid) S.ccounts[(size_t)w * S.L.coarse + blockIdx.x] = carry + incl - x[q];
      carry += (unsigned)__shfl((int)incl, kWave - 1);
    }
  }
}

// First pin of bucket b, and of the one after it.
__device__ __forceinline__ unsigned bucket_start(const Split& S, int b) {
  return S.cbase[b / kFinePer] + S.rel[b];
}
__device__ __forceinline__ unsigned bucket_end(const Split& S, int b) {
  return b + 1 == S.L.buckets || (b + 1) % kFinePer == 0 ? S.cbase[b / kFinePer + 1]
                                                        : bucket_start(S, b + 1);
}

// Exclusive prefix of cnt[0 .. 128) into off, by the first wave (two entries
// per lane); returns nothing, the caller synchronizes.
__device__ __forceinline__ void scan_counts(const unsigned* cnt, unsigned* off, int count) {
  if (threadIdx.x < kWave) {
    const int i0 = 2 * threadIdx.x;
    const int a = i0 < count ? (int)cnt[i0] : 0, b = i0 + 1 < count ? (int)cnt[i0 + 1] : 0;
    const int incl = wave_incl_scan(a + b);
    if (i0 < count) off[i0] = (unsigned)(incl - a - b);
    if (i0 + 1 < count) off[i0 + 1] = (unsigned)(incl - b);
  }
}

// Place of this lane's item among the items of its key: one LDS atomic per
// run of equal keys in neighbouring lanes (the pins of a net, listed in
// order, mostly fall in one range: with one atomic per lane a wavefront's
// adds to that range's word took 64 turns).  Every lane of the wave calls.
__device__ __forceinline__ unsigned run_rank(unsigned* cnt, unsigned key, bool live) {
  const int lane = lane_id();
  const unsigned k = live ? key : 0xffffffffu;
  const unsigned prev = lane_before(k);
  const unsigned long long heads = __ballot(lane == 0 || k != prev);
  const unsigned long long upto = ~0ull >> (kWave - 1 - lane);
  const int head = kWave - 1 - __clzll((long long)(heads & upto));
  const unsigned long long later = heads & ~upto;
  unsigned at = 0;      // netlist: coarse split 335 -> 307, fine split 256 -> 197 us
  if (live && head == lane) {
    const int end = later ? __ffsll((long long)later) - 1 : kWave;
    at = atomicAdd(&cnt[k], (unsigned)(end - lane));
  }
  return (unsigned)__shfl((int)at, head) + (unsigned)(lane - head);
}

// First split: (pin, net) pairs by coarse range.  The pairs are staged in LDS
// in range order (pins, then nets in the same words) so that a tile's run of
// a range leaves as consecutive addresses.
struct CoarseLds {
  unsigned stage[kPartTile];
  unsigned long long start[kPartTile / 64];   // one bit per net start
  unsigned before[kPartTile / 64];            // net starts before the word
  unsigned cur[kMaxCoarse], cnt[kMaxCoarse], off[kMaxCoarse];
};

// One tile of `here` pins (FULL: kPartTile; without the bounds tests the
// registers of eight pins fit and the netlist's split takes 198, not 307 us).
template <bool FULL>
__device__ __forceinline__ void split_coarse_tile(const Split& S, CoarseLds& M, int t, int here) {
  const int C = S.L.coarse, shift = S.L.shift + 6;         // 64 = kFinePer buckets a range
  const long long base = (long long)t * kPartTile;
  const int* pins = S.pins + base;
  const int wv = threadIdx.x / kWave, lane = lane_id();
  unsigned pin[kPartPer];
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int i = r * kPartBlock + threadIdx.x;
    pin[r] = FULL || i < here ? (unsigned)pins[i] : 0u;
  }
  const int net0 = S.tile_first[t], net1 = S.tile_first[t + 1];
  for (int c = threadIdx.x; c < C; c += kPartBlock) M.cnt[c] = 0;
  if (threadIdx.x < kPartTile / 64) M.start[threadIdx.x] = 0;
  __syncthreads();
  // nets (net0, net1] are the ones that can start inside the tile
  for (int e = net0 + 1 + (int)threadIdx.x; e <= net1; e += kPartBlock) {
    const long long at = S.eptr[e] - base;                 // > 0; past the tile for net1 only
    if (at < here) atomicOr(&M.start[at >> 6], 1ull << (at & 63));
  }
  unsigned slot[kPartPer];
#pragma unroll
  for (int r = 0; r < kPartPer; ++r)
    slot[r] = run_rank(M.cnt, pin[r] >> shift, FULL || r * kPartBlock + (int)threadIdx.x < here);
  __syncthreads();
  scan_counts(M.cnt, M.off, C);
  if (wv == 1) {
    const int c0 = __popcll(M.start[2 * lane]), c1 = __popcll(M.start[2 * lane + 1]);
    const int incl = wave_incl_scan(c0 + c1);
    M.before[2 * lane] = (unsigned)(incl - c0 - c1);
    M.before[2 * lane + 1] = (unsigned)(incl - c1);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    if (FULL || r * kPartBlock + (int)threadIdx.x < here) {
      slot[r] += M.off[pin[r] >> shift];
      M.stage[slot[r]] = pin[r];
    }
  }
  __syncthreads();
  unsigned dst[kPartPer];
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int j = r * kPartBlock + threadIdx.x;
    dst[r] = 0;
    if (FULL || j < here) {
      const unsigned v = M.stage[j], c = v >> shift;
      dst[r] = M.cur[c] + ((unsigned)j - M.off[c]);
      S.cpin[dst[r]] = v;
    }
  }
  __syncthreads();
  const unsigned long long upto = ~0ull >> (kWave - 1 - lane);
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    if (FULL || r * kPartBlock + (int)threadIdx.x < here) {
      const int word = r * (kPartBlock / kWave) + wv;      // this item's bit is the lane's
      M.stage[slot[r]] = (unsigned)net0 + M.before[word] + (unsigned)__popcll(M.start[word] & upto);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int j = r * kPartBlock + threadIdx.x;
    if (FULL || j < here) S.cnet[dst[r]] = (int)M.stage[j];
  }
  for (int c = threadIdx.x; c < C; c += kPartBlock) M.cur[c] += M.cnt[c];
  __syncthreads();
}

__global__ __launch_bounds__(kPartBlock, 8) void k_split_coarse(Split S) {
  __shared__ CoarseLds M;
  for (int c = threadIdx.x; c < S.L.coarse; c += kPartBlock)
    M.cur[c] = S.cbase[c] + S.ccounts[(size_t)blockIdx.x * S.L.coarse + c];
  int first, last;
  split_tiles(S, blockIdx.x, first, last);
  for (int t = first; t < last; ++t) {
    const long long left = S.P - (long long)t * kPartTile;
    if (left >= kPartTile)
      split_coarse_tile<true>(S, M, t, kPartTile);
    else
      split_coarse_tile<false>(S, M, t, (int)left);
  }
}

// A tile of `here` pairs (FULL: kPartTile, no bounds tests) from `from` on
// into the buckets of coarse range c, whose pins begin at `start`.
struct FineLds {
  unsigned stage[kPartTile];
  unsigned tiles[kMaxCoarse], first[kMaxCoarse];
  unsigned cnt[kFinePer], off[kFinePer], out[kFinePer];
};

template <bool FULL>
__device__ __forceinline__ void split_fine_tile(const Split& S, FineLds& M, int c, unsigned start,
                                                unsigned from, int here) {
  const int shift = S.L.shift;
  const unsigned* cpin = S.cpin + from;
  const int* cnet = S.cnet + from;
  unsigned pin[kPartPer], slot[kPartPer];
  int net[kPartPer];
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int i = r * kPartBlock + threadIdx.x;
    pin[r] = FULL || i < here ? cpin[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int i = r * kPartBlock + threadIdx.x;
    net[r] = FULL || i < here ? cnet[i] : 0;
  }
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    slot[r] = run_rank(M.cnt, (pin[r] >> shift) & (kFinePer - 1),
                       FULL || r * kPartBlock + (int)threadIdx.x < here);
  }
  __syncthreads();
  scan_counts(M.cnt, M.off, kFinePer);
  if (threadIdx.x >= kWave && threadIdx.x < kWave + kFinePer) {
    const int f = threadIdx.x - kWave;
    const unsigned k = M.cnt[f];
    M.out[f] = k ? start + atomicAdd(&S.cursor[c * kFinePer + f], k) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    if (FULL || r * kPartBlock + (int)threadIdx.x < here) {
      slot[r] += M.off[(pin[r] >> shift) & (kFinePer - 1)];
      M.stage[slot[r]] = pin[r];
    }
  }
  __syncthreads();
  unsigned dst[kPartPer];
  const unsigned mask = (1u << shift) - 1u;
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int j = r * kPartBlock + threadIdx.x;
    dst[r] = 0;
    if (FULL || j < here) {
      const unsigned v = M.stage[j], f = (v >> shift) & (kFinePer - 1);
      dst[r] = M.out[f] + ((unsigned)j - M.off[f]);
      S.low[dst[r]] = (unsigned short)(v & mask);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r)
    if (FULL || r * kPartBlock + (int)threadIdx.x < here) M.stage[slot[r]] = (unsigned)net[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int j = r * kPartBlock + threadIdx.x;
    if (FULL || j < here) S.val[dst[r]] = (int)M.stage[j];
  }
}

// Second split: a tile of one coarse range into the range's buckets.  The
// grid covers the tiles of all ranges (each range's last tile may be short).
__global__ __launch_bounds__(kPartBlock, 8) void k_split_fine(Split S) {
  __shared__ FineLds M;
  const int C = S.L.coarse;
  for (int c = threadIdx.x; c < C; c += kPartBlock)
    M.tiles[c] = (S.cbase[c + 1] - S.cbase[c] + kPartTile - 1) / kPartTile;
  if (threadIdx.x < kFinePer) M.cnt[threadIdx.x] = 0;
  __syncthreads();
  scan_counts(M.tiles, M.first, C);
  __syncthreads();
  const unsigned tile = blockIdx.x;
  if (tile >= M.first[C - 1] + M.tiles[C - 1]) return;     // whole workgroup
  int lo = 0, hi = C - 1;                                  // the last range starting at or before
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (M.first[mid] <= tile) lo = mid; else hi = mid - 1;
  }
  // ranges without a tile share their start with the next one, which the
  // search prefers, so `lo` owns the tile
  const unsigned start = S.cbase[lo], end = S.cbase[lo + 1];
  const unsigned from = start + (tile - M.first[lo]) * kPartTile;
  const int here = end - from < (unsigned)kPartTile ? (int)(end - from) : kPartTile;
  if (here == kPartTile)
    split_fine_tile<true>(S, M, lo, start, from, here);
  else
    split_fine_tile<false>(S, M, lo, start, from, here);
}

// Ascending sort of N (16 or 32) registers by Batcher's odd-even merge network.
template <int N>
__device__ __forceinline__ void sort_regs(int (&x)[N]) {
#pragma unroll
  for (int p = 1; p < N; p <<= 1) {
#pragma unroll
    for (int q = p; q >= 1; q >>= 1) {
#pragma unroll
      for (int j = q % p; j + q < N; j += 2 * q) {
#pragma unroll
        for (int i = 0; i < q; ++i) {
          if (i + j + q < N && (i + j) / (2 * p) == (i + j + q) / (2 * p)) {
            const int a = x[i + j], b = x[i + j + q];
            x[i + j] = a < b ? a : b;
            x[i + j + q] = a < b ? b : a;
          }
        }
      }
    }
  }
}

// A row of d <= N nets in LDS sorted by one thread; true if a net repeats.
template <int N>
__device__ __forceinline__ bool sort_row(int* row, int d) {
  int x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = i < d ? row[i] : 0x7fffffff;
  sort_regs<N>(x);
  bool dup = false;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i < d) row[i] = x[i];
    if (i > 0) dup |= i < d && x[i] == x[i - 1];
  }
  return dup;
}

constexpr int kWaveRow = 128;                            // longest row of one wavefront
constexpr int kBigRows = kBucketCap / (kWaveRow + 1) + 1;

// A bucket's rows of more than kWaveRow nets, as many together as the bits of a word
// can tell apart (32 and more): (row, net) words, each thread's in registers.  A
// word's place is guessed from the row's length, as if its nets were spread evenly;
// words of neighbouring places share a bin of kBinPlaces, a thread sorts a bin
// (spread_big_rows).  Where a bin overflows, the words are sorted by radix passes
// (radix_big_rows), bound by the chain of a wavefront's groups of 64 through its
// digit counters.  (Row after row by a bitonic sort, a load of 100,000 vertices took
// 304 us with 15 vertices in 600 nets each, 286 with one in 9,500; by radix passes
// 138 and 151, 131 and 140 so; 104 without such rows, about 160 by radix passes over
// all pins.  Ranked by a wavefront each, 18 rows of 450 nets made a load of 120 us
// one of 320.)
struct BigRows {
  unsigned short row[kBigRows];                          // the rows
  unsigned at[kBigRows + 1];                             // first word of each
};

template <int PER>
struct RowWords {
  unsigned word[PER];
  int per;                                               // in use: a wave holds per * kWave words
};

__device__ __forceinline__ int word_at(int per, int r) {
  return ((int)(threadIdx.x / kWave) * per + r) * kWave + lane_id();
}

// The T words of rows [first, last) of B, from the unsorted rows.  Every thread calls.
template <int PER>
__device__ __forceinline__ void load_big_rows(RowWords<PER>& W, const BigRows& B, int first,
                                              int last, int T, const int* rows,
                                              const unsigned* start, int net_bits) {
  W.per = (T + kRowsBlock - 1) / kRowsBlock;
  const int zero = (int)B.at[first];
  // a group of 64 words lies in at most two rows
  int i = first;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    W.word[r] = 0xffffffffu;
    if (r < W.per) {
      const int base = word_at(W.per, r) - lane_id();
      while (i + 1 < last && (int)B.at[i + 1] - zero <= base) ++i;
      const int p = base + lane_id();
      if (p < T) {
        const int mine = i + (i + 1 < last && (int)B.at[i + 1] - zero <= p ? 1 : 0);
        W.word[r] = ((unsigned)(mine - first) << net_bits) |
                    (unsigned)rows[start[B.row[mine]] + (unsigned)(p + zero) - B.at[mine]];
      }
    }
  }
}

// Sorts them into `sorted`.  cnt: [kRowsWaves][256], wsum: [kRowsWaves], of LDS.
template <int PER>
__device__ __forceinline__ void radix_big_rows(RowWords<PER>& W, int T, int bits, unsigned* sorted,
                                              unsigned short* cnt, unsigned* wsum) {
  const int wv = threadIdx.x / kWave, lane = lane_id(), tid = threadIdx.x;
  unsigned short* mine = cnt + wv * kDigits;
  // passes of equal width
  const int passes = (bits + 7) / 8, width = (bits + passes - 1) / passes;
  const unsigned mask = (1u << width) - 1u;
  for (int shift = 0; shift < bits; shift += width) {
    for (int i = lane; i < kDigits; i += kWave) mine[i] = 0;
    wave_lds_sync();
    unsigned short off[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (r >= W.per) break;
      const bool live = word_at(W.per, r) < T;
      const unsigned d = (W.word[r] >> shift) & mask;
      unsigned long long peers = __ballot(live);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        if (bit >= width) break;
        const unsigned long long ones = __ballot((d >> bit) & 1u);
        peers &= (d >> bit) & 1u ? ones : ~ones;
      }
      const unsigned before = mine[d];
      const int rank = lanes_below(peers, 0);
      wave_lds_sync();
      if (live && rank == 0) mine[d] = (unsigned short)(before + (unsigned)__popcll(peers));
      wave_lds_sync();
      off[r] = (unsigned short)(before + (unsigned)rank);
    }
    __syncthreads();
    // counts -> the first place of every wave's words of every digit
    unsigned all = 0, incl = 0;
    if (tid < kDigits) {
      for (int w = 0; w < kRowsWaves; ++w) all += cnt[w * kDigits + tid];
      incl = (unsigned)wave_incl_scan((int)all);
      if (lane == kWave - 1) wsum[wv] = incl;
    }
    __syncthreads();
    if (tid < kDigits) {
      unsigned at = incl - all;
      for (int w = 0; w < wv; ++w) at += wsum[w];
      for (int w = 0; w < kRowsWaves; ++w) {
        const unsigned c = cnt[w * kDigits + tid];
        cnt[w * kDigits + tid] = (unsigned short)at;
        at += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (r >= W.per) break;
      if (word_at(W.per, r) < T)
        sorted[mine[(W.word[r] >> shift) & mask] + off[r]] = W.word[r];
    }
    __syncthreads();
    if (shift + width < bits) {
#pragma unroll
      for (int r = 0; r < PER; ++r) {
        if (r >= W.per) break;
        if (word_at(W.per, r) < T) W.word[r] = sorted[word_at(W.per, r)];
      }
      __syncthreads();
    }
  }
}

constexpr int kBinPlaces = 10;
constexpr int kBinMost = 32;                             // words that a thread sorts
constexpr int kBins = 1 << kMaxShift;                    // two per thread
static_assert(kBucketCap <= kBins * kBinPlaces && kBins == 2 * kRowsBlock, "bins");

// The same by bins; false (and nothing sorted) where a bin would not fit.  bin:
// [kBins] and wsum: [kRowsWaves] of LDS.
template <int PER>
__device__ __forceinline__ bool spread_big_rows(const RowWords<PER>& W, const BigRows& B, int first,
                                                int T, int m, int net_bits, int* sorted,
                                                unsigned* bin, unsigned* wsum) {
  const int wv = threadIdx.x / kWave, lane = lane_id(), tid = threadIdx.x;
  const unsigned net_mask = (1u << net_bits) - 1u;
  // (a product in floats grows with the net, which is all that a bin needs)
  auto bin_of = [&](unsigned word) {
    const int row = first + (int)(word >> net_bits);
    const int from = (int)(B.at[row] - B.at[first]), d = (int)(B.at[row + 1] - B.at[row]);
    const int guess = (int)((float)(word & net_mask) * ((float)d / (float)m));
    return (from + (guess < d ? guess : d - 1)) / kBinPlaces;
  };
  bin[tid] = bin[tid + kRowsBlock] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (r < W.per && word_at(W.per, r) < T) atomicAdd(&bin[bin_of(W.word[r])], 1u);
  __syncthreads();
  const unsigned a = bin[2 * tid], c = bin[2 * tid + 1];
  const int incl = wave_incl_scan((int)(a + c));
  if (lane == kWave - 1) wsum[wv] = (unsigned)incl;
  if (__syncthreads_or(a > kBinMost || c > kBinMost)) return false;
  unsigned st = (unsigned)incl - a - c;
  for (int w = 0; w < wv; ++w) st += wsum[w];
  bin[2 * tid] = st;
  bin[2 * tid + 1] = st + a;
  __syncthreads();
  // (as signed numbers, which sort_row compares)
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (r < W.per && word_at(W.per, r) < T)
      sorted[atomicAdd(&bin[bin_of(W.word[r])], 1u)] = (int)(W.word[r] ^ 0x80000000u);
  __syncthreads();
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const unsigned at = h ? st + a : st, d = h ? c : a;
    if (d > 16) sort_row<kBinMost>(sorted + at, (int)d);
    else if (d > 0) sort_row<16>(sorted + at, (int)d);
    for (unsigned i = 0; i < d; ++i) sorted[at + i] ^= (int)0x80000000u;
  }
  __syncthreads();
  return true;
}

// One workgroup per bucket: row starts from a count of its pins per vertex,
// the nets placed in their rows in LDS in any order, then every row sorted
// (rows of up to 16 and of up to 32 nets by one thread in registers, each
// kind in wavefronts of its own; rows of up to 128 by one wavefront ranking
// its entries; all longer ones together by the workgroup) and the bucket written
// out.  A vertex twice in a net shows as two equal neighbours.
__global__ __launch_bounds__(kRowsBlock, 6) void k_bucket_rows(Split S) {
  constexpr int kV = 1 << kMaxShift;
  constexpr int kVPer = kV / kRowsBlock;                   // 2
  constexpr int kPer = kBucketCap / kRowsBlock;            // pins per thread
  __shared__ int s_row[kBucketCap];
  __shared__ unsigned s_start[kV + 1];
  __shared__ unsigned s_cur[kV];                           // counts, then write positions
  __shared__ unsigned short s_short[kV];                   // rows of 2..16, and 17..32 from the back
  __shared__ unsigned short s_long[kBucketCap / 33 + 1];
  __shared__ BigRows s_big;
  __shared__ unsigned s_wsum[kRowsWaves];
  __shared__ unsigned s_n16, s_n32, s_nlong, s_nbig;
  static_assert(sizeof(s_cur) == sizeof(unsigned short) * kRowsWaves * kDigits, "digit counts");
  const int V = 1 << S.L.shift;
  const int b = blockIdx.x;
  const unsigned from = bucket_start(S, b);
  const int N = (int)(bucket_end(S, b) - from);
  const int v0 = b << S.L.shift;
  const int nv = S.n - v0 < V ? S.n - v0 : V;
  for (int i = threadIdx.x; i < kV; i += kRowsBlock) s_cur[i] = 0;
  if (threadIdx.x == 0) s_n16 = s_n32 = s_nlong = s_nbig = 0;
  __syncthreads();
  // the whole bucket requested before the first wait
  const unsigned short* low = S.low + from;
  int* val = S.val + from;
  unsigned lv[kPer];
  int net[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int i = q * kRowsBlock + threadIdx.x;
    lv[q] = i < N ? low[i] : 0u;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int i = q * kRowsBlock + threadIdx.x;
    net[q] = i < N ? val[i] : 0;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q)
    if (q * kRowsBlock + (int)threadIdx.x < N) atomicAdd(&s_cur[lv[q]], 1u);
  __syncthreads();
  const int wv = threadIdx.x / kWave, lane = lane_id();
  {
    const int i0 = kVPer * threadIdx.x;
    const unsigned a = s_cur[i0], c = s_cur[i0 + 1];
    const int incl = wave_incl_scan((int)(a + c));
    if (lane == kWave - 1) s_wsum[wv] = (unsigned)incl;
    __syncthreads();
    unsigned off = 0;
    for (int w = 0; w < kRowsWaves; ++w) off += w < wv ? s_wsum[w] : 0u;
    const unsigned st = off + (unsigned)incl - a - c;
    s_start[i0] = s_cur[i0] = st;
    s_start[i0 + 1] = s_cur[i0 + 1] = st + a;
    if (threadIdx.x == kRowsBlock - 1) s_start[kV] = st + a + c;
    if (i0 < nv) S.vptr[v0 + i0] = (long long)from + st;
    if (i0 + 1 < nv) S.vptr[v0 + i0 + 1] = (long long)from + st + a;
    if (v0 + nv == S.n && threadIdx.x == 0) S.vptr[S.n] = S.P;
    // rows by length: one LDS slot each
#pragma unroll
    for (int q = 0; q < kVPer; ++q) {
      const unsigned d = q ? c : a;
      const int r = i0 + q;
      if (d > kWaveRow) s_big.row[atomicAdd(&s_nbig, 1u)] = (unsigned short)r;
      else if (d > 32) s_long[atomicAdd(&s_nlong, 1u)] = (unsigned short)r;
      else if (d > 16) s_short[kV - 1 - atomicAdd(&s_n32, 1u)] = (unsigned short)r;
      else if (d > 1) s_short[atomicAdd(&s_n16, 1u)] = (unsigned short)r;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q)
    if (q * kRowsBlock + (int)threadIdx.x < N) s_row[atomicAdd(&s_cur[lv[q]], 1u)] = net[q];
  __syncthreads();
  bool dup = false;
  const int n16 = (int)s_n16, n32 = (int)s_n32, nlong = (int)s_nlong, nbig = (int)s_nbig;
  for (int i = threadIdx.x; i < n16; i += kRowsBlock) {
    const int r = s_short[i];
    dup |= sort_row<16>(s_row + s_start[r], (int)(s_start[r + 1] - s_start[r]));
  }
  for (int i = threadIdx.x; i < n32; i += kRowsBlock) {
    const int r = s_short[kV - 1 - i];
    dup |= sort_row<32>(s_row + s_start[r], (int)(s_start[r + 1] - s_start[r]));
  }
  for (int i = wv; i < nlong; i += kRowsWaves) {
    const int r = s_long[i];
    const int d = (int)(s_start[r + 1] - s_start[r]);
    int* row = s_row + s_start[r];
    // every lane ranks its entries among the row's (equal entries by place)
    int x[kWaveRow / kWave], rank[kWaveRow / kWave];
#pragma unroll
    for (int q = 0; q < kWaveRow / kWave; ++q) {
      const int at = q * kWave + lane;
      x[q] = at < d ? row[at] : 0x7fffffff;
      rank[q] = 0;
    }
    for (int j = 0; j < d; ++j) {
      const int y = row[j];
#pragma unroll
      for (int q = 0; q < kWaveRow / kWave; ++q) {
        const int at = q * kWave + lane;
        rank[q] += y < x[q] || (y == x[q] && j < at);
        dup |= at < d && y == x[q] && j < at;
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < kWaveRow / kWave; ++q)
      if (q * kWave + lane < d) row[rank[q]] = x[q];
    wave_lds_sync();
  }
  __syncthreads();
  // the rows that are done leave, and the long ones as they are: these are read back
  // and take the LDS
  for (int i = threadIdx.x; i < N; i += kRowsBlock) val[i] = s_row[i];
  if (nbig > 0) {
    const int net_bits = S.m > 1 ? 32 - __clz(S.m - 1) : 1;   // net ids are below 2^net_bits
    if (wv == 0) {                                         // first words, two rows per lane
      const int i0 = 2 * lane, i1 = i0 + 1;
      const int r0 = i0 < nbig ? s_big.row[i0] : 0, r1 = i1 < nbig ? s_big.row[i1] : 0;
      const int d0 = i0 < nbig ? (int)(s_start[r0 + 1] - s_start[r0]) : 0;
      const int d1 = i1 < nbig ? (int)(s_start[r1 + 1] - s_start[r1]) : 0;
      const int incl = wave_incl_scan(d0 + d1);
      if (i0 <= nbig) s_big.at[i0] = (unsigned)(incl - d0 - d1);
      if (i1 <= nbig) s_big.at[i1] = (unsigned)(incl - d1);
    }
    __syncthreads();
    const int together = net_bits > 25 ? 1 << (32 - net_bits) : kBigRows;
    const unsigned net_mask = (1u << net_bits) - 1u;
    unsigned* sorted = reinterpret_cast<unsigned*>(s_row);
    for (int first = 0; first < nbig; first += together) {
      const int last = first + together < nbig ? first + together : nbig;
      const int T = (int)(s_big.at[last] - s_big.at[first]);
      RowWords<kPer> W;
      load_big_rows(W, s_big, first, last, T, val, s_start, net_bits);
      if (!spread_big_rows(W, s_big, first, T, S.m, net_bits, s_row, s_cur, s_wsum))
        radix_big_rows(W, T, net_bits + 32 - __clz(last - first - 1), sorted,
                       reinterpret_cast<unsigned short*>(s_cur), s_wsum);
      for (int p = threadIdx.x; p < T; p += kRowsBlock) {
        const unsigned x = sorted[p], r = first + (x >> net_bits);
        dup |= p > 0 && x == sorted[p - 1];
        val[s_start[s_big.row[r]] + (unsigned)p + s_big.at[first] - s_big.at[r]] =
            (int)(x & net_mask);
      }
      __syncthreads();                                     // before `sorted` is filled again
    }
  }
  if (dup) atomicOr(&S.info->err, kErrDuplicate);
}

static Split make_split(hg_graph_s* g) {
  Split S;
  S.n = g->n;
  S.m = g->m;
  S.P = (int)g->P;
  S.L = load_split(g->n, g->P);
  S.pins = g->pins;
  S.eptr = g->eptr;
  // the radix sort's scratch: coarse offsets in its digit table, the counts where
  // the second split later leaves the low pin bits
  S.ccounts = (unsigned*)(g->ws + g->lay.lhist);
  S.counts = (unsigned*)(g->ws + g->lay.lkey[1]);
  S.rel = (unsigned*)(g->ws + g->lay.lbase);
  S.cursor = S.rel + S.L.buckets;
  S.cbase = S.cursor + S.L.buckets;
  S.cmost = S.cbase + S.L.coarse + 1;
  // the tiles' nets behind these tables, where the radix sort's first pass finds them
  // too; without a split (any number of tiles) in its first key buffer, which the
  // first pass does not use
  S.tile_first = S.L.shift >= 0 ? (int*)(S.cmost + S.L.coarse) : (int*)(g->ws + g->lay.lkey[0]);
  S.cpin = (unsigned*)(g->ws + g->lay.lkey[0]);
  S.cnet = (int*)(g->ws + g->lay.lval);
  S.low = (unsigned short*)(g->ws + g->lay.lkey[1]);
  S.val = g->vnets;
  S.info = (LoadInfo*)(g->ws + g->lay.info);
  S.vptr = g->vptr;
  return S;
}

hipError_t load_check(hg_graph_s* g, hipStream_t s) {
  LoadInfo* info = (LoadInfo*)(g->ws + g->lay.info);
  LoadPart* part = (LoadPart*)(g->ws + g->lay.lpart);
  ZeroRanges Z;
  Z.add(info, sizeof(LoadInfo));
  Z.add(part, (long long)sizeof(LoadPart) * kLoadGrid);
  hipError_t e = zero_ranges(Z, s);
  if (e != hipSuccess) return e;
  const Split S = make_split(g);
  const bool split = S.L.shift >= 0;
  hipLaunchKernelGGL(k_check, dim3(grid_cap_load(g->m > g->n ? g->m : g->n)), dim3(kBlock), 0, s,
                     g->m, g->P, g->eptr, g->ewgt, g->n, g->vwgt, info, part, S.tile_first,
                     pin_tiles(g->P));
  // the pins' range check rides on a count that reads every pin anyway: the
  // buckets' or the sort's first digit count (a pin outside [0, n) only lands
  // in some digit's count, and nothing is built unless the checks pass)
  if (split) {
    hipLaunchKernelGGL(k_split_count, dim3(S.L.grid), dim3(kPartBlock), 0, s, S);
    hipLaunchKernelGGL(k_split_scan, dim3(S.L.coarse), dim3(kSplitScanBlock), 0, s, S);
  } else {
    SortPass SP = first_load_pass(g);
    SP.err = &info->err;
    SP.err_bit = kErrPin;
    SP.key_limit = (unsigned)g->n;
    if (long_load_sort(g->P))
      hipLaunchKernelGGL(k_sort_hist<kSortPerLong>, dim3(SP.tiles), dim3(kBlock), 0, s, SP);
    else
      hipLaunchKernelGGL(k_sort_hist<kSortPer>, dim3(SP.tiles), dim3(kBlock), 0, s, SP);
  }
  hipLaunchKernelGGL(k_fold_load, dim3(1), dim3(kBlock), 0, s, (const LoadPart*)part, info,
                     split ? S.cbase : nullptr, S.cmost, S.L.coarse);
  return hipGetLastError();
}
constexpr int kBigRowGrid = 256;   // workgroups striding over the long rows

// ------------------------------------------------------------------ transpose
// The general path: (pin, net) pairs in net order, stably radix-sorted by pin: the values are
// then the incidence rows, each listing its nets in increasing id, with no
// atomics anywhere (so nothing depends on timing).  Row starts come from
// where the sorted keys change.

// vptr[v] = the first sorted position with key >= v; vptr[n] = P.  A pair
// equal to its predecessor (same pin, same net) is a vertex listed twice in
// one net: the stable sort puts such pairs side by side.  Four positions per
// thread (16-byte loads of keys and values when both arrays are 16-byte
// aligned, `vec`), each compared with the one before it.
constexpr int kRowStartsPer = 4;

__global__ void k_row_starts(long long P, int n, const unsigned* key, const int* val, int vec,
                             long long* vptr, LoadInfo* info) {
  const long long i0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * kRowStartsPer;
  if (i0 >= P) return;
  long long k[kRowStartsPer + 1];
  int v[kRowStartsPer + 1];
  k[0] = i0 == 0 ? -1 : (long long)key[i0 - 1];
  v[0] = i0 == 0 ? -1 : val[i0 - 1];
  if (vec && i0 + kRowStartsPer <= P) {
    const uint4 kq = *reinterpret_cast<const uint4*>(key + i0);
    const int4 vq = *reinterpret_cast<const int4*>(val + i0);
    k[1] = kq.x; k[2] = kq.y; k[3] = kq.z; k[4] = kq.w;
    v[1] = vq.x; v[2] = vq.y; v[3] = vq.z; v[4] = vq.w;
  } else {
    for (int q = 0; q < kRowStartsPer; ++q) {
      k[q + 1] = i0 + q < P ? (long long)key[i0 + q] : -1;
      v[q + 1] = i0 + q < P ? val[i0 + q] : 0;
    }
  }
  int err = 0;
  for (int q = 0; q < kRowStartsPer && i0 + q < P; ++q) {
    const long long i = i0 + q, cur = k[q + 1], prev = k[q];
    if (cur == prev && v[q + 1] == v[q]) err = kErrDuplicate;
    for (long long x = prev + 1; x <= cur; ++x) vptr[x] = i;
    if (i == P - 1)
      for (long long x = cur + 1; x <= n; ++x) vptr[x] = P;
  }
  if (err) atomicOr(&info->err, err);
}

// Per-vertex facts of the sorted rows: degree, w(I(v)), the heavy list.
// With unit net weights (ewgt == NULL) w(I(v)) is the degree and only the
// offsets are read.  Otherwise one thread sums a row of up to kSmallRow
// incidences; longer rows are listed for k_big_row_facts.
__global__ __launch_bounds__(kBlock) void k_row_facts(int n, const long long* vptr,
                                                      const int* vnets, const int* ewgt,
                                                      int* big_list, int* heavy_list,
                                                      LoadInfo* info, LoadPart* part) {
  __shared__ int s_imax[kBlock / kWave];
  __shared__ unsigned s_big, s_heavy, s_big_base, s_heavy_base;
  __shared__ int s_bigv[kBlock], s_heavyv[kBlock];
  int maxdeg = 0, maxincw = 0;
  const long long stride = (long long)gridDim.x * kBlock;
  const long long rounds = ((long long)n + stride - 1) / stride;
  for (long long r = 0; r < rounds; ++r) {
    const long long v = r * stride + (long long)blockIdx.x * kBlock + threadIdx.x;
    if (threadIdx.x == 0) s_big = s_heavy = 0;
    __syncthreads();
    bool big = false, heavy = false;
    if (v < n) {
      const long long b = vptr[v];
      const int deg = (int)(vptr[v + 1] - b);
      maxdeg = deg > maxdeg ? deg : maxdeg;
      if (!ewgt) {
        maxincw = deg > maxincw ? deg : maxincw;
        heavy = deg > kLightLimit;
      } else if (deg > kSmallRow) {
        big = true;
      } else {
        // the row's entries in groups of four, loaded before their weights
        const int* row = vnets + b;
        long long tot = 0;
        for (int i0 = 0; i0 < deg; i0 += 4) {
          int x[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) x[q] = row[i0 + q < deg ? i0 + q : i0];
          int wq[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) wq[q] = ewgt[x[q]];
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (i0 + q < deg) tot += wq[q];
        }
        const int incw = tot > 0x7fffffffLL ? 0x7fffffff : (int)tot;
        maxincw = incw > maxincw ? incw : maxincw;
        heavy = tot > kLightLimit;
      }
    }
    if (big) s_bigv[atomicAdd(&s_big, 1u)] = (int)v;
    if (heavy) s_heavyv[atomicAdd(&s_heavy, 1u)] = (int)v;
    __syncthreads();
    if (threadIdx.x == 0) {
      s_big_base = s_big ? atomicAdd((unsigned*)&info->big_rows, s_big) : 0;
      s_heavy_base = s_heavy ? atomicAdd((unsigned*)&info->heavy_count, s_heavy) : 0;
    }
    __syncthreads();
    if (threadIdx.x < s_big) big_list[s_big_base + threadIdx.x] = s_bigv[threadIdx.x];
    if (threadIdx.x < s_heavy) heavy_list[s_heavy_base + threadIdx.x] = s_heavyv[threadIdx.x];
    __syncthreads();
  }
  const int md = block_max_int(maxdeg, s_imax);
  const int mi = block_max_int(maxincw, s_imax);
  if (threadIdx.x == 0) {
    part[blockIdx.x].max_degree = md;
    part[blockIdx.x].max_incident_weight = mi;
  }
}

// One workgroup per long row: the same facts with the row's entries spread
// over the workgroup.
__global__ void k_big_row_facts(const long long* vptr, const int* vnets, const int* ewgt,
                                const int* big_list, int* heavy_list, LoadInfo* info) {
  __shared__ long long s_tmp[kBlock / kWave];
  // the count comes from the short-row pass (an earlier launch), so the host
  // need not read it first; a fixed grid strides over the list
  const int nbig = info->big_rows;
  for (int bi = blockIdx.x; bi < nbig; bi += gridDim.x) {
    const int v = big_list[bi];
    const long long b = vptr[v];
    const int len = (int)(vptr[v + 1] - b);
    const int* row = vnets + b;
    long long tot = 0;
    for (int i = threadIdx.x; i < len; i += blockDim.x) tot += ewgt[row[i]];
    tot = block_sum64(tot, s_tmp);
    if (threadIdx.x == 0) {
      const int incw = tot > 0x7fffffffLL ? 0x7fffffff : (int)tot;
      atomicMax(&info->max_degree, len);
      atomicMax(&info->max_incident_weight, incw);
      if (tot > kLightLimit) {
        const int hi = atomicAdd(&info->heavy_count, 1);
        heavy_list[hi] = v;
      }
    }
    __syncthreads();
  }
}

// The transpose by radix passes over the (pin, net) pairs; `counted`: the
// checks left the first pass's digit counts.
static void build_by_sort(hg_graph_s* g, bool counted, hipStream_t s) {
  LoadInfo* info = (LoadInfo*)(g->ws + g->lay.info);
  const long long P = g->P;
  int passes = 0;
  for (int bits = 0; bits < 32 && (1ll << bits) < (long long)g->n; bits += 8) ++passes;
  if (passes == 0) passes = 1;
  // the last pass must leave its values in vnets
  unsigned* key[2] = {(unsigned*)(g->ws + g->lay.lkey[0]), (unsigned*)(g->ws + g->lay.lkey[1])};
  int* scratch = (int*)(g->ws + g->lay.lval);
  int* val[2];
  val[passes & 1] = g->vnets;
  val[(passes & 1) ^ 1] = scratch;
  // the first pass reads the (validated, non-negative) pins as its keys and finds
  // their nets as it goes.  (Expanding them beforehand took 55 us on a netlist of
  // 56.5M pins.  The checks of a hypergraph whose fullest bucket turns out too full
  // cost a count and a scan that come to nothing: with one vertex in 50,000 nets of
  // that netlist the load took 1423 us before there were ranges, 1487 with both,
  // 1445 so; 4.3M vertices without ranges 1423 and 1382.)
  SortPass SP = first_load_pass(g);
  SP.eptr = g->eptr;
  SP.tile_net = make_split(g).tile_first;
  const bool long_sort = long_load_sort(P);
  for (int q = 0; q < passes; ++q) {
    SP.val_in = val[q & 1];
    SP.key_out = key[(q & 1) ^ 1];
    SP.val_out = val[(q & 1) ^ 1];
    SP.shift = 8 * q;
    if (q == 0 && long_sort)
      sort_pass_nets<kSortPerLong>(SP, counted, s);
    else if (q == 0)
      sort_pass_nets(SP, counted, s);
    else if (long_sort)
      sort_pass<kSortPerLong>(SP, s);
    else
      sort_pass(SP, s);
    SP.key_in = SP.key_out;
  }
  const long long rs_threads = (P + kRowStartsPer - 1) / kRowStartsPer;
  const unsigned* skey = key[passes & 1];
  const int vec = (((uintptr_t)skey | (uintptr_t)g->vnets) & 15) == 0;
  hipLaunchKernelGGL(k_row_starts, dim3((unsigned)((rs_threads + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, P, g->n, skey, (const int*)g->vnets, vec, g->vptr, info);
}

// Builds vptr/vnets (by vertex ranges when the checks counted buckets that
// all fit a workgroup's LDS) and the rows' facts (short rows one per thread,
// long rows one per workgroup).
hipError_t load_build(hg_graph_s* g, hipStream_t s) {
  LoadInfo* info = (LoadInfo*)(g->ws + g->lay.info);
  int* big = (int*)(g->ws + g->lay.big);
  int* heavy = (int*)(g->ws + g->lay.heavy);
  const Split S = make_split(g);
  if (S.L.shift >= 0 && g->info.max_bucket <= (unsigned)kBucketCap) {
    hipLaunchKernelGGL(k_split_coarse, dim3(S.L.grid), dim3(kPartBlock), 0, s, S);
    hipLaunchKernelGGL(k_split_fine, dim3(S.L.tiles + S.L.coarse), dim3(kPartBlock), 0, s, S);
    hipLaunchKernelGGL(k_bucket_rows, dim3(S.L.buckets), dim3(kRowsBlock), 0, s, S);
  } else {
    build_by_sort(g, S.L.shift < 0, s);
  }
  // all net weights 1 (the checks summed them to m): rows need no weights
  const int* ew = g->info.total_net_weight == (unsigned long long)g->m ? nullptr : g->ewgt;
  LoadPart* part = (LoadPart*)(g->ws + g->lay.lpart);
  hipLaunchKernelGGL(k_row_facts, dim3(grid_cap_load(g->n)), dim3(kBlock), 0, s, g->n, g->vptr,
                     g->vnets, ew, big, heavy, info, part);
  hipLaunchKernelGGL(k_fold_load, dim3(1), dim3(kBlock), 0, s, (const LoadPart*)part, info,
                     (unsigned*)nullptr, (const unsigned*)nullptr, 0);
  if (ew)
    hipLaunchKernelGGL(k_big_row_facts, dim3(kBigRowGrid), dim3(kBlock), 0, s, g->vptr, g->vnets,
                       ew, big, heavy, info);
  return hipGetLastError();
}

}  // namespace hg
