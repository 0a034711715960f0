// Stable radix sort on the device and the CSR transpose built on it (Sec. 2.1 / Sec. 4.1: the forward
// pass multiplies by A^T, the backward pass by A; a directed graph needs both orientations).
//
// Least-significant digit first, at most 8 bits per pass (the key bits are spread evenly over the
// passes), three launches per pass over tiles of consecutive pairs:
//   count    digit histogram of a tile in LDS -> counts[digit][tile]
//   scan     one workgroup per digit: exclusive scan along the tiles, digit total
//   scatter  ranks inside the tile by ballots (stable), the tile is sorted by digit in LDS and then
//            written out in that order, so that neighbouring lanes store to neighbouring places
// Up to kFewTiles tiles there is no scan: counts[tile][digit], and a tile adds up the others' counts by itself.
// What bounds it: HBM.  A pass reads and writes every key and payload word once and reads the keys once
// more for the counts.  The earlier form (one wavefront per tile, a serial loop over the distinct digits
// of 64 keys, stores in entry order) took 14.4 ms for seven passes over 21 M pairs, almost all of it in
// that loop and in scattered stores.
//
// The transpose sorts the entries by column with their row and value as payload, so no entry index is
// looked up afterwards: the first pass reads the caller's arrays (a tile's rows come from the slice of
// rowptr that covers it), the last pass writes the caller's outputs.  Stability makes the entries of a
// transposed row come out in the order of the rows they came from, and keeps duplicates in stored order.
#include <algorithm>

#include "common.h"

namespace sagnn {
namespace {

constexpr int kMaxBins = 256;
// Tiles of at least 8192 pairs keep the runs of one digit long enough for whole-line stores; fewer pairs
// are cut into smaller tiles while that leaves CUs without work.
constexpr int64_t kTileSmallMax = 1 << 18;   // up to here: tiles of 1024 pairs
constexpr int64_t kTileMidMax = 1 << 22;     // up to here: tiles of 2048 pairs

// Sorts of few tiles are bound by their launches, and the scan is one of three.  (A tile reads all counts, ntiles lines of
// 1 KB.  A pass over 33 k pairs: scan and scatter 3.4 + 5.8 us, now 6.0; over 100 k, 4.2 + 6.5 and 10.6, one launch fewer;
// the reads grow with the tiles, the scan does not.)
constexpr int64_t kFewTiles = 128;

inline int radix_tile(int64_t n) { return n <= kTileSmallMax ? 1024 : (n <= kTileMidMax ? 2048 : 8192); }

struct PassArgs {
  const uint32_t* keys_in;
  const uint32_t* p0_in;      // first payload word (SRC_ARRAYS)
  const uint32_t* p1_in;      // second payload word (NP == 2)
  uint32_t *keys_out, *p0_out, *p1_out;
  int64_t n, ntiles;
  int32_t shift, bits;
  int32_t* counts;            // [bins][ntiles], few tiles: [ntiles][bins]
  int32_t* totals;            // [bins]
  const int32_t* rowptr;      // SRC_ROWS: the first payload word is the row of the entry
  int64_t m;
  int32_t* inverse;           // SRC_ORDER: the place of every pair
};

enum Src { SRC_ARRAYS = 0, SRC_INDEX = 1, SRC_ROWS = 2, SRC_ORDER = 3 };   // (SRC_ORDER: as SRC_INDEX, without sorted keys)

// limit > 0: err[0] = 1 if some key is >= limit
// Eight counters per digit, side by side, taken by the lanes in turn: lanes that add to one counter wait for each other, and the
// low bits of a power-law graph's columns are as uneven as its degrees (40 M columns 93 us with one counter, now 38; the high
// bits 37, 44).
template <int THREADS, int KPT, bool FEW>
__global__ __launch_bounds__(THREADS) void radix_count_kernel(const uint32_t* __restrict__ keys, int64_t n,
                                                              int64_t ntiles, int32_t shift, int32_t bits,
                                                              int32_t* __restrict__ counts, uint32_t limit,
                                                              int32_t* __restrict__ err) {
  constexpr int COPIES = 8;
  __shared__ int32_t hist[kMaxBins * COPIES];
  const int bins = 1 << bits, copy = threadIdx.x & (COPIES - 1);
  for (int i = threadIdx.x; i < bins * COPIES; i += THREADS) hist[i] = 0;
  const int64_t e0 = (int64_t)blockIdx.x * (THREADS * KPT) + threadIdx.x;
  uint32_t key[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) key[j] = e0 + j * THREADS < n ? keys[e0 + j * THREADS] : 0u;
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if (e0 + j * THREADS < n) {
      bad |= limit != 0u && key[j] >= limit;
      atomicAdd(&hist[((key[j] >> shift) & (uint32_t)(bins - 1)) * COPIES + copy], 1);
    }
  if (bad) err[0] = 1;
  __syncthreads();
  for (int i = threadIdx.x; i < bins; i += THREADS) {
    int32_t t = 0;
#pragma unroll
    for (int q = 0; q < COPIES; ++q) t += hist[i * COPIES + q];
    counts[FEW ? (int64_t)blockIdx.x * bins + i : (int64_t)i * ntiles + blockIdx.x] = t;
  }
}

// exclusive scan of one value per thread over the workgroup; *total = sum
template <int THREADS>
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t* wsum, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int32_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    if (w < wave) before += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return before + inc - v;
}

__global__ __launch_bounds__(1024) void radix_scan_kernel(int32_t* __restrict__ counts, int64_t ntiles,
                                                          int32_t* __restrict__ totals) {
  __shared__ int32_t wsum[16];
  int32_t* __restrict__ c = counts + (int64_t)blockIdx.x * ntiles;
  int32_t carry = 0;
  for (int64_t base = 0; base < ntiles; base += 4096) {
    const int64_t i = base + (int64_t)threadIdx.x * 4;
    int32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = i + q < ntiles ? c[i + q] : 0;
    int32_t tot;
    int32_t ex = carry + block_scan<1024>(v[0] + v[1] + v[2] + v[3], wsum, &tot);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i + q < ntiles) c[i + q] = ex;
      ex += v[q];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Largest r in [0, m) with rowptr[r] <= e, found by one wavefront (64 probes per step).
__device__ __forceinline__ int64_t wave_find_row(const int32_t* __restrict__ rowptr, int64_t m, int64_t e) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0, hi = m;            // the answer lies in [lo, hi)
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t p = lo + (int64_t)(lane + 1) * step;      // probes ascend with the lane
    const bool below = p < hi && (int64_t)rowptr[p] <= e;
    const int cnt = __popcll(__ballot(below));              // a prefix of the lanes (rowptr is monotone)
    const int64_t nlo = lo + (int64_t)cnt * step;
    hi = nlo + step < hi ? nlo + step : hi;
    lo = nlo;
  }
  return lo;
}

// The tile of a workgroup.  A tile's run of a digit begins and ends inside lines that it shares with the tiles before and
// behind; workgroups go to the eight XCDs in turn, so that each of these lines was written in parts out of two L2s.  An XCD now
// takes runs of tiles.  40 M pairs, three passes 250, 290, 232 us (3.2 to 4.1 TB/s read and
// written), with runs of 16 234, 233, 209 (3.4 to 4.6), of 64 the same, of 256 240, 243, 217.
constexpr int kXcdRun = 16;
__device__ __forceinline__ int32_t xcd_run(int32_t block, int32_t ntiles) {
  const int32_t first = block / (8 * kXcdRun) * (8 * kXcdRun);
  if (first + 8 * kXcdRun > ntiles) return block;
  const int32_t i = block - first;
  return first + (i & 7) * kXcdRun + (i >> 3);
}

template <int THREADS, int KPT, int NP, int SRC, bool FEW>
__global__ __launch_bounds__(THREADS) void radix_scatter_kernel(const PassArgs a) {
  const int32_t tile = FEW ? (int32_t)blockIdx.x : xcd_run((int32_t)blockIdx.x, (int32_t)a.ntiles);
  constexpr int TILE = THREADS * KPT, WAVES = THREADS / 64;
  __shared__ uint32_t stage[TILE];
  __shared__ int32_t hist[WAVES][kMaxBins];
  __shared__ int32_t gbase[kMaxBins];      // output position of a digit's first pair, minus its staged position
  __shared__ int32_t wsum[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bins = 1 << a.bits;
  const int64_t tile0 = (int64_t)tile * TILE;
  const int cnt = (int)(a.n - tile0 < TILE ? a.n - tile0 : TILE);
  for (int i = tid; i < WAVES * kMaxBins; i += THREADS) (&hist[0][0])[i] = 0;
  // a wavefront owns 64 * KPT consecutive pairs
  const int seg = wave * 64 * KPT + lane;
  uint32_t key[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) key[j] = seg + j * 64 < cnt ? a.keys_in[tile0 + seg + j * 64] : 0u;
  int32_t digit_total = 0, digit_before = 0;       // pairs of digit `tid` in all tiles, in the tiles before this one
  if constexpr (FEW) {
    if (tid < bins) {
#pragma unroll 16
      for (int t = 0; t < (int)a.ntiles; ++t) {
        const int32_t v = a.counts[t * bins + tid];
        digit_total += v;
        digit_before += t < (int)tile ? v : 0;
      }
      if (SRC == SRC_ORDER && tile == 0) a.totals[tid] = digit_total;
    }
  } else {
    if (tid < bins) {
      digit_total = a.totals[tid];
      digit_before = a.counts[(int64_t)tid * a.ntiles + tile];
    }
  }
  __syncthreads();

  // rank of every pair among the wavefront's earlier pairs of its digit
  int32_t pos[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const bool act = seg + j * 64 < cnt;
    const uint32_t d = (key[j] >> a.shift) & (uint32_t)(bins - 1);
    uint64_t peers = __ballot(act);
    for (int b = 0; b < a.bits; ++b) {
      const bool one = (d >> b) & 1u;
      const uint64_t ones = __ballot(one);
      peers &= one ? ones : ~ones;
    }
    const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
    // (the LDS operations of one wavefront are carried out in order: read, then the first peer's update)
    const int32_t have = __hip_atomic_load(&hist[wave][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    pos[j] = have + below;
    if (act && below == 0)
      __hip_atomic_store(&hist[wave][d], have + __popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // digits -> first staged position; hist becomes the staged position of a wavefront's first pair of a digit
  {
    const int d = tid;
    int32_t mine = 0;
    if (d < bins) {
#pragma unroll
      for (int w = 0; w < WAVES; ++w) mine += hist[w][d];
    }
    int32_t tot, dtot;
    const int32_t start = block_scan<THREADS>(mine, wsum, &tot);
    const int32_t before = block_scan<THREADS>(digit_total, wsum, &dtot);
    if (d < bins) {
      gbase[d] = before + digit_before - start;
      int32_t run = start;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const int32_t t = hist[w][d];
        hist[w][d] = run;
        run += t;
      }
    }
  }
  static_assert(THREADS >= kMaxBins, "one thread per digit");
  __syncthreads();
#pragma unroll
  for (int j = 0; j < KPT; ++j) pos[j] += hist[wave][(key[j] >> a.shift) & (uint32_t)(bins - 1)];

  uint32_t row[SRC == SRC_ROWS ? KPT : 1];
  if constexpr (SRC == SRC_ROWS) {
    // Rows of the tile's entries: every row that begins inside the tile leaves its number where it begins (of several, all
    // but the last empty, the last), and an entry's row is the nearest mark at or before it, found in a ballot of 64 entries.
    // (A binary search per entry, nine dependent LDS reads, bound the pass: 40 M entries, 1 M rows 370 us, so 250, in runs
    // for each XCD 234; the passes whose payloads are both read from memory take 209 and 233.)
    __shared__ int64_t ends[2];
    __shared__ int32_t last_mark[WAVES];
    if (wave < 2) {
      const int64_t r = wave_find_row(a.rowptr, a.m, wave == 0 ? tile0 : tile0 + cnt - 1);
      if (lane == 0) ends[wave] = r;
    }
    for (int i = tid; i < TILE; i += THREADS) stage[i] = 0u;
    __syncthreads();
    const int64_t r_lo = ends[0], nstart = ends[1] - r_lo;    // rows that begin inside the tile (the first one aside)
    for (int64_t i = tid; i < nstart; i += THREADS) {
      const int64_t at = (int64_t)a.rowptr[r_lo + 1 + i] - tile0;
      if (at >= 0 && at < TILE) atomicMax(&stage[at], (uint32_t)(i + 1));
    }
    __syncthreads();
    uint32_t mark = 0;                                        // the last one so far, of this wavefront's entries
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const uint32_t here = stage[seg + j * 64];
      const uint64_t marks = __ballot(here != 0u);
      const uint64_t upto = marks & ((2ull << lane) - 1ull);
      const uint32_t near = (uint32_t)__shfl((int)here, upto ? 63 - __builtin_clzll(upto) : 0, 64);
      row[j] = upto ? near : mark;
      if (marks) mark = (uint32_t)__shfl((int)here, 63 - __builtin_clzll(marks), 64);
    }
    if (lane == 0) last_mark[wave] = (int32_t)mark;
    __syncthreads();
    uint32_t before = 0;                                      // of the wavefronts before (marks ascend)
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
      if (w < wave) before = (uint32_t)last_mark[w] > before ? (uint32_t)last_mark[w] : before;
#pragma unroll
    for (int j = 0; j < KPT; ++j) row[j] = (uint32_t)r_lo + (row[j] ? row[j] : before);
    __syncthreads();
  }

#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if (seg + j * 64 < cnt) stage[pos[j]] = key[j];
  __syncthreads();
  int32_t dst[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int i = j * THREADS + tid;
    dst[j] = -1;
    if (i < cnt) {
      const uint32_t k = stage[i];
      dst[j] = gbase[(k >> a.shift) & (uint32_t)(bins - 1)] + i;
      if constexpr (SRC != SRC_ORDER) a.keys_out[dst[j]] = k;
    }
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const uint32_t* __restrict__ in = q == 0 ? a.p0_in : a.p1_in;
    uint32_t* __restrict__ out = q == 0 ? a.p0_out : a.p1_out;
    uint32_t v[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const int i = seg + j * 64;
      if (q == 0 && (SRC == SRC_INDEX || SRC == SRC_ORDER)) v[j] = (uint32_t)(tile0 + i);
      else if (q == 0 && SRC == SRC_ROWS) v[j] = row[SRC == SRC_ROWS ? j : 0];
      else v[j] = i < cnt ? in[tile0 + i] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KPT; ++j)
      if (seg + j * 64 < cnt) stage[pos[j]] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KPT; ++j)
      if (dst[j] >= 0) {
        out[dst[j]] = stage[j * THREADS + tid];
        if constexpr (SRC == SRC_ORDER) a.inverse[stage[j * THREADS + tid]] = dst[j];
      }
  }
}

template <int THREADS, int KPT, bool FEW>
int run_pass(const PassArgs& a, int np, int src, uint32_t limit, int32_t* err, hipStream_t s) {
  const dim3 grid((unsigned)a.ntiles);
  hipLaunchKernelGGL((radix_count_kernel<THREADS, KPT, FEW>), grid, dim3(THREADS), 0, s, a.keys_in, a.n, a.ntiles, a.shift,
                     a.bits, a.counts, limit, err);
  SAGNN_LAUNCH_CHECK();
  if (!FEW) {
    hipLaunchKernelGGL(radix_scan_kernel, dim3(1u << a.bits), dim3(1024), 0, s, a.counts, a.ntiles, a.totals);
    SAGNN_LAUNCH_CHECK();
  }
  const auto scatter = src == SRC_ROWS    ? radix_scatter_kernel<THREADS, KPT, 2, SRC_ROWS, FEW>
                       : src == SRC_INDEX ? radix_scatter_kernel<THREADS, KPT, 1, SRC_INDEX, FEW>
                       : src == SRC_ORDER ? radix_scatter_kernel<THREADS, KPT, 1, SRC_ORDER, FEW>
                       : np == 2          ? radix_scatter_kernel<THREADS, KPT, 2, SRC_ARRAYS, FEW>
                                          : radix_scatter_kernel<THREADS, KPT, 1, SRC_ARRAYS, FEW>;
  hipLaunchKernelGGL(scatter, grid, dim3(THREADS), 0, s, a);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

int run_pass(PassArgs a, int np, int src, uint32_t limit, int32_t* err, hipStream_t s) {
  const int tile = radix_tile(a.n);
  a.ntiles = ceil_div(a.n, tile);
  if (tile == 1024) {
    return a.ntiles <= kFewTiles ? run_pass<256, 4, true>(a, np, src, limit, err, s)
                                 : run_pass<256, 4, false>(a, np, src, limit, err, s);
  }
  if (tile == 2048) return run_pass<256, 8, false>(a, np, src, limit, err, s);
  return run_pass<512, 16, false>(a, np, src, limit, err, s);
}

inline int passes_of(int bits) { return (bits + 7) / 8; }

}  // namespace

RadixWs carve_radix(void* base, int64_t n) {
  RadixWs w{};
  const int64_t cap = n > 0 ? n : 1;
  // sized for the count that needs the most tiles among all counts <= cap
  const int64_t max_tiles = std::max(ceil_div(cap, radix_tile(cap)),
                                     std::max(std::min(ceil_div(cap, 1024), ceil_div(kTileSmallMax, 1024)),
                                              std::min(ceil_div(cap, 2048), ceil_div(kTileMidMax, 2048))));
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? static_cast<char*>(base) + off : nullptr;
    off += round_up(bytes, 256);
    return p;
  };
  for (int i = 0; i < 2; ++i) {
    w.keys[i] = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)cap));
    w.pay[i] = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)cap));
  }
  w.counts = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * kMaxBins * (size_t)max_tiles));
  w.totals = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (kMaxBins + 1)));
  w.cap = cap;
  w.bytes = off;
  return w;
}

int radix_sort_pairs(const uint32_t* keys_in, const uint32_t* pay_in, int64_t n, int bits, const RadixWs& w,
                     hipStream_t s, int* result, int64_t limit, int32_t* err) {
  if (n < 0 || n > w.cap || bits < 1 || bits > 32 || (limit > 0 && !err)) return SAGNN_EINVAL;
  const int passes = passes_of(bits);
  *result = (passes - 1) & 1;
  if (n == 0) return SAGNN_OK;
  const int per = (bits + passes - 1) / passes;
  for (int p = 0; p < passes; ++p) {
    PassArgs a{};
    a.n = n;
    a.keys_in = p == 0 ? keys_in : w.keys[(p - 1) & 1];
    a.p0_in = p == 0 ? pay_in : w.pay[(p - 1) & 1];
    a.keys_out = w.keys[p & 1];
    a.p0_out = w.pay[p & 1];
    a.shift = p * per;
    a.bits = std::min(per, bits - p * per);
    a.counts = w.counts;
    a.totals = w.totals;
    const int rc = run_pass(a, 1, p == 0 && !pay_in ? SRC_INDEX : SRC_ARRAYS, p == 0 ? (uint32_t)limit : 0u, err, s);
    if (rc != SAGNN_OK) return rc;
  }
  return SAGNN_OK;
}

int radix_order(const uint32_t* keys, int64_t n, int bits, const RadixWs& w, int32_t* order, int32_t* inverse, hipStream_t s,
                int64_t limit) {
  if (n < 1 || n > w.cap || bits < 1 || bits > 8 || !w.keys[0]) return SAGNN_EINVAL;
  PassArgs a{};
  a.keys_in = keys;
  a.p0_out = reinterpret_cast<uint32_t*>(order);
  a.inverse = inverse;
  a.n = n;
  a.bits = bits;
  a.counts = w.counts;
  a.totals = w.totals;
  return run_pass(a, 1, SRC_ORDER, (uint32_t)limit, w.totals + kMaxBins, s);
}

namespace {

constexpr int kThreads = 256;

// rowptr[c] = number of sorted keys below c, c in [0, n], from the places where the sorted keys change: the
// pair at i fills rowptr(previous key .. its key] = i.  Long gaps (runs of empty rows) are filled by the
// whole wavefront.  A thread takes four keys, one wide load (bound by requests: 40 M keys 80 us with one key a thread, now 41;
// the keys lie at the start of a workspace array, 256-byte aligned).
constexpr int kRowptrKeys = 4;
__global__ __launch_bounds__(kThreads) void sorted_rowptr_kernel(const uint32_t* __restrict__ keys, int64_t cnt,
                                                                 int64_t n, int32_t* __restrict__ rowptr) {
  const int lane = threadIdx.x & 63;
  const int64_t i0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * kRowptrKeys;
  // (the place behind the last pair closes the array; keys are clamped, an out-of-range key is an error elsewhere)
  int64_t key[kRowptrKeys + 1];
  key[0] = i0 > 0 && i0 <= cnt ? (int64_t)keys[i0 - 1] : -1;
  if (i0 + kRowptrKeys <= cnt) {
    const uint4 k = *reinterpret_cast<const uint4*>(keys + i0);
    key[1] = k.x; key[2] = k.y; key[3] = k.z; key[4] = k.w;
  } else {
#pragma unroll
    for (int j = 0; j < kRowptrKeys; ++j) key[j + 1] = i0 + j < cnt ? (int64_t)keys[i0 + j] : n;
  }
#pragma unroll
  for (int j = 0; j < kRowptrKeys; ++j) {
    const int64_t i = i0 + j;
    const int64_t from = (key[j] < n ? key[j] : n) + 1, to = i <= cnt ? (key[j + 1] < n ? key[j + 1] : n) : -1;
    const bool wide = to - from >= 8;
    if (!wide)
      for (int64_t c = from; c <= to; ++c) rowptr[c] = (int32_t)i;
    for (uint64_t left = __ballot(wide); left; left &= left - 1) {
      const int src = __builtin_ctzll(left);
      const int64_t f = __shfl(from, src, 64), t = __shfl(to, src, 64), v = __shfl(i, src, 64);
      for (int64_t c = f + lane; c <= t; c += 64) rowptr[c] = (int32_t)v;
    }
  }
}

int bits_for(int64_t n) {
  int bits = 1;
  while (bits < 31 && (1ll << bits) < n) ++bits;
  return bits;
}

}  // namespace

int launch_sorted_rowptr(const uint32_t* keys, int64_t cnt, int64_t n, int32_t* rowptr, hipStream_t s) {
  hipLaunchKernelGGL(sorted_rowptr_kernel, dim3((unsigned)ceil_div(cnt + 1, kThreads * kRowptrKeys)), dim3(kThreads), 0, s,
                     keys, cnt, n, rowptr);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

size_t transpose_ws_bytes(int64_t nnz) { return carve_radix(nullptr, nnz).bytes + 256; }   // sort, error flag

// d_err[0] is set to 1 if a column is outside [0, n); the caller has cleared it
int launch_transpose(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m, int64_t n, int64_t nnz,
                     int32_t* rowptr_t, int32_t* colidx_t, float* val_t, void* ws, int32_t* d_err, hipStream_t s) {
  const RadixWs w = carve_radix(ws, nnz);
  uint32_t* val_ws = w.pay[1];   // (w.pay[0] takes the rows)
  const int bits = bits_for(n), passes = passes_of(bits), per = (bits + passes - 1) / passes;
  int last = 0;
  for (int p = 0; p < passes && nnz > 0; ++p) {
    // the passes alternate between the workspace and the output arrays so that the last one ends in the outputs
    const bool to_out = ((passes - 1 - p) & 1) == 0;
    uint32_t* rows_out = to_out ? reinterpret_cast<uint32_t*>(colidx_t) : w.pay[0];
    uint32_t* vals_out = to_out ? reinterpret_cast<uint32_t*>(val_t) : val_ws;
    PassArgs a{};
    a.n = nnz;
    a.keys_in = p == 0 ? reinterpret_cast<const uint32_t*>(colidx) : w.keys[(p - 1) & 1];
    a.p0_in = p == 0 ? nullptr : (to_out ? w.pay[0] : reinterpret_cast<const uint32_t*>(colidx_t));
    a.p1_in = p == 0 ? reinterpret_cast<const uint32_t*>(val)
                     : (to_out ? val_ws : reinterpret_cast<const uint32_t*>(val_t));
    a.keys_out = w.keys[p & 1];
    a.p0_out = rows_out;
    a.p1_out = vals_out;
    a.shift = p * per;
    a.bits = std::min(per, bits - p * per);
    a.counts = w.counts;
    a.totals = w.totals;
    a.rowptr = rowptr;
    a.m = m;
    const int rc = run_pass(a, 2, p == 0 ? SRC_ROWS : SRC_ARRAYS, p == 0 ? (uint32_t)n : 0u, d_err, s);
    if (rc != SAGNN_OK) return rc;
    last = p & 1;
  }
  return launch_sorted_rowptr(w.keys[last], nnz, n, rowptr_t, s);
}

}  // namespace sagnn

SAGNN_EXPORT int spmm_transpose_workspace_bytes(int64_t nnz, size_t* bytes) {
  using namespace sagnn;
  if (!bytes || nnz < 0 || nnz > 0x7FFFFFFFll) return SAGNN_EINVAL;
  *bytes = transpose_ws_bytes(nnz);
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_transpose(const int32_t* d_rowptr, const int32_t* d_colidx,
                                    const float* d_val, int64_t m, int64_t n, int64_t nnz,
                                    int32_t* d_rowptr_t, int32_t* d_colidx_t, float* d_val_t,
                                    void* d_ws, size_t ws_bytes, void* stream) {
  using namespace sagnn;
  if (m < 0 || n < 0 || nnz < 0 || m > 0x7FFFFFFFll || n > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  if (!d_rowptr || !d_rowptr_t || !d_ws) return SAGNN_EINVAL;
  if (nnz > 0 && (!d_colidx || !d_val || !d_colidx_t || !d_val_t)) return SAGNN_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ws) & 255u) return SAGNN_EINVAL;
  const size_t need = transpose_ws_bytes(nnz);
  if (ws_bytes < need) return SAGNN_ECAPACITY;
  if (n == 0 && nnz > 0) return SAGNN_EFORMAT;   // no column index can be valid
  hipStream_t s = (hipStream_t)stream;
  int32_t* d_err = reinterpret_cast<int32_t*>(static_cast<char*>(d_ws) + need - 256);
  SAGNN_HIP(hipMemsetAsync(d_err, 0, sizeof(int32_t), s));
  const int rc = launch_transpose(d_rowptr, d_colidx, d_val, m, n, nnz, d_rowptr_t, d_colidx_t, d_val_t, d_ws, d_err, s);
  if (rc != SAGNN_OK) return rc;
  int32_t h_err = 0;
  SAGNN_HIP(hipMemcpyAsync(&h_err, d_err, sizeof(h_err), hipMemcpyDeviceToHost, s));
  SAGNN_HIP(hipStreamSynchronize(s));
  if (h_err) return SAGNN_EFORMAT;
  return SAGNN_OK;
}
