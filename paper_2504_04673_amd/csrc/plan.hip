// Needed-row planning: NnzCols of every column block of a CSR row block (Sec. 4.1, the
// paragraph that defines NnzCols(i,j) as the nonzero column indices of block A_ij, i.e. the
// rows of H_j that P(i) has to receive).
//
// Integer only, result unique.  Pipeline (all kernels on the caller's stream, launched without a wait in between):
//   mark     one pass over colidx -> membership words, by one of three ways (see below): byte flags in memory,
//            LDS bitmaps, range buckets; the words' population counts are summed per tile of 2048 words
//   prefix   rank of the first column of every word (each workgroup adds up the tiles before its own)
//   finish   block offsets and N to the host record (first workgroup), needed[] and the remap:
//            a wavefront per word, lane l owns column 64w+l, the ballot mask and mbcnt give each set lane its slot
//            (needed[] comes out ascending); compact[e] = prefix[c>>6] + popcount(word & bits below c): position of
//            column c in needed[]; monotone in c, so sorted rows stay sorted
// The block offsets are written straight into pinned host memory and the call returns as soon as they are there,
// while needed[] and the remap may still be in the making on the stream; capacity and validity are checked by the
// kernels before they write.  (Ten launches, three copies and a wait in the middle before: a block of 100 k columns and
// 1 M entries took 363 us, now 35.)
// Traffic: nnz*4 (mark) + nnz*8 (remap read+write) + N*4 + a few passes over n bytes.
#include <atomic>
#include <mutex>

#include "common.h"

namespace sagnn {
namespace {

constexpr int kThreads = 256;
constexpr int kWordsPerBlock = 2048;  // scan tile: 256 threads x 8 words

// LDS marking (column ranges small enough to be covered by a few LDS-resident bitmaps):
// a workgroup owns a private bitmap of kLdsCols columns in LDS and a share of the entries.
constexpr int kLdsThreads = 1024;
constexpr int kLdsWords = 38912;                    // 32-bit words: 152 KB of the CU's 160 KB
constexpr int64_t kLdsCols = (int64_t)kLdsWords * 32;
constexpr int kLdsMaxPasses = 4;
constexpr int kLdsGroups = 256;                     // workgroups in total (one per CU)
constexpr int64_t kLdsMinNnz = 1ll << 22;

inline bool lds_mark_eligible(int64_t n, int64_t nnz) {
  return nnz >= kLdsMinNnz && n > 0 && n <= kLdsMaxPasses * kLdsCols;
}

// Wider column ranges: the entries are first partitioned by column range (count, offsets, scatter:
// streaming passes over colidx with LDS counters), then every range is marked from its own bucket
// by one workgroup whose LDS holds one flag BYTE per column (plain stores: LDS atomics run at about
// one lane per five clocks, a bit per column would cost more than the byte flags in memory do) and
// which turns the bytes into the range's membership words itself.  Byte flags in memory cost one
// cache-line fill per entry; this costs three streaming passes.
constexpr int64_t kBktCols = 155648;                // columns per range: 152 KB of flag bytes, a multiple of 64
constexpr int kBktMaxRanges = 2048;
constexpr int kBktGroups = 256;                     // workgroups of the partition passes
constexpr int kBktThreads = 1024;                   // their size: 16 wavefronts keep enough loads in flight
inline int64_t bucket_ranges(int64_t n) { return ceil_div(n > 0 ? n : 1, kBktCols); }
inline bool bucket_mark_eligible(int64_t n, int64_t nnz) {
  return nnz >= kLdsMinNnz && n > kLdsMaxPasses * kLdsCols && bucket_ranges(n) <= kBktMaxRanges;
}

struct PlanWs {
  uint8_t* flag;      // n bytes (rounded up to 64W)
  uint64_t* bitmap;   // W words
  int32_t* prefix;    // W + 1
  uint4* rank16;      // W: {word lo, word hi, prefix, 0}: one 16-byte lookup per remapped entry
  int32_t* blocksum;  // nblk + 1
  int64_t* colblk;    // nb + 1 (device copy of the block boundaries)
  int64_t* blkoff;    // the record of the call: {done, err, blkoff[nb + 1]} (calls without a host record)
  int32_t* err;       // 4 counters
  uint32_t* part;     // LDS marking only: kLdsGroups private bitmaps of kLdsWords words
  int32_t* bkt_cols;  // bucketed marking only: the column ids partitioned by range (nnz)
  int32_t* bkt_place; // bucketed marking only: where in bkt_cols every entry went (nnz; -1: column out of range)
  int32_t* bkt_cnt;   // bucketed marking only: [ranges][kBktGroups] counts, then offsets inside the range
  int32_t* bkt_start; // bucketed marking only: first entry of every range (+ total)
  int64_t W, nblk;
  size_t bytes;
};

PlanWs carve(void* base, int64_t n, int32_t nb, int64_t nnz) {
  PlanWs w;
  w.W = ceil_div(n > 0 ? n : 1, 64);
  w.nblk = ceil_div(w.W, kWordsPerBlock);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += round_up(bytes, 256);
    return reinterpret_cast<char*>(base) + o;
  };
  w.flag = reinterpret_cast<uint8_t*>(take((size_t)w.W * 64));
  w.bitmap = reinterpret_cast<uint64_t*>(take(sizeof(uint64_t) * (size_t)w.W));
  w.prefix = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(w.W + 1)));
  w.rank16 = reinterpret_cast<uint4*>(take(sizeof(uint4) * (size_t)w.W));
  w.blocksum = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(w.nblk + 1)));
  w.colblk = reinterpret_cast<int64_t*>(take(sizeof(int64_t) * (size_t)(nb + 1)));
  w.blkoff = reinterpret_cast<int64_t*>(take(sizeof(int64_t) * (size_t)(nb + 4)));
  w.err = reinterpret_cast<int32_t*>(take(256));
  const bool bucketed = bucket_mark_eligible(n, nnz);
  w.part = lds_mark_eligible(n, nnz)
               ? reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)kLdsGroups * kLdsWords))
               : nullptr;
  w.bkt_cols = bucketed ? reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)nnz)) : nullptr;
  w.bkt_place = bucketed ? reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)nnz)) : nullptr;
  w.bkt_cnt = bucketed ? reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(bucket_ranges(n) * kBktGroups)))
                       : nullptr;
  w.bkt_start = bucketed ? reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(bucket_ranges(n) + 1))) : nullptr;
  w.bytes = off;
  return w;
}

__device__ __forceinline__ int64_t ceil_div_dev(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Whether the outputs may be written: the rows fit and, where asked for, the CSR is valid.
struct Verdict {
  const int32_t* total;    // N
  int64_t cap;
  const int32_t* err;      // NULL: not asked
  __device__ __forceinline__ bool go() const {
    return (int64_t)*total <= cap && !(err && (err[0] || err[1]));
  }
};

// What a call reports, in pinned host memory (or, for calls that may not allocate, in the workspace).
struct PlanRecord {
  int64_t done;            // the call's ticket, written last
  int32_t err[4];          // [0] rowptr malformed, [1] column out of range
  int64_t blkoff[1];       // nb + 1
};

__device__ __forceinline__ void report_done(PlanRecord* rec, int64_t ticket) {
  __threadfence_system();
  __hip_atomic_store(&rec->done, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kThreads) void clear_kernel(uint4* __restrict__ flag16, int64_t n16,
                                                         int32_t* __restrict__ err,
                                                         int32_t* __restrict__ blocksum, int64_t nblk) {
  const int64_t t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x, stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = t0; i < n16; i += stride) flag16[i] = make_uint4(0u, 0u, 0u, 0u);
  for (int64_t i = t0; i < nblk; i += stride) blocksum[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 4) err[threadIdx.x] = 0;
}

// Sparsity-oblivious plan: every column of [0, n) counts as needed (the whole block row of H
// is transferred, Sec. 4.1 "sparsity-oblivious algorithm"); bytes past n stay clear.
__global__ __launch_bounds__(kThreads) void fill_all_kernel(uint8_t* __restrict__ flag, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x; c < n; c += stride) flag[c] = 1;
}

// err[0]: rowptr malformed, err[1]: column out of range
__global__ __launch_bounds__(kThreads) void validate_rowptr_kernel(
    const int32_t* __restrict__ rowptr, int64_t m, int64_t nnz, int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x; r < m; r += stride)
    if (rowptr[r] > rowptr[r + 1]) err[0] = 1;
  if (blockIdx.x == 0 && threadIdx.x == 0)
    if (rowptr[0] != 0 || (int64_t)rowptr[m] != nnz) err[0] = 1;
}

__device__ __forceinline__ void mark_one(int32_t c, int64_t n, uint8_t* __restrict__ flag,
                                         int32_t* __restrict__ err) {
  if (c < 0 || c >= n) {
    err[1] = 1;
    return;
  }
  // benign race: all writers store 1.  Testing first is measurably faster than storing
  // unconditionally on power-law graphs (hub columns are hit thousands of times).
  if (flag[c] == 0) flag[c] = 1;
}

// 4 entries per thread per iteration (16-byte loads when the index array is aligned).  (Issuing
// the probes of eight entries before the first store was measured slower: 546 against 517 us on
// 27 M entries over 111 M columns -- the kernel is bound by the line fills, not by their latency.)
__global__ __launch_bounds__(kThreads) void mark_kernel(const int32_t* __restrict__ colidx,
                                                        int64_t nnz, int64_t n,
                                                        uint8_t* __restrict__ flag,
                                                        int32_t* __restrict__ err, int aligned) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  const int64_t quads = nnz >> 2;
  if (aligned) {
    const int4* __restrict__ c4 = reinterpret_cast<const int4*>(colidx);
    for (int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x; q < quads; q += stride) {
      const int4 c = c4[q];
      mark_one(c.x, n, flag, err);
      mark_one(c.y, n, flag, err);
      mark_one(c.z, n, flag, err);
      mark_one(c.w, n, flag, err);
    }
    for (int64_t e = (quads << 2) + (int64_t)blockIdx.x * kThreads + threadIdx.x; e < nnz; e += stride)
      mark_one(colidx[e], n, flag, err);
  } else {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < nnz; e += stride)
      mark_one(colidx[e], n, flag, err);
  }
}

// --- LDS marking ---------------------------------------------------------------------------
// Byte probes into a flag array cost one cache-line fill each (the array is far larger than
// a CU's L1), which is what bounds mark_kernel.  When a few LDS-sized bitmaps cover all
// columns, a workgroup instead ORs the bits of its share of the entries into a private LDS
// bitmap of one column range (pass), reading colidx once per pass as a stream, and writes
// the bitmap out; merge_kernel ORs the private bitmaps into the membership words.
// c0, cols: the range; a column outside [0, n) lies in no range.  Test first: lanes that read one
// address are served by a broadcast, lanes that update one address are serialised, and hub columns
// come up thousands of times.  The words of all N entries are read before the first is tested
// (entry by entry the reads wait for each other).
template <int N>
__device__ __forceinline__ void lds_mark(const int32_t (&c)[N], uint32_t c0, uint32_t cols, uint32_t* bits) {
  uint32_t rel[N], word[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    rel[i] = (uint32_t)c[i] - c0;
    word[i] = __hip_atomic_load(&bits[rel[i] < cols ? rel[i] >> 5 : 0u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (rel[i] < cols && ((word[i] >> (rel[i] & 31)) & 1u) == 0u)
      __hip_atomic_fetch_or(&bits[rel[i] >> 5], 1u << (rel[i] & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// `spec` (may be NULL): also write the range-checked copy of colidx that the remap is if every
// column turns out to be needed (a whole graph planned as one block): the entries are in registers
// anyway, and the separate copy pass is then skipped.  The workgroups of the column ranges take
// turns at that and at the check of the range, so that those of one share, which lie on one XCD
// for two and four ranges, go through the entries together and the second read finds them in its
// L2.  The next sixteen entries of a thread are requested before the present ones are marked.
// Bound by HBM: 125 M entries, 2.45 M columns, one read and one write of 500 MB; 267 us with all
// copies made by the workgroups of the first range and nothing requested ahead, now 242 (the copy
// past the caches 268); 5 M entries over 123 k columns 20, now 16.
__device__ __forceinline__ int32_t identity_or_bad(int32_t c, int64_t n) { return (c < 0 || c >= n) ? -1 : c; }

__global__ __launch_bounds__(kLdsThreads) void mark_lds_kernel(const int32_t* __restrict__ colidx,
                                                               int64_t nnz, int64_t n,
                                                               int32_t groups_per_pass,
                                                               uint32_t* __restrict__ part,
                                                               int32_t* __restrict__ err, int aligned,
                                                               int32_t* __restrict__ spec,
                                                               int32_t* __restrict__ blocksum, int64_t nblk) {
  extern __shared__ __attribute__((aligned(16))) uint32_t bits[];
  if (blockIdx.x == 0)   // (merge_kernel adds to them)
    for (int64_t i = threadIdx.x; i < nblk; i += kLdsThreads) blocksum[i] = 0;
  const int pass = blockIdx.x / groups_per_pass, share = blockIdx.x % groups_per_pass, passes = gridDim.x / groups_per_pass;
  const int64_t c0 = (int64_t)pass * kLdsCols;
  const uint32_t c0w = (uint32_t)c0, cols = (uint32_t)(n - c0 < kLdsCols ? n - c0 : kLdsCols);
  uint4* b4 = reinterpret_cast<uint4*>(bits);
  for (int i = threadIdx.x; i < kLdsWords / 4; i += kLdsThreads) b4[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  bool bad = false;
  auto copy4 = [&](const int4& c, int64_t q) {
    const int4 d = make_int4(identity_or_bad(c.x, n), identity_or_bad(c.y, n), identity_or_bad(c.z, n), identity_or_bad(c.w, n));
    bad |= (d.x | d.y | d.z | d.w) < 0;
    if (spec) reinterpret_cast<int4*>(spec)[q] = d;
  };
  if (aligned) {
    const int64_t quads = nnz >> 2;
    const int64_t per = ceil_div_dev(quads, groups_per_pass);
    const int64_t q0 = (int64_t)share * per;
    const int64_t q1 = q0 + per < quads ? q0 + per : quads;
    const int4* __restrict__ c4 = reinterpret_cast<const int4*>(colidx);
    int turn = pass;                       // 0: this workgroup copies
    int64_t q = q0;
    int4 c[4];
    if (q + 4 * kLdsThreads <= q1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = c4[q + j * kLdsThreads + threadIdx.x];
    }
    for (; q + 4 * kLdsThreads <= q1; q += 4 * kLdsThreads) {
      int4 next[4] = {};
      const int64_t qn = q + 4 * kLdsThreads;
      if (qn + 4 * kLdsThreads <= q1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) next[j] = c4[qn + j * kLdsThreads + threadIdx.x];
      }
      if (turn == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) copy4(c[j], q + j * kLdsThreads + threadIdx.x);
      }
      turn = turn == 0 ? passes - 1 : turn - 1;
      const int32_t all[16] = {c[0].x, c[0].y, c[0].z, c[0].w, c[1].x, c[1].y, c[1].z, c[1].w,
                               c[2].x, c[2].y, c[2].z, c[2].w, c[3].x, c[3].y, c[3].z, c[3].w};
      lds_mark(all, c0w, cols, bits);
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = next[j];
    }
    for (q += threadIdx.x; q < q1; q += kLdsThreads) {
      const int4 t = c4[q];
      if (turn == 0) copy4(t, q);
      const int32_t all[4] = {t.x, t.y, t.z, t.w};
      lds_mark(all, c0w, cols, bits);
    }
    if (share == 0)
      for (int64_t e = (quads << 2) + threadIdx.x; e < nnz; e += kLdsThreads) {
        const int32_t t = colidx[e];
        bad |= identity_or_bad(t, n) < 0;
        if (spec && pass == 0) spec[e] = identity_or_bad(t, n);
        const int32_t one[1] = {t};
        lds_mark(one, c0w, cols, bits);
      }
  } else {
    const int64_t per = ceil_div_dev(nnz, groups_per_pass);
    const int64_t e0 = (int64_t)share * per;
    const int64_t e1 = e0 + per < nnz ? e0 + per : nnz;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kLdsThreads) {
      const int32_t t = colidx[e];
      bad |= identity_or_bad(t, n) < 0;
      if (spec && pass == 0) spec[e] = identity_or_bad(t, n);
      const int32_t one[1] = {t};
      lds_mark(one, c0w, cols, bits);
    }
  }
  if (bad) err[1] = 1;
  __syncthreads();
  // only the words that cover columns below n are ever read back
  const int64_t cols_here = n - c0 < kLdsCols ? n - c0 : kLdsCols;
  const int used4 = cols_here > 0 ? (int)((cols_here + 127) >> 7) : 0;
  uint4* __restrict__ out = reinterpret_cast<uint4*>(part + (size_t)blockIdx.x * kLdsWords);
  for (int i = threadIdx.x; i < used4; i += kLdsThreads) out[i] = b4[i];
}

// --- bucketed marking ------------------------------------------------------------------------
// entries of workgroup g: [g * per, (g + 1) * per); cnt[b * kBktGroups + g] = its entries in range b
//
// Columns are ascending inside a row, so neighbouring lanes often fall into the same range (about
// 13 of 64 lanes share one on an R-MAT block) and their LDS atomics on one counter would run one
// after the other.  A run of equal ranges in adjacent lanes is therefore counted by its first lane
// alone: heads = lanes whose lower neighbour differs, the run's length comes from the ballot of heads.
struct LaneRun {
  int head;    // first lane of this lane's run
  int len;     // length of the run (meaningful in its first lane)
  bool first;
};
__device__ __forceinline__ LaneRun lane_run(int32_t b, int lane) {
  const int32_t prev = __shfl_up(b, 1, 64);
  LaneRun r;
  r.first = lane == 0 || prev != b;
  const uint64_t heads = __ballot(r.first);
  r.head = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
  const uint64_t above = lane == 63 ? 0ull : heads >> (lane + 1);
  r.len = above ? __ffsll((long long)above) : 64 - lane;
  return r;
}

// per workgroup: how many of its entries fall into every range (out-of-range columns are flagged and left out)
__global__ __launch_bounds__(kBktThreads) void bucket_count_kernel(const int32_t* __restrict__ colidx, int64_t nnz,
                                                                int64_t n, int32_t nbk, int32_t* __restrict__ cnt,
                                                                int32_t* __restrict__ err,
                                                                int32_t* __restrict__ blocksum, int64_t nblk) {
  __shared__ int32_t h[kBktMaxRanges];
  if (blockIdx.x == 0)   // (mark_bucket_kernel adds to them)
    for (int64_t i = threadIdx.x; i < nblk; i += kBktThreads) blocksum[i] = 0;
  for (int b = threadIdx.x; b < nbk; b += kBktThreads) h[b] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int64_t per = ceil_div_dev(nnz, kBktGroups);
  const int64_t e0 = (int64_t)blockIdx.x * per, e1 = e0 + per < nnz ? e0 + per : nnz;
  // eight independent loads per thread in flight; the trip count is the same for every lane (ballots inside)
  for (int64_t base = e0; base < e1; base += 8 * kBktThreads) {
    const int64_t e = base + threadIdx.x;
    int32_t c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = e + j * kBktThreads < e1 ? colidx[e + j * kBktThreads] : 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      int32_t b = -1;                                    // past the end or out of range: no bucket
      if (e + j * kBktThreads < e1) {
        if (c[j] < 0 || c[j] >= n) err[1] = 1;
        else b = (int32_t)((uint32_t)c[j] / (uint32_t)kBktCols);
      }
      const LaneRun r = lane_run(b, lane);
      if (r.first && b >= 0) atomicAdd(&h[b], r.len);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbk; b += kBktThreads) cnt[(int64_t)b * kBktGroups + blockIdx.x] = h[b];
}

// one workgroup per range: the counts of the kBktGroups workgroups become offsets inside the
// range, the range's total goes to tot[range]
__global__ __launch_bounds__(kBktGroups) void bucket_within_kernel(int32_t* __restrict__ cnt, int32_t* __restrict__ tot) {
  __shared__ int32_t wsum[kBktGroups / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t* __restrict__ c = cnt + (int64_t)blockIdx.x * kBktGroups;
  const int32_t v = c[threadIdx.x];
  int32_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int32_t before = 0;
  for (int j = 0; j < w; ++j) before += wsum[j];
  c[threadIdx.x] = before + inc - v;
  if (threadIdx.x == kBktGroups - 1) tot[blockIdx.x] = before + inc;
}

// exclusive scan in place of the range totals (nbk <= kBktMaxRanges), grand total to a[nbk]; one workgroup
__global__ __launch_bounds__(1024) void bucket_starts_kernel(int32_t* __restrict__ a, int32_t nbk) {
  __shared__ int32_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i0 = threadIdx.x * 2;
  const int32_t v0 = i0 < nbk ? a[i0] : 0, v1 = i0 + 1 < nbk ? a[i0 + 1] : 0;
  int32_t inc = v0 + v1;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int32_t before = 0;
  for (int j = 0; j < w; ++j) before += wsum[j];
  const int32_t excl = before + inc - v0 - v1;
  __syncthreads();
  if (i0 < nbk) a[i0] = excl;
  if (i0 + 1 < nbk) a[i0 + 1] = excl + v0;
  if (threadIdx.x == 1023) a[nbk] = before + inc;
}

// Every workgroup places its entries behind its own offset of every range.  A batch of 8192 entries
// is first sorted by range inside LDS (count per range, scan, place; runs of adjacent lanes with one
// range share one atomic) and then written out in that order, so that neighbouring lanes store to
// neighbouring places of one range (about a dozen entries per range and batch on a wide block)
// instead of to as many ranges as there are lanes.
constexpr int kBktBatch = 8 * kBktThreads;
__global__ __launch_bounds__(kBktThreads) void bucket_scatter_kernel(const int32_t* __restrict__ colidx, int64_t nnz,
                                                                  int64_t n, int32_t nbk,
                                                                  const int32_t* __restrict__ within,
                                                                  const int32_t* __restrict__ start,
                                                                  int32_t* __restrict__ cols,
                                                                  int32_t* __restrict__ place_e) {
  __shared__ int32_t off[kBktMaxRanges];   // this workgroup's next free place in every range
  __shared__ int32_t cur[kBktMaxRanges];   // batch: entries per range
  __shared__ int32_t cs[kBktMaxRanges];    // batch: first staged position of every range
  __shared__ int32_t stage[kBktBatch];
  __shared__ int32_t wsum[kBktThreads / 64];
  static_assert(kBktMaxRanges == 2 * kBktThreads, "a thread scans two ranges");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b0 = 2 * tid, b1 = 2 * tid + 1;                      // the two ranges this thread keeps
  off[b0] = b0 < nbk ? start[b0] + within[(int64_t)b0 * kBktGroups + blockIdx.x] : 0;
  off[b1] = b1 < nbk ? start[b1] + within[(int64_t)b1 * kBktGroups + blockIdx.x] : 0;
  cur[b0] = 0;
  cur[b1] = 0;
  __syncthreads();
  const int64_t per = ceil_div_dev(nnz, kBktGroups);
  const int64_t e0 = (int64_t)blockIdx.x * per, e1 = e0 + per < nnz ? e0 + per : nnz;
  for (int64_t base = e0; base < e1; base += kBktBatch) {
    const int64_t e = base + tid;
    int32_t c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = e + j * kBktThreads < e1 ? colidx[e + j * kBktThreads] : -1;
    // count per range; the value an atomic returns is the entry's place among its range's entries of
    // this batch, so one pass of LDS atomics (about one lane per clock) serves both the counts and the order
    int32_t b[8], rank[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      b[j] = (c[j] < 0 || c[j] >= n) ? -1 : (int32_t)((uint32_t)c[j] / (uint32_t)kBktCols);
      const LaneRun r = lane_run(b[j], lane);
      int32_t first_rank = 0;
      if (r.first && b[j] >= 0) first_rank = atomicAdd(&cur[b[j]], r.len);
      rank[j] = __shfl(first_rank, r.head, 64) + (lane - r.head);
    }
    __syncthreads();
    // exclusive scan of the counts: cs = first staged position of a range
    const int v0 = cur[b0], v1 = cur[b1];
    int inc = v0 + v1;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kBktThreads / 64; ++w) {
      if (w < wave) before += wsum[w];
      total += wsum[w];
    }
    const int ex = before + inc - (v0 + v1);
    cs[b0] = ex;
    cs[b1] = ex + v0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // (the order inside a range does not matter: the marks are a set)
      if (b[j] >= 0) {
        const int32_t pos = cs[b[j]] + rank[j];
        if (pos >= 0 && pos < kBktBatch) stage[pos] = c[j];
      }
      // where the entry ends up in the partitioned array (the remap finds its rank there)
      if (place_e && e + j * kBktThreads < e1) place_e[e + j * kBktThreads] = b[j] >= 0 ? off[b[j]] + rank[j] : -1;
    }
    __syncthreads();
    for (int i = tid; i < total; i += kBktThreads) {
      const int32_t col = stage[i];
      const int32_t rb = (int32_t)((uint32_t)col / (uint32_t)kBktCols);
      const int64_t place = (int64_t)off[rb] + (i - cs[rb]);
      if (place >= 0 && place < nnz) cols[place] = col;
    }
    __syncthreads();
    off[b0] += cur[b0];
    off[b1] += cur[b1];
    cur[b0] = 0;
    cur[b1] = 0;
    __syncthreads();
  }
}

// The remap of a wide block from the partitioned entries.  Looked up in entry order, every rank
// costs a line of a table that no L2 holds (27.7 MB of rank records for 111 M columns).  In range
// order the records of one range (39 KB) sit in LDS: a workgroup per range replaces every
// column id of its bucket by the column's rank, in place; the entries then fetch their rank from
// the place the scatter noted for them.  That gather is local: a workgroup's share of the entries
// went to its own segment of every range, a few lines per range that stay in L2 while the share
// is walked.
__global__ __launch_bounds__(kLdsThreads) void remap_bucket_kernel(int32_t* __restrict__ cols,
                                                                   const int32_t* __restrict__ start, int64_t nnz,
                                                                   int64_t n, int64_t W,
                                                                   const uint4* __restrict__ rank16,
                                                                   const Verdict vd) {
  if (!vd.go()) return;
  // per 32 columns: {membership bits, needed columns before them}: a lookup is one 8-byte LDS read
  __shared__ uint2 rec[kBktCols / 32];
  const int range = blockIdx.x;
  const int64_t w0 = (int64_t)range * (kBktCols / 64);
  for (int i = threadIdx.x; i < (int)(kBktCols / 64); i += kLdsThreads) {
    const uint4 t = w0 + i < W ? rank16[w0 + i] : make_uint4(0u, 0u, 0u, 0u);
    rec[2 * i] = make_uint2(t.x, t.z);
    rec[2 * i + 1] = make_uint2(t.y, t.z + (uint32_t)__popc(t.x));
  }
  __syncthreads();
  const int64_t c0 = (int64_t)range * kBktCols;
  int64_t e0 = start[range], e1 = start[range + 1];
  e0 = e0 < 0 ? 0 : e0;
  e1 = e1 > nnz ? nnz : e1;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 8 * kLdsThreads) {
    int32_t c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = e + j * kLdsThreads < e1 ? cols[e + j * kLdsThreads] : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (e + j * kLdsThreads >= e1) continue;
      const int64_t rel = (int64_t)c[j] - c0;
      int32_t rk = -1;
      if (rel >= 0 && rel < kBktCols && c[j] < n) {
        const uint2 t = rec[rel >> 5];
        rk = (int32_t)t.y + __popc(t.x & ((1u << (rel & 31)) - 1u));
      }
      cols[e + j * kLdsThreads] = rk;
    }
  }
}

// compact[e] = rank found at the entry's place (same shares of the entries as the scatter)
__global__ __launch_bounds__(kBktThreads) void remap_gather_kernel(const int32_t* __restrict__ place_e,
                                                                  const int32_t* __restrict__ ranks, int64_t nnz,
                                                                  int32_t* __restrict__ compact, const Verdict vd) {
  if (!vd.go()) return;
  const int64_t per = ceil_div_dev(nnz, kBktGroups);
  const int64_t e0 = (int64_t)blockIdx.x * per, e1 = e0 + per < nnz ? e0 + per : nnz;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 8 * kBktThreads) {
    int32_t p[8], r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = e + j * kBktThreads < e1 ? __builtin_nontemporal_load(&place_e[e + j * kBktThreads]) : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = (p[j] >= 0 && p[j] < nnz) ? ranks[p[j]] : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (e + j * kBktThreads < e1) __builtin_nontemporal_store(r[j], &compact[e + j * kBktThreads]);
  }
}

// one workgroup per range: flag bytes in LDS from the range's bucket, then the range's membership
// words (kBktCols / 64 of them, the last range fewer) straight into the bitmap
__global__ __launch_bounds__(kLdsThreads) void mark_bucket_kernel(const int32_t* __restrict__ cols,
                                                                  const int32_t* __restrict__ start, int64_t nnz,
                                                                  int64_t n, int64_t W, uint64_t* __restrict__ bm,
                                                                  int32_t* __restrict__ blocksum) {
  __shared__ int32_t tally[kBktCols / 64 / kWordsPerBlock + 2];   // set bits per tile of words the range touches
  if (threadIdx.x < sizeof(tally) / sizeof(tally[0])) tally[threadIdx.x] = 0;
  extern __shared__ __attribute__((aligned(16))) uint32_t bits[];
  uint8_t* flag = reinterpret_cast<uint8_t*>(bits);
  const int range = blockIdx.x;
  const int64_t c0 = (int64_t)range * kBktCols;
  uint4* b4 = reinterpret_cast<uint4*>(bits);
  int64_t e0 = start[range], e1 = start[range + 1];
  e0 = e0 < 0 ? 0 : e0;
  e1 = e1 > nnz ? nnz : e1;
  // sixteen loads per thread in flight, the first batch requested before the flags are cleared (one
  // workgroup per CU: nothing else hides the latency of the stream)
  constexpr int U = 16;
  int32_t c[U];
#pragma unroll
  for (int j = 0; j < U; ++j) c[j] = e0 + threadIdx.x + j * kLdsThreads < e1 ? cols[e0 + threadIdx.x + j * kLdsThreads] : -1;
  for (int i = threadIdx.x; i < (int)(kBktCols / 16); i += kLdsThreads) b4[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  for (int64_t base = e0; base < e1; base += U * kLdsThreads) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int64_t rel = (int64_t)c[j] - c0;
      if (c[j] >= 0 && rel >= 0 && rel < kBktCols) flag[rel] = 1;
    }
    const int64_t en = base + U * kLdsThreads + threadIdx.x;
#pragma unroll
    for (int j = 0; j < U; ++j) c[j] = en + j * kLdsThreads < e1 ? cols[en + j * kLdsThreads] : -1;
  }
  __syncthreads();
  // 64 flag bytes -> one word: a lane squeezes its 8 bytes into 8 bits, eight lanes make a word
  const int64_t w0 = c0 >> 6;
  const int words_here = (int)((W - w0 < kBktCols / 64) ? (W - w0) : (kBktCols / 64));
  const uint2* f8 = reinterpret_cast<const uint2*>(bits);
  for (int i = threadIdx.x; i < words_here * 8; i += kLdsThreads) {
    const uint2 t = f8[i];
    // bytes are 0 or 1: gather bit 0 of every byte
    const uint32_t lo = ((t.x & 0x01010101u) * 0x01020408u) >> 24;
    const uint32_t hi = ((t.y & 0x01010101u) * 0x01020408u) >> 24;
    uint64_t piece = (uint64_t)((lo & 0xFu) | ((hi & 0xFu) << 4)) << ((i & 7) * 8);
    // combine the eight lanes of a word (consecutive lanes)
    piece |= __shfl_xor(piece, 1, 64);
    piece |= __shfl_xor(piece, 2, 64);
    piece |= __shfl_xor(piece, 4, 64);
    if ((i & 7) == 0) {
      const int64_t wi = w0 + (i >> 3);
      const int64_t col = wi * 64;
      if (n - col < 64) piece &= (1ull << (n - col)) - 1ull;
      bm[wi] = piece;
      if (piece) atomicAdd(&tally[wi / kWordsPerBlock - w0 / kWordsPerBlock], __popcll(piece));
    }
  }
  __syncthreads();
  if (threadIdx.x < sizeof(tally) / sizeof(tally[0]) && tally[threadIdx.x])
    atomicAdd(&blocksum[w0 / kWordsPerBlock + threadIdx.x], tally[threadIdx.x]);
}

// Membership words from the private bitmaps.  A workgroup owns 64 consecutive 64-bit words, a lane a word; wavefront sl ORs
// the bitmaps of groups sl, sl + 16, .., LDS combines the 16 slices.  Whole lines of a bitmap, and one sum to a tile's counter
// per 64 words: the counters are few, additions to one of them follow each other across the XCDs, and with 16 words a
// workgroup (128 of them to a counter) that was the kernel: 2 M columns, 128 bitmaps 27 -> 11 us.
constexpr int kMergeWords = 64, kMergeSlices = 16;
__global__ __launch_bounds__(kMergeWords * kMergeSlices) void merge_kernel(const uint32_t* __restrict__ part,
                                                                           int32_t groups_per_pass, int64_t W, int64_t n,
                                                                           uint64_t* __restrict__ bm, int32_t* __restrict__ blocksum) {
  __shared__ uint64_t red[kMergeSlices][kMergeWords];
  const int wi = threadIdx.x % kMergeWords, sl = threadIdx.x / kMergeWords;
  const int64_t w = (int64_t)blockIdx.x * kMergeWords + wi;
  uint64_t word = 0;
  if (w < W) {
    const int64_t col = w * 64;
    const int pass = (int)(col / kLdsCols);          // kLdsCols is a multiple of 64
    const int64_t idx = (col - (int64_t)pass * kLdsCols) >> 5;
    const uint32_t* __restrict__ p = part + ((size_t)pass * groups_per_pass) * kLdsWords + idx;
#pragma unroll 8
    for (int g = sl; g < groups_per_pass; g += kMergeSlices) {
      const uint2 t = *reinterpret_cast<const uint2*>(p + (size_t)g * kLdsWords);
      word |= (uint64_t)t.x | ((uint64_t)t.y << 32);
    }
  }
  red[sl][wi] = word;
  __syncthreads();
  if (sl == 0) {   // (their words lie in one tile)
    int cnt = 0;
    if (w < W) {
#pragma unroll
      for (int j = 1; j < kMergeSlices; ++j) word |= red[j][wi];
      const int64_t col = w * 64;
      if (n - col < 64) word &= (1ull << (n - col)) - 1ull;
      bm[w] = word;
      cnt = __popcll(word);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (wi == 0 && cnt) atomicAdd(&blocksum[w / kWordsPerBlock], cnt);
  }
}

__device__ __forceinline__ int wave_inclusive_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

// exclusive scan over the kThreads threads of a block; returns the exclusive prefix of v and
// the block total through *total
__device__ __forceinline__ int block_exclusive_scan(int v, int* total) {
  __shared__ int wsum[kThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    const int s = wsum[w];
    if (w < wave) base += s;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// Membership words from the flag bytes.  A wavefront makes 64 words, 16 (1024 flag bytes) per step: a lane loads 16
// flags with one 16-byte load and squeezes them into 16 bits (flags are 0 or 1: a multiply gathers the low
// bit of every byte), four neighbouring lanes OR their quarters into one word.  (2048 words per workgroup, so that its
// sum was the tile's, was a chain of 32 loads: 14 us for 100 k columns, now 4.)
__device__ __forceinline__ uint32_t squeeze8(uint64_t x) {
  return (uint32_t)(((x & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
}

constexpr int kWordsPerGroup = kThreads;   // 64 per wavefront
__global__ __launch_bounds__(kThreads) void words_kernel(const uint8_t* __restrict__ flag, int64_t W,
                                                         uint64_t* __restrict__ bm,
                                                         int32_t* __restrict__ blocksum) {
  __shared__ int wsum[kThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  static_assert(kWordsPerBlock % kWordsPerGroup == 0, "a workgroup's words lie in one tile");
  const int64_t w0 = (int64_t)blockIdx.x * kWordsPerGroup + (int64_t)wave * 64;
  const ulonglong2* __restrict__ f16 = reinterpret_cast<const ulonglong2*>(flag);   // flag is 256-byte aligned
  int cnt = 0;
  ulonglong2 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = make_ulonglong2(0ull, 0ull);
    if (w0 + i * 16 + (lane >> 2) < W) v[i] = f16[(w0 + i * 16) * 4 + lane];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t w = w0 + i * 16 + (lane >> 2);
    const uint64_t quarter = (uint64_t)(squeeze8(v[i].x) | (squeeze8(v[i].y) << 8));
    cnt += __popcll(quarter);
    uint64_t word = quarter << (16 * (lane & 3));
    word |= __shfl_xor(word, 1, 64);
    word |= __shfl_xor(word, 2, 64);
    if ((lane & 3) == 0 && w < W) bm[w] = word;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_down(cnt, o, 64);
  if (lane == 0) wsum[wave] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += wsum[w];
    if (t) atomicAdd(&blocksum[w0 / kWordsPerBlock], t);
  }
}

// A tile of kWordsPerBlock words goes through LDS so that both the loads of the words and the
// stores of the prefix counts and rank records are coalesced (thread t of step i moves element
// t + 256 i), while the scan still gives a thread eight consecutive words.
__global__ __launch_bounds__(kThreads) void prefix_kernel(const uint64_t* __restrict__ bm,
                                                          int64_t W,
                                                          const int32_t* __restrict__ blocksum,
                                                          int64_t nblk, int32_t* __restrict__ prefix,
                                                          uint4* __restrict__ rank16) {
  __shared__ uint64_t words[kWordsPerBlock];
  __shared__ int32_t pre[kWordsPerBlock];
  __shared__ int32_t wbase[kThreads / 64];
  const int64_t tile0 = (int64_t)blockIdx.x * kWordsPerBlock;
  int32_t base = 0;                                   // set bits of the tiles before this one
  for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kThreads) base += blocksum[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) base += __shfl_xor(base, o, 64);
  if ((threadIdx.x & 63) == 0) wbase[threadIdx.x >> 6] = base;
#pragma unroll
  for (int i = 0; i < kWordsPerBlock / kThreads; ++i) {
    const int j = threadIdx.x + i * kThreads;
    words[j] = tile0 + j < W ? bm[tile0 + j] : 0ull;
  }
  __syncthreads();
  int c[8];
  int s = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    c[i] = __popcll(words[threadIdx.x * 8 + i]);
    s += c[i];
  }
  base = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) base += wbase[w];
  int total;
  int run = base + block_exclusive_scan(s, &total);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    pre[threadIdx.x * 8 + i] = run;
    run += c[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kWordsPerBlock / kThreads; ++i) {
    const int j = threadIdx.x + i * kThreads;
    if (tile0 + j < W) {
      const uint64_t word = words[j];
      const int32_t p = pre[j];
      prefix[tile0 + j] = p;
      rank16[tile0 + j] = make_uint4((uint32_t)word, (uint32_t)(word >> 32), (uint32_t)p, 0u);
    }
  }
  if ((int64_t)blockIdx.x == nblk - 1 && threadIdx.x == 0) prefix[W] = base + total;
}

__device__ __forceinline__ int32_t remap_one(int32_t c, int64_t n, const uint4* __restrict__ rank16) {
  if (c < 0 || c >= n) return -1;
  const uint4 t = rank16[c >> 6];
  const uint64_t word = (uint64_t)t.x | ((uint64_t)t.y << 32);
  return (int32_t)t.z + __popcll(word & ((1ull << (c & 63)) - 1ull));
}

// Block boundaries: as a kernel argument while they are few (no copy to the device).
constexpr int kArgBlocks = 64;
struct Colblk {
  const int64_t* mem;              // NULL: v holds them
  int64_t v[kArgBlocks + 1];
};

// The last launch: record, needed[], remap.  The first `emit_blocks` workgroups write needed[], the others the remap.
//   needed[]  a wavefront per word; where fewer than eight columns of a word are needed on average a thread per word
//             that walks its set bits (a wavefront would write a handful of ids with 64 lanes)
//   remap     range-checked copy if every column is needed (position = column), else one 16-byte lookup per entry
struct FinishArgs {
  const uint64_t* bm; const int32_t* prefix; const uint4* rank16;
  int64_t W, n, nnz;
  int32_t* needed;
  const int32_t* colidx; int32_t* compact;     // compact == NULL: no remap here
  int32_t identity_done;                       // the remap has been written for the case that all are needed
  int32_t aligned, nb, emit_blocks;
  PlanRecord* rec; int64_t ticket;
  Verdict vd;
};

__global__ __launch_bounds__(kThreads) void finish_kernel(const FinishArgs a, const Colblk cb) {
  const int64_t N = a.prefix[a.W];
  if (blockIdx.x == 0) {
    if (threadIdx.x < 4) a.rec->err[threadIdx.x] = a.vd.err ? a.vd.err[threadIdx.x] : 0;
    for (int q = threadIdx.x; q <= a.nb; q += kThreads) {
      const int64_t c = cb.mem ? cb.mem[q] : cb.v[q];
      const int64_t w = c >> 6;
      a.rec->blkoff[q] = (c >= a.n || w >= a.W) ? N : (int64_t)a.prefix[w] + __popcll(a.bm[w] & ((1ull << (c & 63)) - 1ull));
    }
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) report_done(a.rec, a.ticket);
  }
  if (!a.vd.go()) return;
  if ((int)blockIdx.x < a.emit_blocks) {
    const int64_t t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x, stride = (int64_t)a.emit_blocks * kThreads;
    if (N * 8 < a.n) {
      for (int64_t w = t0; w < a.W; w += stride) {
        uint64_t word = a.bm[w];
        if (word == 0ull) continue;
        int64_t pos = a.prefix[w];
        const int64_t base = w * 64;
        while (word) {
          const int b = __builtin_ctzll(word);
          word &= word - 1ull;
          if (base + b < a.n) a.needed[pos++] = (int32_t)(base + b);
        }
      }
    } else {
      const int lane = threadIdx.x & 63;
      for (int64_t w = t0 >> 6; w < a.W; w += stride >> 6) {
        const uint64_t word = a.bm[w];
        const int64_t c = w * 64 + lane;
        const bool set = ((word >> lane) & 1ull) != 0 && c < a.n;
        const uint64_t mask = __ballot(set);
        const int slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
        if (set) a.needed[(int64_t)a.prefix[w] + slot] = (int32_t)c;
      }
    }
    return;
  }
  if (!a.compact) return;
  const bool identity = N == a.n;
  if (identity && a.identity_done) return;
  const int64_t t0 = (int64_t)(blockIdx.x - a.emit_blocks) * kThreads + threadIdx.x;
  const int64_t stride = (int64_t)(gridDim.x - a.emit_blocks) * kThreads;
  const int64_t quads = a.aligned ? (a.nnz >> 2) : 0;
  const int4* __restrict__ c4 = reinterpret_cast<const int4*>(a.colidx);
  int4* __restrict__ o4 = reinterpret_cast<int4*>(a.compact);
  if (identity) {
    for (int64_t q = t0; q < quads; q += stride) {
      const int4 c = c4[q];
      o4[q] = make_int4(identity_or_bad(c.x, a.n), identity_or_bad(c.y, a.n), identity_or_bad(c.z, a.n),
                        identity_or_bad(c.w, a.n));
    }
    for (int64_t e = (quads << 2) + t0; e < a.nnz; e += stride) a.compact[e] = identity_or_bad(a.colidx[e], a.n);
    return;
  }
  for (int64_t q = t0; q < quads; q += stride) {
    const int4 c = c4[q];
    int4 o;
    o.x = remap_one(c.x, a.n, a.rank16);
    o.y = remap_one(c.y, a.n, a.rank16);
    o.z = remap_one(c.z, a.n, a.rank16);
    o.w = remap_one(c.w, a.n, a.rank16);
    o4[q] = o;
  }
  for (int64_t e = (quads << 2) + t0; e < a.nnz; e += stride) a.compact[e] = remap_one(a.colidx[e], a.n, a.rank16);
}

inline unsigned grid_for(int64_t items, int64_t per_thread = 1) {
  int64_t b = ceil_div(ceil_div(items, per_thread), kThreads);
  const int64_t cap = 256 * 32;  // enough workgroups to fill 256 CUs several times over
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (unsigned)b;
}

}  // namespace
}  // namespace sagnn

SAGNN_EXPORT int spmm_plan_workspace_bytes(int64_t m, int64_t n, int64_t nnz, int32_t nb,
                                           size_t* bytes) {
  using namespace sagnn;
  if (!bytes || m < 0 || n < 0 || nnz < 0 || nb < 1 || n > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  *bytes = carve(nullptr, n, nb, nnz).bytes;
  return SAGNN_OK;
}

namespace sagnn {
namespace {

// ---------------------------------------------------------------------------------------------
// Small blocks (the launch-latency regime: a few thousand rows and columns): the whole plan in one
// launch.  Every workgroup marks all entries in its own LDS (they are few, and no workgroup then waits for another)
// and counts and ranks the columns; the first one writes the record, the others their shares of needed[] and of the
// remap.
// One flag byte per column where they fit (plain stores: LDS atomics, one lane per clock, were half of the
// kernel's time), bits beyond.  Same results as the general path: needed[] ascending, remap -1
// for a column outside [0, n), nothing written to needed[] / the remap when N exceeds the
// capacity or the validation fails.  36,864 entries over 4096 columns: 8 us (of which
// launch and report are 7), 16 us by one workgroup with bits.
constexpr int64_t kSmallMaxCols = 262144;   // 4096 membership words of 64 columns
constexpr int64_t kSmallByteCols = 131072;
constexpr int64_t kSmallMaxNnz = 65536;
constexpr int64_t kSmallMaxRows = 262144;
constexpr int32_t kSmallMaxBlocks = 16;
constexpr int kSmallLoads = 40;             // entries a thread has in flight
constexpr int kSmallOwn = 4;                // entries of the remap per thread
struct SmallColblk { int64_t v[kSmallMaxBlocks + 1]; };

// dynamic LDS: words, their ranks, flag bytes
inline size_t small_lds_bytes(int64_t n) {
  const size_t W = (size_t)((n + 63) >> 6);
  return W * 8 + (W + 2) * 4 + (n <= kSmallByteCols ? W * 64 + 32 : 0);   // (one byte more than columns: the bad ones)
}

template <bool BYTES>
__global__ __launch_bounds__(1024) void plan_small_kernel(const int32_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ colidx, int64_t m, int64_t n,
                                                          int64_t nnz, const SmallColblk cb, int32_t nb,
                                                          int32_t* __restrict__ needed, int64_t needed_cap,
                                                          int32_t* __restrict__ compact, int32_t validate,
                                                          PlanRecord* __restrict__ rec, int64_t ticket) {
  extern __shared__ __attribute__((aligned(16))) char small_lds[];
  __shared__ int32_t wsum[16];
  __shared__ int32_t bad[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = (int)((n + 63) >> 6);
  uint64_t* bm = reinterpret_cast<uint64_t*>(small_lds);
  int32_t* pre = reinterpret_cast<int32_t*>(bm + W);
  uint8_t* flag = reinterpret_cast<uint8_t*>((reinterpret_cast<uintptr_t>(pre + W + 1) + 15) & ~(uintptr_t)15);
  if constexpr (BYTES) {
    uint4* f16 = reinterpret_cast<uint4*>(flag);
    for (int i = tid; i < W * 4 + 1; i += 1024) f16[i] = make_uint4(0u, 0u, 0u, 0u);
  } else {
    for (int i = tid; i < W; i += 1024) bm[i] = 0ull;
  }
  if (tid < 2) bad[tid] = 0;
  const int nwg = (int)gridDim.x - 1, wg = (int)blockIdx.x - 1;
  int32_t own[kSmallOwn];
  if (compact && wg >= 0)
#pragma unroll
    for (int j = 0; j < kSmallOwn; ++j) {
      const int64_t e = ((int64_t)wg * kSmallOwn + j) * 1024 + tid;
      own[j] = e < nnz ? colidx[e] : 0;
    }
  __syncthreads();
  if (validate) {
    for (int64_t r = tid; r < m; r += 1024)
      if (rowptr[r] > rowptr[r + 1]) bad[0] = 1;
    if (tid == 0 && (rowptr[0] != 0 || (int64_t)rowptr[m] != nnz)) bad[0] = 1;
  }
  uint32_t* bits = reinterpret_cast<uint32_t*>(bm);   // bit c of the 64-bit word c >> 6 = bit c & 31 of 32-bit word c >> 5
  // (no branch per entry: past the end the last entry is marked again, a bad column marks the byte behind the flags)
  const uint32_t nc = (uint32_t)n;
  const int last = (int)nnz - 1;
  bool off = false;
  for (int e0 = tid; e0 - tid < (int)nnz; e0 += kSmallLoads * 1024) {
    uint32_t c[kSmallLoads];
#pragma unroll
    for (int j = 0; j < kSmallLoads; ++j) c[j] = (uint32_t)colidx[e0 + j * 1024 < last ? e0 + j * 1024 : last];
#pragma unroll
    for (int j = 0; j < kSmallLoads; ++j) {
      off |= c[j] >= nc;
      if constexpr (BYTES) {
        flag[c[j] < nc ? c[j] : (uint32_t)W * 64] = 1;
      } else if (c[j] < nc) {
        const uint32_t bit = 1u << (c[j] & 31);
        if ((__hip_atomic_load(&bits[c[j] >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit) == 0)
          __hip_atomic_fetch_or(&bits[c[j] >> 5], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
  if (off) bad[1] = 1;
  __syncthreads();
  if constexpr (BYTES) {
    // as in words_kernel: a lane squeezes 16 flags, four make a word
    const ulonglong2* f16 = reinterpret_cast<const ulonglong2*>(flag);
    for (int i = tid; i < W * 4; i += 1024) {
      const ulonglong2 v = f16[i];
      uint64_t word = (uint64_t)(squeeze8(v.x) | (squeeze8(v.y) << 8)) << (16 * (lane & 3));
      word |= __shfl_xor(word, 1, 64);
      word |= __shfl_xor(word, 2, 64);
      if ((lane & 3) == 0) bm[i >> 2] = word;
    }
    __syncthreads();
  }
  // prefix counts: thread t owns words 4t .. 4t + 3
  int cnt[4], sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int w = 4 * tid + k;
    cnt[k] = w < W ? __popcll(bm[w]) : 0;
    sum += cnt[k];
  }
  int inc = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int before = 0, N = 0;
  for (int j = 0; j < 16; ++j) {
    if (j < wave) before += wsum[j];
    N += wsum[j];
  }
  int run = before + inc - sum;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int w = 4 * tid + k;
    if (w < W) pre[w] = run;
    run += cnt[k];
  }
  if (tid == 0) pre[W] = N;
  __syncthreads();
  auto rank = [&](int64_t c) -> int32_t {
    if (c >= n) return N;
    const int w = (int)(c >> 6);
    return pre[w] + __popcll(bm[w] & ((1ull << (c & 63)) - 1ull));
  };
  if (wg < 0) {
    if (tid <= nb) rec->blkoff[tid] = rank(cb.v[tid]);
    if (tid < 2) rec->err[tid] = bad[tid];
    // (the lanes that wrote are all in the first wavefront)
    if (tid < 64) __threadfence_system();
    if (tid == 0) report_done(rec, ticket);
    return;
  }
  if ((int64_t)N > needed_cap || (validate && (bad[0] || bad[1]))) return;
  for (int w = wg * 16 + wave; w < W; w += 16 * nwg) {     // one wavefront per word: lane = column, slot from the lanes below
    const uint64_t x = bm[w];
    const bool set = (x >> lane) & 1ull;
    const int slot = __popcll(x & ((1ull << lane) - 1ull));
    if (set) needed[pre[w] + slot] = w * 64 + lane;
  }
  if (compact)
#pragma unroll
    for (int j = 0; j < kSmallOwn; ++j) {
      const int64_t e = ((int64_t)wg * kSmallOwn + j) * 1024 + tid;
      if (e < nnz) compact[e] = (uint32_t)own[j] < nc ? rank(own[j]) : -1;
    }
}

// ---------------------------------------------------------------------------------------------
// Pinned host records.  A call takes one, the kernels write into it, the host watches `done`; then it goes back.
// Idle records are kept (at most kIdleRecords, 16 KB each) because pinning memory costs more than a plan.
constexpr size_t kRecordBytes = 16384;
constexpr int32_t kRecordMaxBlocks = (int32_t)((kRecordBytes - sizeof(PlanRecord)) / sizeof(int64_t));
constexpr int kIdleRecords = 8;
std::mutex g_record_mutex;
PlanRecord* g_records[kIdleRecords] = {};
int g_n_records = 0;
std::atomic<int64_t> g_ticket{1};

PlanRecord* record_take() {
  {
    std::lock_guard<std::mutex> lock(g_record_mutex);
    if (g_n_records > 0) return g_records[--g_n_records];
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, kRecordBytes, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  static_cast<PlanRecord*>(p)->done = 0;
  return static_cast<PlanRecord*>(p);
}

void record_give_back(PlanRecord* r) {
  {
    std::lock_guard<std::mutex> lock(g_record_mutex);
    if (g_n_records < kIdleRecords) {
      g_records[g_n_records++] = r;
      return;
    }
  }
  (void)hipHostFree(r);
}

// Waits until the kernels have written `ticket`; the wait ends with the stream's work at the latest.
int record_wait(const PlanRecord* r, int64_t ticket, hipStream_t s) {
  const volatile int64_t* done = &r->done;
  for (;;) {
    for (int i = 0; i < 4096; ++i) {
      if (*done == ticket) {
        std::atomic_thread_fence(std::memory_order_acquire);
        return SAGNN_OK;
      }
      __builtin_ia32_pause();
    }
    const hipError_t e = hipStreamQuery(s);
    if (e == hipErrorNotReady) continue;
    if (e != hipSuccess) return hip_fail(e);
    if (*done == ticket) return SAGNN_OK;
    return hip_fail(hipErrorUnknown);   // the kernels are done and have not reported: a launch was lost
  }
}

}  // namespace
}  // namespace sagnn

namespace sagnn {
namespace {

// host-side argument checks shared by the two planning entry points (no HIP call is made)
int plan_check_args(const int32_t* d_rowptr, const int32_t* d_colidx, int64_t m, int64_t n,
                    int64_t nnz, const int64_t* h_colblk, int32_t nb, const int32_t* d_needed,
                    int64_t needed_cap, const int64_t* h_blk_off) {
  if (m < 0 || n < 0 || nnz < 0 || nb < 1 || needed_cap < 0 || n > 0x7FFFFFFFll ||
      nnz > 0x7FFFFFFFll || m > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  if (!h_colblk || !h_blk_off || !d_rowptr) return SAGNN_EINVAL;
  if (nnz > 0 && !d_colidx) return SAGNN_EINVAL;
  if (needed_cap > 0 && !d_needed) return SAGNN_EINVAL;
  if (h_colblk[0] != 0 || h_colblk[nb] != n) return SAGNN_EFORMAT;
  for (int32_t q = 0; q < nb; ++q)
    if (h_colblk[q] > h_colblk[q + 1]) return SAGNN_EFORMAT;
  return SAGNN_OK;
}

// The planning pipeline on an already carved workspace (w.part == nullptr: byte-flag marking).  rec: the pinned record
// of the call, or NULL: the record then lies in the workspace and is copied back.
int plan_launch(const int32_t* d_rowptr, const int32_t* d_colidx, int64_t m, int64_t n, int64_t nnz,
                const int64_t* h_colblk, int32_t nb, int32_t* d_needed, int64_t needed_cap, int32_t* d_colidx_compact,
                const PlanWs& w, uint32_t flags, PlanRecord* rec, int64_t ticket, hipStream_t s) {
  if (!rec) rec = reinterpret_cast<PlanRecord*>(w.blkoff);
  const bool validate = (flags & SAGNN_PLAN_VALIDATE) != 0;
  if ((flags & (SAGNN_PLAN_OBLIVIOUS | SAGNN_PLAN_MULTIPASS)) == 0 && n <= kSmallMaxCols && nnz <= kSmallMaxNnz && m <= kSmallMaxRows &&
      nb <= kSmallMaxBlocks) {
    SmallColblk cb{};
    for (int32_t q = 0; q <= nb; ++q) cb.v[q] = h_colblk[q];
    const size_t lds = small_lds_bytes(n);
    const auto kernel = n <= kSmallByteCols ? plan_small_kernel<true> : plan_small_kernel<false>;
    if (lds > 48 * 1024)
      SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    const int64_t by_entry = ceil_div(nnz > 0 ? nnz : 1, kSmallOwn * 1024), by_word = ceil_div(n, 16384);
    const int64_t wgs = 1 + (by_entry > by_word ? by_entry : by_word);   // at most 17
    hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(1024), lds, s, d_rowptr, d_colidx, m, n, nnz, cb, nb,
                       d_needed, needed_cap, d_colidx_compact, validate ? 1 : 0, rec, ticket);
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  }
  Colblk cb{};
  if (nb <= kArgBlocks) {
    for (int32_t q = 0; q <= nb; ++q) cb.v[q] = h_colblk[q];
  } else {
    cb.mem = w.colblk;
    SAGNN_HIP(hipMemcpyAsync(w.colblk, h_colblk, sizeof(int64_t) * (size_t)(nb + 1), hipMemcpyHostToDevice, s));
  }
  const bool oblivious = (flags & SAGNN_PLAN_OBLIVIOUS) != 0;
  const bool bucket_mark = !oblivious && w.bkt_cols != nullptr;
  const bool lds_mark = !oblivious && !bucket_mark && w.part != nullptr;
  int32_t* err = w.err;   // (read only where validation is asked for, and cleared only then)
  if ((!bucket_mark && !lds_mark) || validate) {
    const int64_t clear16 = bucket_mark || lds_mark ? 0 : w.W * 4;
    hipLaunchKernelGGL(clear_kernel, dim3(grid_for(clear16)), dim3(kThreads), 0, s, reinterpret_cast<uint4*>(w.flag),
                       clear16, err, w.blocksum, w.nblk);
    SAGNN_LAUNCH_CHECK();
  }
  if (validate) {
    hipLaunchKernelGGL(validate_rowptr_kernel, dim3(grid_for(m)), dim3(kThreads), 0, s, d_rowptr,
                       m, nnz, err);
    SAGNN_LAUNCH_CHECK();
  }
  bool speculated = false;   // the marking pass has already written the identity remap
  if (bucket_mark) {
    const int32_t nbk = (int32_t)bucket_ranges(n);
    const size_t lds = (size_t)kBktCols;
    hipLaunchKernelGGL(bucket_count_kernel, dim3(kBktGroups), dim3(kBktThreads), 0, s, d_colidx, nnz, n, nbk, w.bkt_cnt,
                       err, w.blocksum, w.nblk);
    SAGNN_LAUNCH_CHECK();
    hipLaunchKernelGGL(bucket_within_kernel, dim3((unsigned)nbk), dim3(kBktGroups), 0, s, w.bkt_cnt, w.bkt_start);
    SAGNN_LAUNCH_CHECK();
    hipLaunchKernelGGL(bucket_starts_kernel, dim3(1), dim3(1024), 0, s, w.bkt_start, nbk);
    SAGNN_LAUNCH_CHECK();
    hipLaunchKernelGGL(bucket_scatter_kernel, dim3(kBktGroups), dim3(kBktThreads), 0, s, d_colidx, nnz, n, nbk,
                       w.bkt_cnt, w.bkt_start, w.bkt_cols, d_colidx_compact ? w.bkt_place : (int32_t*)nullptr);
    SAGNN_LAUNCH_CHECK();
    SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(mark_bucket_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(mark_bucket_kernel, dim3((unsigned)nbk), dim3(kLdsThreads), lds, s, w.bkt_cols, w.bkt_start,
                       nnz, n, w.W, w.bitmap, w.blocksum);
    SAGNN_LAUNCH_CHECK();
  } else if (lds_mark) {
    const int passes = (int)ceil_div(n, kLdsCols);
    const int groups_per_pass = kLdsGroups / passes;
    const size_t lds = sizeof(uint32_t) * (size_t)kLdsWords;
    SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(mark_lds_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    // dense enough that every column is probably needed: write the identity remap on the way
    speculated = d_colidx_compact && nnz >= 8 * n;
    const bool al = aligned16(d_colidx) && (!speculated || aligned16(d_colidx_compact));
    hipLaunchKernelGGL(mark_lds_kernel, dim3((unsigned)(passes * groups_per_pass)), dim3(kLdsThreads),
                       lds, s, d_colidx, nnz, n, (int32_t)groups_per_pass, w.part, err, al ? 1 : 0,
                       speculated ? d_colidx_compact : (int32_t*)nullptr, w.blocksum, w.nblk);
    SAGNN_LAUNCH_CHECK();
    hipLaunchKernelGGL(merge_kernel, dim3((unsigned)ceil_div(w.W, kMergeWords)), dim3(kMergeWords * kMergeSlices), 0, s, w.part,
                       (int32_t)groups_per_pass, w.W, n, w.bitmap, w.blocksum);
    SAGNN_LAUNCH_CHECK();
  } else {
    if (nnz > 0 && (!oblivious || validate)) {
      hipLaunchKernelGGL(mark_kernel, dim3(grid_for(nnz, 8)), dim3(kThreads), 0, s, d_colidx, nnz,
                         n, w.flag, err, aligned16(d_colidx) ? 1 : 0);
      SAGNN_LAUNCH_CHECK();
    }
    if (oblivious && n > 0) {
      hipLaunchKernelGGL(fill_all_kernel, dim3(grid_for(n)), dim3(kThreads), 0, s, w.flag, n);
      SAGNN_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(words_kernel, dim3((unsigned)ceil_div(w.W > 0 ? w.W : 1, kWordsPerGroup)), dim3(kThreads), 0, s, w.flag, w.W,
                       w.bitmap, w.blocksum);
    SAGNN_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(prefix_kernel, dim3((unsigned)w.nblk), dim3(kThreads), 0, s, w.bitmap, w.W,
                     w.blocksum, w.nblk, w.prefix, w.rank16);
  SAGNN_LAUNCH_CHECK();

  FinishArgs fa{};
  fa.bm = w.bitmap; fa.prefix = w.prefix; fa.rank16 = w.rank16; fa.W = w.W; fa.n = n; fa.nnz = nnz;
  fa.needed = d_needed; fa.colidx = d_colidx; fa.compact = bucket_mark ? nullptr : d_colidx_compact;
  fa.identity_done = speculated ? 1 : 0;
  fa.aligned = aligned16(d_colidx) && aligned16(d_colidx_compact) ? 1 : 0;
  fa.nb = nb; fa.rec = rec; fa.ticket = ticket;
  fa.vd = Verdict{w.prefix + w.W, needed_cap, validate ? err : nullptr};
  fa.emit_blocks = (int32_t)grid_for(w.W * 16);
  const unsigned remap_blocks = fa.compact && nnz > 0 ? grid_for(nnz, 8) : 0u;
  hipLaunchKernelGGL(finish_kernel, dim3((unsigned)fa.emit_blocks + remap_blocks), dim3(kThreads), 0, s, fa, cb);
  SAGNN_LAUNCH_CHECK();
  if (bucket_mark && d_colidx_compact && nnz > 0) {
    // ranks inside the buckets (in place), then every entry fetches the rank at its place
    hipLaunchKernelGGL(remap_bucket_kernel, dim3((unsigned)bucket_ranges(n)), dim3(kLdsThreads), 0, s, w.bkt_cols,
                       w.bkt_start, nnz, n, w.W, w.rank16, fa.vd);
    SAGNN_LAUNCH_CHECK();
    hipLaunchKernelGGL(remap_gather_kernel, dim3(kBktGroups), dim3(kBktThreads), 0, s, w.bkt_place, w.bkt_cols, nnz,
                       d_colidx_compact, fa.vd);
    SAGNN_LAUNCH_CHECK();
  }
  return SAGNN_OK;
}

int plan_run(const int32_t* d_rowptr, const int32_t* d_colidx, int64_t m, int64_t n, int64_t nnz,
             const int64_t* h_colblk, int32_t nb, int32_t* d_needed, int64_t needed_cap,
             int64_t* h_blk_off, int32_t* d_colidx_compact, const PlanWs& w, uint32_t flags, bool may_pin,
             hipStream_t s) {
  PlanRecord* rec = may_pin && nb <= kRecordMaxBlocks ? record_take() : nullptr;
  const int64_t ticket = g_ticket.fetch_add(1);
  int32_t bad = 0;
  int rc;
  if (rec) {
    rc = plan_launch(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, d_colidx_compact, w, flags, rec,
                     ticket, s);
    if (rc == SAGNN_OK) rc = record_wait(rec, ticket, s);
    else (void)hipStreamSynchronize(s);   // (whatever was launched may still write into the record)
    if (rc == SAGNN_OK) {
      for (int32_t q = 0; q <= nb; ++q) h_blk_off[q] = rec->blkoff[q];
      bad = rec->err[0] | rec->err[1];
    }
    record_give_back(rec);
  } else {
    rc = plan_launch(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, d_colidx_compact, w, flags,
                     nullptr, ticket, s);
    if (rc == SAGNN_OK) {
      const PlanRecord* d_rec = reinterpret_cast<const PlanRecord*>(w.blkoff);
      int32_t h_err[4] = {0, 0, 0, 0};
      SAGNN_HIP(hipMemcpyAsync(h_blk_off, d_rec->blkoff, sizeof(int64_t) * (size_t)(nb + 1), hipMemcpyDeviceToHost, s));
      SAGNN_HIP(hipMemcpyAsync(h_err, d_rec->err, sizeof(h_err), hipMemcpyDeviceToHost, s));
      SAGNN_HIP(hipStreamSynchronize(s));
      bad = h_err[0] | h_err[1];
    }
  }
  if (rc != SAGNN_OK) return rc;
  if ((flags & SAGNN_PLAN_VALIDATE) && bad) return SAGNN_EFORMAT;
  if (h_blk_off[nb] > needed_cap) return SAGNN_ECAPACITY;
  return SAGNN_OK;
}

}  // namespace
}  // namespace sagnn

SAGNN_EXPORT int spmm_plan_needed_rows(const int32_t* d_rowptr, const int32_t* d_colidx,
                                       int64_t m, int64_t n, int64_t nnz,
                                       const int64_t* h_colblk, int32_t nb, int32_t* d_needed,
                                       int64_t needed_cap, int64_t* h_blk_off,
                                       int32_t* d_colidx_compact, void* d_ws, size_t ws_bytes,
                                       uint32_t flags, void* stream) {
  using namespace sagnn;
  int rc = plan_check_args(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, h_blk_off);
  if (rc != SAGNN_OK) return rc;
  if (!d_ws || (reinterpret_cast<uintptr_t>(d_ws) & 255u)) return SAGNN_EINVAL;
  const PlanWs w = carve(d_ws, n, nb, nnz);
  if (ws_bytes < w.bytes) return SAGNN_ECAPACITY;
  return plan_run(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, h_blk_off,
                  d_colidx_compact, w, flags, true, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// Planning without a caller workspace and without any allocation: the scratch arrays (column
// flags, membership words, rank records, block sums, block boundaries, error counters) live
// in a fixed array in device memory that every GPU the library runs on holds for the life of
// the process.  The host only ever sees the array through the address hipGetSymbolAddress
// returns for the current device (the symbol's name is not a device address in host code).
namespace sagnn {
namespace {

constexpr size_t kPlanStaticBytes = 8u << 20;   // 8 MiB per GPU
constexpr int kPlanStaticMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kPlanStaticBytes];

std::mutex g_scratch_mutex;
void* g_scratch_ptr[kPlanStaticMaxDevices] = {};

// address of `scratch` on the current device, resolved once per device
int plan_static_scratch(void** out) {
  int dev = -1;
  SAGNN_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kPlanStaticMaxDevices) return SAGNN_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SAGNN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return SAGNN_EINVAL;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return SAGNN_OK;
}

}  // namespace
}  // namespace sagnn

SAGNN_EXPORT int spmm_plan_needed_rows_noalloc(const int32_t* d_rowptr, const int32_t* d_colidx,
                                               int64_t m, int64_t n, int64_t nnz,
                                               const int64_t* h_colblk, int32_t nb,
                                               int32_t* d_needed, int64_t needed_cap,
                                               int64_t* h_blk_off, int32_t* d_colidx_compact,
                                               uint32_t flags, void* stream) {
  using namespace sagnn;
  int rc = plan_check_args(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, h_blk_off);
  if (rc != SAGNN_OK) return rc;
  if (n > SAGNN_PLAN_NOALLOC_MAX_COLS || nb > SAGNN_PLAN_NOALLOC_MAX_BLOCKS) return SAGNN_ECAPACITY;
  // nnz = 0 in the layout: no private LDS bitmaps, the byte-flag marking path is used
  if (carve(nullptr, n, nb, 0).bytes > kPlanStaticBytes) return SAGNN_ECAPACITY;
  void* base = nullptr;
  rc = plan_static_scratch(&base);
  if (rc != SAGNN_OK) return rc;
  const PlanWs w = carve(base, n, nb, 0);
  return plan_run(d_rowptr, d_colidx, m, n, nnz, h_colblk, nb, d_needed, needed_cap, h_blk_off,
                  d_colidx_compact, w, flags, false, (hipStream_t)stream);
}
