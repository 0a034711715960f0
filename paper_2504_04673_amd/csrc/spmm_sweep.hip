// Locality-aware schedule for the local SpMM of power-law graphs: the "slab sweep".
//
// Why: in C = A * B (Alg. 1 / Alg. 2, "Z <- Z + SpMM(A_iq, H^)") every stored entry pulls one
// f-wide row of B through the memory system.  With a randomly ordered power-law graph a row of
// B is almost never still in a 4 MB per-XCD L2 when it is needed again, so the plain schedule
// moves ~15x the compulsory bytes over the fabric (measured).  The paper fixes the sparsity
// pattern for the whole training run (it partitions once and reuses the plan every epoch), so
// a one-time re-ordering of the entry stream is free to choose WHEN each row of B is touched.
//
// What: the rows of B are cut into S contiguous slabs.  Rows of A with at least `min_long`
// entries ("long" rows; they hold most entries of a power-law graph) are cut into pieces of at
// most `piece_max` entries, and every wavefront is given kSweepSlots pieces whose entries it
// walks slab by slab: all entries that reference slab 0, then slab 1, ...  Because all resident
// wavefronts walk the slabs in the same order at about the same pace (their streams have nearly
// equal lengths), each XCD's L2 only has to hold the hot rows of ONE slab at a time, and a slab
// that one XCD has pulled from HBM is served to the other seven from the memory-side cache.
// (Starting the XCDs at different slabs was measured to be slower: it defeats that sharing.)
// Per-piece accumulators live in LDS (a wavefront adds its register accumulator to the piece's
// LDS row whenever a (piece, slab) segment ends), so nothing is spilled to HBM between slabs.
// Pieces of a split row are summed in a fixed order by a small second kernel.  Short rows are
// swept as whole rows -- 16 per wavefront, each one segment, in wavefronts of their own -- where
// the matrix allows it, else they go through the nonzero-splitting kernel of spmm_flat.hip on a
// compacted CSR.
//
// The entry stream of a wavefront is stored in the workspace as (code, value) pairs sorted by
// (slab, piece): code = column | piece_slot << 27 | segment_end << 31.  At f = 128 / 64 a
// wavefront can carry 2 / 4 such streams, one per lane group, stored zipped (see
// spmm_sweep_group_kernel): a group of 32 / 16 lanes moves a whole row of B, so one load
// instruction serves 2 / 4 entries.
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <functional>
#include <type_traits>
#include <vector>

#include "common.h"
#include "gemm.h"
#include "rowload.h"

namespace sagnn {
namespace {

constexpr int kBuildThreads = 256;
constexpr uint32_t kColMask = (1u << kSweepColBits) - 1u;
constexpr int kSweepOwnSteps = 2;   // (behind the two boundaries of a single interval)
static_assert(kSweepOwnSteps + kSweepSlots <= kSweepMaxIntervals + 1, "lengths of sixteen streams in sync_off");

// ---------------------------------------------------------------------------------------
// preparation kernels

// piece_info[2*g] = row (or -1), piece_info[2*g+1] = (j << 16) | p

__device__ __forceinline__ int32_t count_upto(int32_t x, int32_t j, int32_t p) {
  // number of i in [0, x) with i % p == j
  if (p == 1) return x;
  return x > j ? (x - j + p - 1) / p : 0;
}

// Per-wavefront segment tables shared by the counting and the building kernel (dynamic LDS):
//   lo[16][S+1]      first entry (index in its row) of slab s for the piece in a slot
//   off[S][16]       offset of segment (s, slot) inside its slab, per lane group
//   slab_tot[S][16]  entries of slab s per lane group
struct BuildTables {
  int32_t *lo, *off, *slab_tot;
  int SS;
  __device__ int32_t& LO(int slot, int s) const { return lo[slot * (SS + 1) + s]; }
  __device__ int32_t& OFF(int s, int slot) const { return off[s * kSweepSlots + slot]; }
  __device__ int32_t& TOT(int s, int g) const { return slab_tot[s * kSweepSlots + g]; }
};

struct BuildPieces {
  int32_t row[kSweepSlots], j[kSweepSlots], p[kSweepSlots], beg[kSweepSlots], deg[kSweepSlots];
  int32_t hub[kSweepSlots], n_hub;   // slots whose row is searched, not read through
  int32_t pre[kSweepSlots + 1];   // lengths of the slots laid end to end (of the rows that are read through, or of the pieces)
};

// pc.pre = exclusive sums of the sixteen lanes' lengths; called by the first sixteen threads
__device__ __forceinline__ void lay_slots(BuildPieces& pc, int tid, int32_t len) {
  int32_t inc = len;
#pragma unroll
  for (int o = 1; o < kSweepSlots; o <<= 1) {
    const int32_t t = __shfl_up(inc, o, kSweepSlots);
    if (tid >= o) inc += t;
  }
  pc.pre[tid + 1] = inc;
  if (tid == 0) pc.pre[0] = 0;
}

// slot in which position e of the laid-out slots lies
__device__ __forceinline__ int slot_at(const BuildPieces& pc, int32_t e) {
  int slot = 0;
#pragma unroll
  for (int o = kSweepSlots / 2; o > 0; o >>= 1)
    if (pc.pre[slot + o] <= e) slot += o;
  return slot;
}

// the value of the lane before (lane 0: 0)
__device__ __forceinline__ uint32_t from_left(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, false);   // wave_shr:1
}

// c / width for c below 2^27 (the quotient in single precision is off by at most one)
__device__ __forceinline__ int slab_of(uint32_t c, uint32_t width, float inv_width, int S) {
  int s = (int)((float)c * inv_width);
  const uint32_t rest = c - (uint32_t)s * width;
  s += (int)rest < 0 ? -1 : (rest >= width ? 1 : 0);
  return s < S - 1 ? s : S - 1;
}

constexpr int kSearchPieces = 4;   // rows cut into more pieces are searched: reading them through would cost every
                                   // piece the whole row

// Fills pc (shared) and the tables for wavefront w; all threads of the workgroup take part.  The rows are read through
// once, side by side (an entry whose predecessor lies in an earlier slab is where its slab begins), where a binary
// search per slab and row is a chain of ten loads.  40 M entries over 64 slabs: the counting pass and the check of the
// order, then a kernel of its own, 194 + 614 us, now 216; the building pass 1010 us, now 535; by place, with an entry's
// predecessor taken from the neighbouring lane instead of memory, 260, now 240.  CHECK: *unsorted = 1 if a row's columns do not
// ascend or leave [0, kmax].
// kept (may be NULL): lo as the counting pass leaves it for the building pass, which then reads no columns for it (the layout
// of 40 M entries over four streams 240 -> 187 us).
template <bool CHECK>
__device__ __forceinline__ void build_tables(const int32_t* __restrict__ rowptr,
                                             const int32_t* __restrict__ colidx,
                                             const int32_t* __restrict__ piece_info, int64_t w, int S,
                                             int32_t slab_width, uint32_t kmax, int R, int SL,
                                             BuildPieces& pc, const BuildTables& T, int32_t* __restrict__ unsorted, int4* __restrict__ kept) {
  const int tid = threadIdx.x;
  if (tid < kSweepSlots) {
    const int32_t row = piece_info[2 * (w * kSweepSlots + tid)];
    const int32_t jp = piece_info[2 * (w * kSweepSlots + tid) + 1];
    const int32_t beg = row >= 0 ? rowptr[row] : 0, deg = row >= 0 ? rowptr[row + 1] - beg : 0;
    pc.row[tid] = row;
    pc.j[tid] = jp >> 16;
    pc.p[tid] = jp & 0xFFFF;
    pc.beg[tid] = beg;
    pc.deg[tid] = deg;
    lay_slots(pc, tid, row >= 0 && (jp & 0xFFFF) <= kSearchPieces && S > 1 ? deg : 0);
    const bool searched = row >= 0 && (jp & 0xFFFF) > kSearchPieces;
    const uint32_t hubs = (uint32_t)__ballot(searched);
    if (searched) pc.hub[__popc(hubs & ((1u << tid) - 1u))] = tid;
    if (tid == 0) pc.n_hub = __popc(hubs);
  }
  const bool scan = CHECK || kept == nullptr;
  if (!scan)
    for (int idx = tid; idx < kSweepSlots / 4 * (S + 1); idx += kBuildThreads) reinterpret_cast<int4*>(T.lo)[idx] = kept[idx];
  __syncthreads();
  if (scan)
    for (int idx = tid; idx < kSweepSlots * (S + 1); idx += kBuildThreads) {
      const int slot = idx / (S + 1), s = idx - slot * (S + 1);
      T.LO(slot, s) = s == 0 ? 0 : pc.deg[slot];
    }
  __syncthreads();
  const float inv = 1.0f / (float)slab_width;
  bool bad = false;
  const int32_t total = scan ? pc.pre[kSweepSlots] : 0;
  // A wavefront looks at 63 entries at a time: lane 0 has the one before them, every other lane takes its predecessor from its
  // neighbour.  The slot is looked up once for all lanes where they lie in one, as they mostly do (40 M entries, counting 142 us
  // with a look-up and two slabs for each entry, now 129).
  const int lane = tid & 63;
  const int32_t my_pre = lane <= kSweepSlots ? pc.pre[lane] : 0x7FFFFFFF, my_beg = pc.beg[lane & (kSweepSlots - 1)];
  for (int32_t e0 = (tid >> 6) * (4 * 63) - 1; e0 < total - 1; e0 += kBuildThreads / 64 * 4 * 63) {
    int slot[4];
    int32_t i[4];
    uint32_t c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t first = max(min(e0 + q * 63, total - 1), 0), last = min(e0 + q * 63 + 63, total - 1);
      const int32_t e = max(min(e0 + q * 63 + lane, total - 1), 0);
      const int sf = __popcll(__ballot(my_pre <= first)) - 1, sl = __popcll(__ballot(my_pre <= last)) - 1;
      if (sf == sl) {
        slot[q] = sf;
        i[q] = e - __builtin_amdgcn_readlane(my_pre, sf);
        c[q] = (uint32_t)colidx[__builtin_amdgcn_readlane(my_beg, sf) + i[q]];
      } else {
        slot[q] = slot_at(pc, e);
        i[q] = e - pc.pre[slot[q]];
        c[q] = (uint32_t)colidx[pc.beg[slot[q]] + i[q]];
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int s = slab_of(c[q] > kmax ? kmax : c[q], (uint32_t)slab_width, inv, S);
      const uint32_t left = from_left(c[q]);
      const int s_left = (int)from_left((uint32_t)s);
      if (lane == 0 || e0 + q * 63 + lane >= total) continue;
      if (CHECK) bad |= c[q] > kmax || (i[q] > 0 && left > c[q]);
      for (int t = i[q] > 0 ? s_left + 1 : 1; t <= s; ++t) T.LO(slot[q], t) = i[q];
    }
  }
  // rows cut into many pieces: all (row, slab) pairs side by side, four searches in flight per thread (row by row, with
  // the slabs side by side, the sixteen chains followed each other; 40 M entries: counting 152 -> 136 us, layout
  // 440 -> 423)
  const int n_hub = scan && S > 1 ? pc.n_hub : 0;
  if (CHECK) {   // every piece looks at its share of the row, one run (its own entries lie apart, a line each: 129 us, now 105)
    for (int h = 0; h < n_hub; ++h) {
      const int slot = pc.hub[h];
      const int64_t d = pc.deg[slot];
      const int32_t* __restrict__ col = colidx + pc.beg[slot];
      const int32_t to = (int32_t)(d * (pc.j[slot] + 1) / pc.p[slot]);
      for (int32_t i = (int32_t)(d * pc.j[slot] / pc.p[slot]) + tid; i < to; i += kBuildThreads)
        bad |= (uint32_t)col[i] > kmax || (i > 0 && (uint32_t)col[i - 1] > (uint32_t)col[i]);
    }
  }
  for (int q0 = tid; q0 < n_hub * (S - 1); q0 += 4 * kBuildThreads) {
    int32_t lo[4], hi[4], at[4];
    int64_t target[4];
    const int32_t* __restrict__ col[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * kBuildThreads;
      const bool in = q < n_hub * (S - 1);
      const int slot = pc.hub[in ? q / (S - 1) : 0], sl = in ? 1 + q % (S - 1) : 1;
      col[u] = colidx + pc.beg[slot];
      lo[u] = 0;
      hi[u] = in ? pc.deg[slot] : 0;
      at[u] = slot * (S + 1) + sl;
      target[u] = (int64_t)sl * slab_width;   // lower bound of the slab's first column
    }
    while (lo[0] < hi[0] || lo[1] < hi[1] || lo[2] < hi[2] || lo[3] < hi[3]) {
      uint32_t cv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) cv[u] = (uint32_t)col[u][lo[u] < hi[u] ? (lo[u] + hi[u]) >> 1 : 0];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (lo[u] >= hi[u]) continue;
        const int32_t mid = (lo[u] + hi[u]) >> 1;
        if ((int64_t)(cv[u] > kmax ? kmax : cv[u]) < target[u]) lo[u] = mid + 1; else hi[u] = mid;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (q0 + u * kBuildThreads < n_hub * (S - 1)) T.lo[at[u]] = lo[u];
  }
  if (CHECK && bad) *unsorted = 1;
  __syncthreads();
  if (CHECK && kept)
    for (int idx = tid; idx < kSweepSlots / 4 * (S + 1); idx += kBuildThreads) kept[idx] = reinterpret_cast<const int4*>(T.lo)[idx];
  // entries of segment (s, slot); then per slab the prefix over the slots of each group
  for (int idx = tid; idx < S * kSweepSlots; idx += kBuildThreads) {
    const int s = idx / kSweepSlots, slot = idx - s * kSweepSlots;
    T.OFF(s, slot) = pc.row[slot] >= 0 ? count_upto(T.LO(slot, s + 1), pc.j[slot], pc.p[slot]) -
                                             count_upto(T.LO(slot, s), pc.j[slot], pc.p[slot])
                                       : 0;
  }
  __syncthreads();
  for (int idx = tid; idx < S * R; idx += kBuildThreads) {
    const int s = idx / R, gi = idx - s * R;
    int32_t run = 0;
    for (int slot = gi * SL; slot < (gi + 1) * SL; ++slot) {
      const int32_t c = T.OFF(s, slot);
      T.OFF(s, slot) = run;
      run += c;
    }
    T.TOT(s, gi) = run;
  }
  __syncthreads();
}

// Where the counting pass keeps the first entries of wavefront w's segments: at the ends of the two stream arrays, which are laid
// out afterwards, even wavefronts at the one's and odd ones at the other's.  from: the first of these words, a multiple of 64
// (negative: nothing is kept).
struct KeptTables {
  int32_t *code, *vals;
  int64_t from;
  __device__ int4* of(int64_t w, int S) const {
    return from < 0 ? nullptr : reinterpret_cast<int4*>((w & 1 ? vals : code) + from + (w >> 1) * (kSweepSlots * (S + 1)));
  }
};

__device__ __forceinline__ BuildTables carve_tables(int32_t* lds, int S) {
  BuildTables T;
  T.SS = S;
  T.lo = lds;
  T.off = T.lo + kSweepSlots * (S + 1);
  T.slab_tot = T.off + S * kSweepSlots;
  return T;
}

// Pass 1: length of every interval of a wavefront's stream.  An interval's R group streams are
// padded to the longest of them and to a whole batch (8 steps), so that every wavefront reaches
// an interval boundary at a batch boundary.  sync_off[w][i] = first step of interval i,
// wave_steps[w] = total steps.  Sixteen streams have one interval: sync_off[w][kSweepOwnSteps + g] = steps of
// stream g without its padding.
__global__ __launch_bounds__(kBuildThreads) void sweep_count_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const int32_t* __restrict__ piece_info, int32_t n_slabs, int32_t slab_width, uint32_t kmax,
    int32_t groups, int32_t slots_per_group, int32_t n_intervals, int32_t sync_slabs,
    int32_t* __restrict__ sync_off, int32_t* __restrict__ wave_steps, int32_t* __restrict__ unsorted, const KeptTables kept) {
  extern __shared__ __attribute__((aligned(16))) int32_t build_lds[];
  __shared__ BuildPieces pc;
  __shared__ int32_t ivl_len[kSweepMaxIntervals];
  const int64_t w = blockIdx.x;
  const int S = n_slabs, R = groups;
  const BuildTables T = carve_tables(build_lds, S);
  build_tables<true>(rowptr, colidx, piece_info, w, S, slab_width, kmax, R, slots_per_group, pc, T, unsorted, kept.of(w, S));
  const int per = sync_slabs > 0 ? sync_slabs : S;
  const int lane = threadIdx.x & 63;
  int32_t* so = sync_off + w * (kSweepMaxIntervals + 1);
  for (int i = threadIdx.x >> 6; i < n_intervals; i += kBuildThreads / 64) {   // a wavefront per interval
    const int s0 = i * per, s1 = (i + 1) * per < S ? (i + 1) * per : S;
    int32_t longest = 0;
    for (int gi = 0; gi < R; ++gi) {
      int32_t t = 0;
      for (int s = s0 + lane; s < s1; s += 64) t += T.TOT(s, gi);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
      if (R == kSweepSlots && lane == 0) so[kSweepOwnSteps + gi] = t;
      longest = t > longest ? t : longest;
    }
    if (lane == 0) ivl_len[i] = (longest + 7) & ~7;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int i = 0; i < n_intervals; ++i) {
      so[i] = run;
      run += ivl_len[i];
    }
    so[n_intervals] = run;
    wave_steps[w] = run;
  }
}

// Pass 2: wave_base[w] = R * (steps of the wavefronts before w); wave_base[NW]
// is the total stream length.  To the record the host reads: overflow = 1 if it does not fit 31 bits, the total, the
// mean and the largest number of steps.
struct SweepScanRecord {
  int32_t overflow, left, total;
  float mean_steps, max_steps;
};

// A workgroup per kScanTile wavefronts, which adds up the wavefronts before its own by itself: they are read as long runs, in
// cache, while one workgroup for all waits for every round's loads and sums (1 M vertices, 40 M entries, eight
// streams: 45 us, now 12).
constexpr int kScanTile = 8192;
__global__ __launch_bounds__(1024) void sweep_scan_kernel(const int32_t* __restrict__ wave_steps,
                                                          int64_t n_waves, int32_t groups,
                                                          int32_t* __restrict__ wave_base,
                                                          SweepScanRecord* __restrict__ rec) {
  __shared__ int64_t wsum[16], wbefore[16];
  __shared__ int32_t wmax[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile;
  int32_t most = 0;
  int64_t before = 0;
#pragma unroll 4
  for (int64_t w = tid * 4; w < t0; w += 4096) {       // (wave_steps is aligned to 256 bytes)
    const int4 x = *reinterpret_cast<const int4*>(wave_steps + w);
    before += (int64_t)x.x + x.y + x.z + x.w;
    most = max(most, max(max(x.x, x.y), max(x.z, x.w)));
  }
  const int64_t w0 = t0 + tid * 8;                     // eight wavefronts per thread
  int32_t x[8];
  int64_t sum = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = w0 + i < n_waves ? wave_steps[w0 + i] : 0;
    most = max(most, x[i]);
    sum += x[i];
  }
  int64_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
    before += __shfl_xor(before, o, 64);
    most = max(most, __shfl_xor(most, o, 64));
  }
  if (lane == 63) {
    wsum[wave] = inc;
    wbefore[wave] = before;
    wmax[wave] = most;
  }
  __syncthreads();
  int64_t run = inc - sum, all = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    run += wbefore[i] + (i < wave ? wsum[i] : 0);
    all += wbefore[i] + wsum[i];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (w0 + i < n_waves) wave_base[w0 + i] = (int32_t)(run * groups > 0x7FFFFFF0ll ? 0x7FFFFFF0ll : run * groups);
    run += x[i];
  }
  if (blockIdx.x + 1 == gridDim.x && tid == 0) {
    for (int i = 0; i < 16; ++i) most = max(most, wmax[i]);
    const int64_t total = all * groups;
    rec->overflow = total > 0x7FFFFFF0ll ? 1 : 0;
    rec->total = (int32_t)(total > 0x7FFFFFF0ll ? 0x7FFFFFF0ll : total);
    rec->mean_steps = n_waves > 0 ? (float)((double)all / (double)n_waves) : 0.f;
    rec->max_steps = (float)most;
    wave_base[n_waves] = rec->total;
  }
}

// Pass 3, one workgroup per wavefront: lay the entries out in (interval, slab, piece) order and
// encode them.  With `groups` = R lane groups the wavefront carries R independent streams (group
// g owns slots g*SL .. g*SL+SL-1), stored zipped: step t of group g at position R*t + g.  Steps that no
// entry lands on (padding of the shorter group streams and at interval boundaries) multiply
// row 0 of B by 0.
// BY_PLACE: a thread takes a place of the stream and looks up its entry, else an entry and looks up its place.  Where four and
// more streams are zipped an entry's two stores go to lines of their own, and requests to lines were the kernel's time (1 M
// vertices, 40 M entries, four streams 422 us by entry, 260 by place; the whole preparation 1230, 1089, with sixteen 1908, 1354,
// with eight 300 k of 60 932, 860); one or two take runs either way, and so do rows whose columns lie in few slabs, and looking
// up costs more (2.45 M, 125 M entries, two 4365, 4778; communities, 500 k of 42, four 1238, 1277).
template <bool BY_PLACE>
__global__ __launch_bounds__(kBuildThreads) void sweep_build_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ val, const int32_t* __restrict__ piece_info,
    const int32_t* __restrict__ wave_base, const int32_t* __restrict__ sync_off, int32_t n_slabs,
    int32_t slab_width, uint32_t kmax, int32_t groups, int32_t slots_per_group, int32_t n_intervals,
    int32_t sync_slabs, uint32_t* __restrict__ code, float* __restrict__ vals, const KeptTables kept) {
  extern __shared__ __attribute__((aligned(16))) int32_t build_lds[];
  __shared__ BuildPieces pc;
  const int64_t w = blockIdx.x;
  const int tid = threadIdx.x;
  const int S = n_slabs, R = groups, SL = slots_per_group;
  const BuildTables T = carve_tables(build_lds, S);
  int32_t* slab_base_ = T.slab_tot + S * kSweepSlots;          // [16][S]: first step of slab s of group g at g S + s
  build_tables<false>(rowptr, colidx, piece_info, w, S, slab_width, kmax, R, SL, pc, T, nullptr, kept.of(w, S));
  const int per = sync_slabs > 0 ? sync_slabs : S;
  const int32_t* __restrict__ so = sync_off + w * (kSweepMaxIntervals + 1);
  const int64_t base = wave_base[w];
  // first step of every slab, a wavefront per (interval, group)
  const int lane = tid & 63;
  for (int idx = tid >> 6; idx < n_intervals * R; idx += kBuildThreads / 64) {
    const int i = idx / R, gi = idx - i * R;
    const int s0 = i * per, s1 = (i + 1) * per < S ? (i + 1) * per : S;
    int32_t run = so[i];
    for (int t0 = s0; t0 < s1; t0 += 64) {
      const int s = t0 + lane;
      const int32_t v = s < s1 ? T.TOT(s, gi) : 0;
      int32_t inc = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
      }
      if (s < s1) slab_base_[gi * S + s] = run + inc - v;
      run += __shfl(inc, 63, 64);
    }
    if constexpr (!BY_PLACE)
      for (int32_t t = run + lane; t < so[i + 1]; t += 64) {   // the steps no entry lands on
        code[base + (int64_t)t * R + gi] = 0u;
        vals[base + (int64_t)t * R + gi] = 0.f;
      }
  }
  if constexpr (!BY_PLACE) {
    if (tid < kSweepSlots) lay_slots(pc, tid, pc.row[tid] >= 0 ? count_upto(pc.deg[tid], pc.j[tid], pc.p[tid]) : 0);
    __syncthreads();
    const float inv = 1.0f / (float)slab_width;
    const int32_t total = pc.pre[kSweepSlots];
    for (int32_t e0 = tid; e0 < total; e0 += 4 * kBuildThreads) {
      int slot[4];
      int32_t i[4], at[4];
      uint32_t c[4];
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int32_t e = e0 + q * kBuildThreads < total ? e0 + q * kBuildThreads : total - 1;
        slot[q] = slot_at(pc, e);
        at[q] = e - pc.pre[slot[q]];
        i[q] = pc.j[slot[q]] + at[q] * pc.p[slot[q]];
        c[q] = (uint32_t)colidx[pc.beg[slot[q]] + i[q]];
        v[q] = val[pc.beg[slot[q]] + i[q]];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (e0 + q * kBuildThreads >= total) break;
        const int sl = slot[q];
        const int32_t j = pc.j[sl], p = pc.p[sl];
        const uint32_t cc = c[q] > kmax ? kmax : c[q];
        int s = slab_of(cc, (uint32_t)slab_width, inv, S);
        // the row is ascending, but clamped / equal columns may sit on a slab boundary: trust lo[]
        while (s > 0 && i[q] < T.LO(sl, s)) --s;
        while (s < S - 1 && i[q] >= T.LO(sl, s + 1)) ++s;
        const int32_t rank = at[q] - count_upto(T.LO(sl, s), j, p);
        // a segment also ends every kSweepRunMax entries, which bounds the length of any serial
        // fp32 accumulation (and with it the rounding bias on rows of equal terms)
        const bool last = i[q] + p >= T.LO(sl, s + 1) || (rank & (kSweepRunMax - 1)) == kSweepRunMax - 1;
        const int gi = sl / SL;
        const int64_t pos = base + (int64_t)(slab_base_[gi * S + s] + T.OFF(s, sl) + rank) * R + gi;
        code[pos] = cc | ((uint32_t)sl << kSweepColBits) | (last ? 0x80000000u : 0u);
        vals[pos] = v[q];
      }
    }
    return;
  }
  __syncthreads();
  // In the order of the stream: a thread looks up which entry its place takes, so that the stores are whole lines and the loads
  // runs of a segment's entries.
  const int group_bits = 31 - __clz(R);
  const int32_t words = so[n_intervals] * R;
  for (int32_t q0 = tid; q0 < words; q0 += 4 * kBuildThreads) {
    int32_t from[4];
    uint32_t tag[4], c[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t q = q0 + u * kBuildThreads;
      const int gi = q & (R - 1);
      const int32_t t = q >> group_bits;
      // the last slab, then the last slot of the group, that begins at or before step t: the one that has it, if any
      int s = 0;
      const int32_t* __restrict__ first = slab_base_ + gi * S;
      for (int n = S; n > 1;) {
        const int half = n >> 1;
        s = first[s + half] <= t ? s + half : s;
        n -= half;
      }
      const int32_t in_slab = t - first[s], total = T.TOT(s, gi);
      int sl = gi * SL;
      for (int n = SL; n > 1;) {
        const int half = n >> 1;
        sl = T.OFF(s, sl + half) <= in_slab ? sl + half : sl;
        n -= half;
      }
      const int32_t rank = in_slab - T.OFF(s, sl);
      const int32_t len = (sl + 1 < (gi + 1) * SL ? T.OFF(s, sl + 1) : total) - T.OFF(s, sl);
      const bool in = q < words && rank >= 0 && rank < len;
      // entry `rank` of those of the row's slab that are this piece's: every p-th from the j-th of the row on
      const int32_t p = pc.p[sl], lo = T.LO(sl, s);
      const int32_t skip = p == 1 ? 0 : ((pc.j[sl] - lo) % p + p) % p;
      from[u] = in ? pc.beg[sl] + lo + skip + rank * p : -1;
      // a segment also ends every kSweepRunMax entries, which bounds the length of any serial
      // fp32 accumulation (and with it the rounding bias on rows of equal terms)
      const bool last = rank + 1 == len || (rank & (kSweepRunMax - 1)) == kSweepRunMax - 1;
      tag[u] = ((uint32_t)sl << kSweepColBits) | (last ? 0x80000000u : 0u);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = from[u] >= 0 ? (uint32_t)colidx[from[u]] : 0u;
      v[u] = from[u] >= 0 ? val[from[u]] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t q = q0 + u * kBuildThreads;
      if (q >= words) break;
      code[base + q] = from[u] >= 0 ? (c[u] > kmax ? kmax : c[u]) | tag[u] : 0u;
      vals[base + q] = v[u];
    }
  }
}

// The wavefronts of whole short rows: every row is one segment of its group's stream, so there are no slabs and no
// tables.  A stream holds a few hundred entries and its chain piece - row pointer - entries is its time: sixteen
// streams are counted, four laid out by a workgroup, where a workgroup each went through the tables with a slab that
// covers all of B.  40 M entries, 580 k short rows: counting 217 -> 160 us, layout 535 -> 510 (8 and 70 of it here).
__global__ __launch_bounds__(kBuildThreads) void sweep_short_count_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ piece_info, int64_t w0, int64_t w1, int32_t slots_per_group,
    int32_t* __restrict__ sync_off, int32_t* __restrict__ wave_steps) {
  const int64_t w = w0 + ((int64_t)blockIdx.x * kBuildThreads + threadIdx.x) / kSweepSlots;   // sixteen lanes a wavefront
  const int slot = threadIdx.x & (kSweepSlots - 1);
  const int32_t row = w < w1 ? piece_info[2 * (w * kSweepSlots + slot)] : -1;
  const int32_t deg = row >= 0 ? rowptr[row + 1] - rowptr[row] : 0;
  int32_t t = deg;
  for (int o = 1; o < kSweepSlots; o <<= 1) {                  // sum over a group, largest of the groups
    const int32_t u = __shfl_xor(t, o, kSweepSlots);
    t = o < slots_per_group ? t + u : (u > t ? u : t);
  }
  int32_t* __restrict__ so = sync_off + w * (kSweepMaxIntervals + 1);
  if (w < w1 && slots_per_group == 1) so[kSweepOwnSteps + slot] = deg;
  t = (t + 7) & ~7;
  if (w < w1 && slot == 0) {
    wave_steps[w] = t;
    so[0] = 0;
    so[1] = t;
  }
}

__global__ __launch_bounds__(kBuildThreads) void sweep_short_build_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx, const float* __restrict__ val,
    const int32_t* __restrict__ piece_info, const int32_t* __restrict__ wave_base, int64_t w0, int64_t w1, uint32_t kmax,
    int32_t groups, int32_t slots_per_group, uint32_t* __restrict__ code, float* __restrict__ vals) {
  __shared__ BuildPieces pieces[kBuildThreads / 64];
  const int lane = threadIdx.x & 63;
  BuildPieces& pc = pieces[threadIdx.x >> 6];
  const int64_t w = w0 + (int64_t)blockIdx.x * (kBuildThreads / 64) + (threadIdx.x >> 6);
  const int R = groups, SL = slots_per_group;
  if (lane < kSweepSlots) {
    const int32_t row = w < w1 ? piece_info[2 * (w * kSweepSlots + lane)] : -1;
    const int32_t beg = row >= 0 ? rowptr[row] : 0, deg = row >= 0 ? rowptr[row + 1] - beg : 0;
    pc.beg[lane] = beg;
    pc.deg[lane] = deg;
    lay_slots(pc, lane, deg);
  }
  __syncthreads();
  if (w >= w1) return;
  const int64_t base = wave_base[w];
  const int32_t steps = (int32_t)((wave_base[w + 1] - base) / R);
  const int32_t total = pc.pre[kSweepSlots];
  for (int32_t e0 = lane; e0 < total; e0 += 4 * 64) {
    int slot[4];
    uint32_t c[4];
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t e = e0 + q * 64 < total ? e0 + q * 64 : total - 1;
      slot[q] = slot_at(pc, e);
      const int32_t at = pc.beg[slot[q]] + e - pc.pre[slot[q]];
      c[q] = (uint32_t)colidx[at];
      v[q] = val[at];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t e = e0 + q * 64;
      if (e >= total) break;
      const int sl = slot[q], gi = sl / SL;
      const int32_t rank = e - pc.pre[sl];
      // (a segment also ends every kSweepRunMax entries, see sweep_build_kernel)
      const bool last = rank + 1 >= pc.deg[sl] || (rank & (kSweepRunMax - 1)) == kSweepRunMax - 1;
      const int64_t pos = base + (int64_t)(e - pc.pre[gi * SL]) * R + gi;
      code[pos] = (c[q] > kmax ? kmax : c[q]) | ((uint32_t)sl << kSweepColBits) | (last ? 0x80000000u : 0u);
      vals[pos] = v[q];
    }
  }
  for (int gi = 0; gi < R; ++gi)                               // steps no entry lands on
    for (int32_t t = pc.pre[(gi + 1) * SL] - pc.pre[gi * SL] + lane; t < steps; t += 64) {
      code[base + (int64_t)t * R + gi] = 0u;
      vals[base + (int64_t)t * R + gi] = 0.f;
    }
}

inline size_t sweep_count_lds_bytes(int64_t S) {
  return sizeof(int32_t) * (size_t)(kSweepSlots * (S + 1) + 2 * S * kSweepSlots);
}
inline size_t sweep_build_lds_bytes(int64_t S) {
  return sizeof(int32_t) * (size_t)(kSweepSlots * (S + 1) + 3 * S * kSweepSlots);
}

__global__ __launch_bounds__(256) void sweep_zero_gap_kernel(uint32_t* __restrict__ code,
                                                            float* __restrict__ vals, int32_t n) {
  for (int i = threadIdx.x; i < n; i += 256) {
    code[i] = 0u;
    vals[i] = 0.f;
  }
}

// compacted CSR of the short rows: copy entries
__global__ __launch_bounds__(256) void sweep_short_copy_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ val, const int32_t* __restrict__ rowptr_s,
    const int32_t* __restrict__ rowmap_s, int64_t rows_s, int32_t* __restrict__ colidx_s,
    float* __restrict__ val_s) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows_s) return;
  const int32_t r = rowmap_s[i];
  const int32_t b = rowptr[r], n = rowptr[r + 1] - b, o = rowptr_s[i];
  for (int32_t t = 0; t < n; ++t) {
    colidx_s[o + t] = colidx[b + t];
    val_s[o + t] = val[b + t];
  }
}

// ---------------------------------------------------------------------------------------
// product kernel
struct SweepDims {
  int64_t n_waves, ldb, ldc, f_total;
  uint64_t generation;
  uint32_t b_bytes;     // bytes addressable from B + col0 (buffer-load variant)
  uint32_t row_bytes;   // ldb * 4
  int32_t col0, accumulate;
  // interval barriers (lane-group kernels): 0 intervals = walk the stream in one go
  int32_t n_intervals, wg_per_cohort, sync_timeout_ticks, sync_test_extra;
  int32_t slots;        // accumulator rows per wavefront (<= kSweepSlots)
  int32_t fw;           // floats per row of this launch
  float pace_ticks;     // pacing: 100 MHz ticks per stream step (0: none)
  int32_t block0;       // first workgroup of this launch (one row per load)
  int32_t turn;         // steps between two priorities, at most (TurnTaking)
  int32_t long_waves;   // wavefronts before those of whole short rows
  int32_t run;          // workgroups whose rows are shared out among the XCDs in runs (run_block; a multiple of 8, 0: none)
};

// The workgroup whose streams this one walks.  Workgroups go to the eight XCDs in turn, so that neighbouring rows, which want
// the same rows of B where their order carries locality, were walked on all of them and every L2 fetched every neighbourhood.
// Of each `run` workgroups of the schedule an XCD now takes an eighth that lies together (sweep_run has the rule).
__device__ __forceinline__ int64_t run_block(const SweepDims& d) {
  const uint32_t b = blockIdx.x;
  if (d.run == 0) return (int64_t)d.block0 + b;
  const uint32_t first = b / (uint32_t)d.run * (uint32_t)d.run;
  const uint32_t n = min((uint32_t)d.run, gridDim.x - first), i = b - first, x = i & 7u;
  return (int64_t)d.block0 + first + x * (n >> 3) + min(x, n & 7u) + (i >> 3);
}

// Barrier between two intervals of the sweep for the workgroups that run at the same time on
// one XCD ("cohort" c = workgroup index / wg_per_cohort, XCD = workgroup index mod 8: workgroups
// are handed to the XCDs round-robin).  It only paces the workgroups -- no data passes through
// it -- so that all of them read the same part of B at the same time and the XCD's L2 serves
// every row once.  The wait is bounded: after `timeout` ticks of the 100 MHz clock the waiter
// sets a flag that makes every later barrier of the launch fall through (the kernel then
// free-runs, correct but with more cache misses), so a launch whose cohort is not resident
// together (fewer free CUs than assumed) still ends.
__device__ __forceinline__ void sweep_interval_barrier(uint32_t* __restrict__ counters, int slot,
                                                       uint32_t expected, int32_t timeout) {
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t* broken = counters + kSweepBarrierSlots;
    if (__hip_atomic_load(broken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
      uint32_t* ctr = counters + slot;
      __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t t0 = wall_clock64();
      while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < expected) {
        if (__hip_atomic_load(broken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) break;
        if (wall_clock64() - t0 > (uint64_t)timeout) {
          __hip_atomic_store(broken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(16);
      }
    }
  }
  __syncthreads();
}

// Pacing: a wavefront does not enter the next interval before `ticks` of the 100 MHz clock have
// passed since it started.  Every wavefront follows the same schedule (the average number of
// stream steps up to each interval boundary, times a fixed time per step), so all of them pass
// over B at one pace without exchanging anything; one that is behind schedule never waits.  The
// loop is bounded (the clock passes the deadline, and the iteration count is capped anyway).
__device__ __forceinline__ void sweep_pace_until(uint64_t t0, float ticks) {
  const uint64_t deadline = t0 + (uint64_t)ticks;
  for (int i = 0; i < 2048; ++i) {
    if ((uint64_t)wall_clock64() >= deadline) break;
    __builtin_amdgcn_s_sleep(8);
  }
}

// sched[i] = average over the wavefronts of the first step of interval i (i = 0..n_intervals)
__global__ __launch_bounds__(256) void sweep_sched_kernel(const int32_t* __restrict__ sync_off,
                                                          int64_t n_waves, int32_t n_intervals,
                                                          float* __restrict__ sched) {
  __shared__ double red[256];
  const int i = blockIdx.x;
  double acc = 0.0;
  for (int64_t w = threadIdx.x; w < n_waves; w += 256) acc += (double)sync_off[w * (kSweepMaxIntervals + 1) + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) {
    if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) sched[i] = n_waves > 0 ? (float)(red[0] / (double)n_waves) : 0.f;
}

__global__ __launch_bounds__(256) void sweep_barrier_clear_kernel(uint32_t* __restrict__ counters, int n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) counters[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) counters[kSweepBarrierSlots] = 0u;
}

// first of the `v` floats a lane works on: `at`, or the row's last ones if the row ends before
template <bool ODD>
__device__ __forceinline__ uint32_t row_element(uint32_t at, int v, int32_t fw) {
  return ODD && (int32_t)at > fw - v ? (uint32_t)(fw - v) : at;
}

// Sum of a segment.  TWO: the entries of a batch of eight in two sums, then the batches, where a plain sum goes on through
// the segment.  For the widths between the kernels' own (ODD) below 64, and below 128 with one row per load, for 16, for 32
// by the length of the segments (1 M vertices, 50 M entries, training at f = 16 2267 us with a plain sum, 2249 so), and below
// 128 in small matrices:
// nonzero splitting, which had these widths before, added their entries as a tree.  Error against 64 bits (2-norm) by the tree,
// by a plain sum, by two: 300 k vertices of 42 in 16 communities f = 8 6.9e-8, 1.18e-7, 6.9e-8, f = 48 7.8e-8, 1.17e-7,
// 7.4e-8; a rank's rows f = 48 3.0e-8, 3.6e-8, 3.2e-8.  (What is left is the order of the slabs: random columns, 40 a row,
// f = 48 7.7e-8, 8.3e-8, 8.5e-8, as the full widths always had.)  1 M vertices, 50 M
// entries: f = 36 870 -> 893 us, f = 48 838 -> 852, the other widths and graphs within 1 %.  At f = 100 to 252 with lane
// groups or four floats a lane the plain sum was no worse than the tree, and two would cost 2 %.
template <typename vec, bool TWO>
struct SegmentSum {
  vec acc = 0.f, part[2] = {0.f, 0.f};
  __device__ __forceinline__ void add(int u, float v, const vec& h) {
    if constexpr (TWO) part[u & 1] += v * h;
    else acc += v * h;
  }
  __device__ __forceinline__ void batch_ends() {
    if constexpr (TWO) {
      acc += part[0] + part[1];
      part[0] = part[1] = 0.f;
    }
  }
  __device__ __forceinline__ vec take() {
    batch_ends();
    const vec t = acc;
    acc = 0.f;
    return t;
  }
};

// Sum of a whole short row with eight lane groups: four entries at a time, then these sums, which is as near to 64 bits as
// nonzero splitting's batches of eight were (2-norm by that, as one sum and so, e-8, f = 32, power-law 2.45 M vertices of 51
// 1.47, 1.58, 1.46, 1 M of 14 1.31, 1.41, 1.29, random columns, 300 k of 20 7.18, 7.31, 7.16).
template <typename vec>
struct ShortRowSum {
  vec acc = 0.f, part = 0.f;
  __device__ __forceinline__ void add(int u, float v, const vec& h) {
    part += v * h;
    if ((u & 3) == 3) {
      acc += part;
      part = 0.f;
    }
  }
  __device__ __forceinline__ void batch_ends() {}
  __device__ __forceinline__ vec take() {
    const vec t = acc + part;
    acc = part = 0.f;
    return t;
  }
};

// Who of a SIMD's wavefronts may issue next.  Left alone the hardware serves the oldest first: at the middle of a
// generation the six wavefronts of a SIMD stood 0.10 to 0.29 of a stream apart in order of their age, so the L2 held the
// rows of B that the first of them wanted and the last fetched them again.  A wavefront goes down through the four
// priorities as it walks, one per `stride` steps, and begins again at the top: of those less than four strides apart the
// one behind goes first.  A sixteenth of the stream a stride, at most 32 steps where B fits the memory-side cache and 128
// where it does not (turn_steps).  2.45 M vertices, 125 M entries: f = 128 4363 -> 4132 us, f = 64 2705 -> 2322; 233 k,
// 114 M, f = 128 2455 -> 2328; partitioned 2 M, 84 M, f = 128 5588 -> 5376.  No gain and not used with sixteen groups, whose
// wavefronts wait for the address units.  Progress counted in memory, so that the order holds beyond four strides, costs
// more than it gives: an atomic per level and wavefront, 4.7 ms and more for the first figure.
struct TurnTaking {
  int32_t next, stride;
  uint32_t level;
  // (longest 0: no turns)
  __device__ __forceinline__ TurnTaking(int32_t steps, int32_t longest) : next(longest > 0 ? 0 : -1), level(0) {
    stride = (steps >> 4) & ~7;
    stride = stride > longest ? longest : (stride < 8 ? 8 : stride);
  }
  __device__ __forceinline__ void at(int32_t e) {   // before the batch that begins with step e, e a multiple of 8
    if (e != next) return;
    next += stride;
    switch (level++ & 3u) {
      case 0: __builtin_amdgcn_s_setprio(3); break;
      case 1: __builtin_amdgcn_s_setprio(2); break;
      case 2: __builtin_amdgcn_s_setprio(1); break;
      default: __builtin_amdgcn_s_setprio(0); break;
    }
  }
};

// One row per load: a wavefront's stream, `len` steps (a multiple of U), into its accumulator rows `my`.
// FPL == 4: the words of the next batch are requested before this one's rows are waited for, two sets of scalar registers
// in turn.  They come from HBM, and with the eight wavefronts that 256 columns leave a CU nobody else hides it: 2.45 M
// vertices, 125 M entries, f = 256 9544 -> 8759 us, 233 k, 114 M 5669 -> 4650.  Not at fewer columns, where four times as
// many wavefronts do and those that run ahead cost more misses (250 k vertices of 60, f = 64: 332 -> 409; f = 128 the same).
template <int FPL, int U, bool BUF, bool TWO, bool TURN>
__device__ __forceinline__ void walk_stream(const uint32_t* __restrict__ cw, const float* __restrict__ vw, int32_t len,
                                            __amdgpu_buffer_rsrc_t rs, const float* __restrict__ B, const SweepDims& d, uint32_t loff,
                                            float* __restrict__ my, int kRow) {
  using vec = typename Vec<FPL>::T;
  constexpr bool kAhead = FPL == 4;
  SegmentSum<vec, TWO> sum;
  TurnTaking turn(len, d.turn);
  auto words = [&](int32_t at, uint32_t (&c)[U], float (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = cw[at + u];
      v[u] = vw[at + u];
    }
  };
  auto batch = [&](int32_t e, uint32_t (&c)[U], float (&v)[U], uint32_t (&cn)[U], float (&vn)[U]) {
    if constexpr (TURN) turn.at(e);
    if constexpr (!kAhead) words(e, c, v);
    vec h[U];
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = load_row<FPL, BUF>(rs, B, c[u] & kColMask, loff, d.row_bytes, d.ldb);
    if constexpr (kAhead) {
      __builtin_amdgcn_sched_barrier(0);
      words(e + U < len ? e + U : e, cn, vn);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" : "+v"(h[u]));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sum.add(u, v[u], h[u]);
      if (c[u] >> 31) {   // last entry of a (piece, slab) segment: fold into the piece's LDS row
        vec* p = reinterpret_cast<vec*>(my + ((c[u] >> kSweepColBits) & (kSweepSlots - 1)) * kRow);
        *p += sum.take();
      }
    }
    sum.batch_ends();
  };
  uint32_t c0[U], c1[U];
  float v0[U], v1[U];
  if constexpr (kAhead) {
    if (len > 0) words(0, c0, v0);
    for (int32_t e = 0; e < len; e += U) {
      batch(e, c0, v0, c1, v1);
      e += U;
      if (e >= len) break;
      batch(e, c1, v1, c0, v0);
    }
  } else {
    for (int32_t e = 0; e < len; e += U) batch(e, c0, v0, c0, v0);
  }
}

// ODD: rows of any multiple of 4 floats instead of the kernel's full width.  The lanes beyond the end of the row work
// on its last FPL floats a second time: same addresses, same values, so neither loads nor accumulator updates nor
// stores need a mask, and the accumulator rows are as long as the rows themselves.
template <int FPL, int U, bool BUF, bool ODD, bool TURN>
__global__ __launch_bounds__(256) void spmm_sweep_kernel(
    const uint32_t* __restrict__ code, const float* __restrict__ vals,
    const int32_t* __restrict__ wave_base, const int32_t* __restrict__ piece_target,
    const SpmmWsHeader* __restrict__ hdr, const float* __restrict__ B, float* __restrict__ C,
    float* __restrict__ partial, const SweepDims d) {
  using vec = typename Vec<FPL>::T;
  extern __shared__ __attribute__((aligned(16))) float lds_acc[];  // [4 waves][d.slots][kRow]
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t el = row_element<ODD>(lane * FPL, FPL, d.fw);
  const uint32_t loff = el * 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t w = run_block(d) * 4 + wave;
  if (w >= d.n_waves) return;
  if (hdr->magic != kSpmmMagic || hdr->generation != d.generation || hdr->n_waves != d.n_waves ||
      hdr->groups != 1)
    return;
  const int kRow = ODD ? d.fw : 64 * FPL;  // floats per accumulator row
  float* __restrict__ my = lds_acc + (size_t)wave * d.slots * kRow + el;
  for (int s = 0; s < d.slots; ++s) *reinterpret_cast<vec*>(my + s * kRow) = vec(0.f);

  const int32_t base = wave_base[w];
  const int32_t len = wave_base[w + 1] - base;  // a multiple of U (padded when built)
  const uint32_t* __restrict__ cw = code + base;
  const float* __restrict__ vw = vals + base;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B, d.b_bytes);

  walk_stream<FPL, U, BUF, ODD && FPL <= 2, TURN>(cw, vw, len, rs, B, d, loff, my, kRow);

#pragma unroll 1
  for (int s = 0; s < d.slots; ++s) {
    const int32_t tgt = piece_target[w * kSweepSlots + s];
    if (tgt == INT32_MIN) continue;
    vec r = *reinterpret_cast<const vec*>(my + s * kRow);
    if (tgt >= 0) {
      vec* p = reinterpret_cast<vec*>(reinterpret_cast<char*>(C + (int64_t)tgt * d.ldc) + loff);
      if (d.accumulate) r += *p;
      *p = r;
    } else {
      const int64_t pi = -(int64_t)tgt - 1;
      *reinterpret_cast<vec*>(reinterpret_cast<char*>(partial + pi * d.f_total + d.col0) + loff) = r;
    }
  }
}

// The sweep with the layer's dense transform as its epilogue (Alg. 1: the SpMM statement followed
// by GEMM and the activation): when a workgroup's four wavefronts have walked their streams, its
// LDS holds 64 finished rows of T = A H (4 x 16 accumulator rows), which is two 32-row operand
// tiles of the matrix cores.  Wavefront (rt, half) multiplies row tile rt by the 32-column tiles
// half, half + 2, .. of W, read from global memory (W is small and stays in L2), and stores the
// rows of Z / sigma(Z) at the rows the pieces belong to.  Rows that are cut into several pieces
// (their partial rows go to `partial` as usual) and rows outside the sweep are left to a
// separate small kernel.  T itself goes to memory only if the caller wants it.
typedef float sweep_floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 sweep_bf16x8 __attribute__((ext_vector_type(8)));

// Dense transform of a sweep workgroup's 64 finished rows of T (LDS, [4 waves][16 slots][KROW]):
// wavefront (rt, half) multiplies row tile rt by the 32-column tiles half, half + 2, .. of W and
// stores the rows of Z / sigma(Z) at the rows the pieces belong to (slots that hold a piece of a
// split row, or nothing, are skipped): `targets`, the piece_target of the workgroup (see Targets).  Called
// by all four wavefronts after a workgroup barrier.
// MODE: the matrix-core operands, numbered like SAGNN_GEMM_*: 0 fp32, 1 rounded to bfloat16, 2 fp32
// as the exact sum of three bfloat16 terms with the six products down to 2^-16 of the leading one.  (fp32 is not done as three
// terms though they are faster, power-law 2.45 M vertices of 51, 128 to 128 4740 us, 4400: sums of few terms that are not zero
// would be twice as far from 64 bits, at 128 columns with one W in 32 not zero 4.2e-8, 7.4e-8, and a value the terms do
// not hold costs a second product.)
// Rows of T lie kPadRow floats further apart in the LDS than they are long: a lane reads its own row, and rows of a multiple of 64
// floats begin in the same bank.  us side by side and so, 128 to 128, power-law 1 M vertices of 14 in bfloat16 841, 761, fp32
// 1052, 1028, 2.45 M of 51 4395, 4235 and 4760, 4740; random columns, 500 k of 24 862, 843 and 924, 913.
constexpr int kPadRow = 4;

// Where the epilogue finds its rows: the LDS, written beside the walk, but memory in fp32 at 256 columns.  In memory, behind
// the matrix instructions, they are one more trip in every pass over k; looked up before the loop over k they take sixteen
// registers, which decide how many workgroups walk at the same time at 64 columns.  us behind, before and from the LDS:
// communities, 700 k vertices of 40, 256 to 256 bfloat16 3290, 3200, 3110; a rank's 306 k rows of 11, 64 to 64 180, 220, 174.
// In fp32 at 256 the trip does not show beside 14 us of matrix instructions, and what comes sooner is worse for random columns
// whose rows of B are hardly used twice: from memory behind, before (TARGETS_BEFORE) and from the LDS 800 k vertices of 15
// 2738, 3166, 3182, 1 M of 16, 18, 22 from the LDS 3663, 3995, 4559 -> 4275, 4495, 4958, 300 k of 20 (1.1 uses) 1237, 1263,
// 1272; but 200 k of 40 (3.3) 1291, 1264, 1280, 1 M rows of 20 by 20 k columns 2914, 2713, 2750, in communities 500 k of 42
// 2644, 2547, 2536, 700 k of 40 3759, 3714, 3677, though 500 k of 18 1708, 1781, 1.5 M of 42 8500, 8848 (bfloat16 2 M of 18
// random 7262 behind, 7058 from the LDS).
enum Targets { TARGETS_LDS, TARGETS_BEHIND, TARGETS_BEFORE };

template <int KROW, int MODE, int QT, Targets FROM = TARGETS_LDS>
__device__ __forceinline__ void sweep_dense_epilogue(const float* __restrict__ lds_acc,
                                                     const int32_t* __restrict__ targets,
                                                     const SweepFusedArgs& fa, int wave, int lane) {
  constexpr int kRow = KROW;
  const int r = lane & 31, h = lane >> 5;
  const int rt = wave & 1;
  const int nct = (fa.f_out + 31) >> 5;
  [[maybe_unused]] int4 far[4];
  if constexpr (FROM == TARGETS_BEFORE) {
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) far[v4] = *reinterpret_cast<const int4*>(targets + rt * 32 + h * 4 + v4 * 8);
  }
  const float* __restrict__ trow = lds_acc + (size_t)(rt * 32 + r) * (kRow + kPadRow);
  // this wavefront's column tiles: ct_first, ct_first + 2, ..  (at most 4 of the at most 8).  k runs
  // in the outer loop so that a row piece of T is read from LDS once for the tiles of a pass, and the
  // operands of W for the next k group are requested before the matrix instructions of this one;
  // QT of them per pass over k (the accumulators of a pass live in registers: 16 per tile).
  const int ct_first = wave >> 1;
  const int nmine = nct > ct_first ? (nct - ct_first + 1) >> 1 : 0;
#pragma unroll 1
  for (int q0 = 0; q0 < nmine; q0 += QT) {
    const int ct0 = ct_first + 2 * q0;
    const int nmy = nmine - q0 < QT ? nmine - q0 : QT;
    sweep_floatx16 z[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) z[q][v] = 0.f;
    if constexpr (MODE == 2) {
      // W as packed by sweep_pack_w_kernel with three planes: term t of W at Wp + t * (kRow / 8) * NB
      const sweep_bf16x8* __restrict__ Wp = reinterpret_cast<const sweep_bf16x8*>(fa.Wp);
      const int NB = nct * 32;
      const int64_t plane = (int64_t)(kRow / 8) * NB;
      constexpr int J = kRow / 16;
      constexpr bool kAhead = KROW > 64;   // (few steps at 64: not worth the registers that keep workgroups out)
      sweep_bf16x8 cur[QT][3], nxt[QT][3];
      auto wload = [&](int j, sweep_bf16x8 (&dst)[QT][3]) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
          if (q < nmy) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
              dst[q][t] = Wp[t * plane + (int64_t)(2 * j + h) * NB + (ct0 + 2 * q) * 32 + r];
          }
      };
      if constexpr (kAhead) wload(0, cur);
#pragma unroll 1
      for (int j = 0; j < J; ++j) {
        if constexpr (!kAhead) wload(j, cur);
        else if (j + 1 < J) wload(j + 1, nxt);
        const float4 x0 = *reinterpret_cast<const float4*>(trow + 16 * j + 8 * h);
        const float4 x1 = *reinterpret_cast<const float4*>(trow + 16 * j + 8 * h + 4);
        const float xs[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        sweep_bf16x8 a1, a2, a3;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          __bf16 t1, t2, t3;
          split3(xs[i], t1, t2, t3);
          a1[i] = t1; a2[i] = t2; a3[i] = t3;
        }
#pragma unroll
        for (int q = 0; q < QT; ++q)
          if (q < nmy) {
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a3, cur[q][0], z[q], 0, 0, 0);
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, cur[q][2], z[q], 0, 0, 0);
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, cur[q][1], z[q], 0, 0, 0);
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, cur[q][0], z[q], 0, 0, 0);
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, cur[q][1], z[q], 0, 0, 0);
            z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, cur[q][0], z[q], 0, 0, 0);
          }
        if constexpr (kAhead) {
#pragma unroll
          for (int q = 0; q < QT; ++q)
#pragma unroll
            for (int t = 0; t < 3; ++t) cur[q][t] = nxt[q][t];
        }
      }
    } else if constexpr (MODE == 1) {
      // W as packed by sweep_pack_w_kernel: [k / 8][NB] vectors of 8 bfloat16 (zero beyond f_out)
      const sweep_bf16x8* __restrict__ Wp = reinterpret_cast<const sweep_bf16x8*>(fa.Wp);
      const int NB = nct * 32;
      constexpr int J = kRow / 16;
      sweep_bf16x8 cur[QT], nxt[QT];
#pragma unroll
      for (int q = 0; q < QT; ++q)
        if (q < nmy) cur[q] = Wp[(int64_t)h * NB + (ct0 + 2 * q) * 32 + r];
#pragma unroll 1
      for (int j = 0; j < J; ++j) {
        if (j + 1 < J) {
#pragma unroll
          for (int q = 0; q < QT; ++q)
            if (q < nmy) nxt[q] = Wp[(int64_t)(2 * (j + 1) + h) * NB + (ct0 + 2 * q) * 32 + r];
        }
        const float4 x0 = *reinterpret_cast<const float4*>(trow + 16 * j + 8 * h);
        const float4 x1 = *reinterpret_cast<const float4*>(trow + 16 * j + 8 * h + 4);
        sweep_bf16x8 a;
        a[0] = (__bf16)x0.x; a[1] = (__bf16)x0.y; a[2] = (__bf16)x0.z; a[3] = (__bf16)x0.w;
        a[4] = (__bf16)x1.x; a[5] = (__bf16)x1.y; a[6] = (__bf16)x1.z; a[7] = (__bf16)x1.w;
#pragma unroll
        for (int q = 0; q < QT; ++q)
          if (q < nmy) z[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, cur[q], z[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < QT; ++q) cur[q] = nxt[q];
      }
    } else {
      constexpr int J = kRow / 8;
      float cur[QT][4], nxt[QT][4];
      auto wload = [&](int j, float (&dst)[QT][4]) {
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          const int col = (ct0 + 2 * q) * 32 + r;
          const bool ok = q < nmy && col < fa.f_out;
#pragma unroll
          for (int i = 0; i < 4; ++i) dst[q][i] = ok ? fa.W[(int64_t)(8 * j + 4 * h + i) * fa.f_out + col] : 0.f;
        }
      };
      wload(0, cur);
#pragma unroll 1
      for (int j = 0; j < J; ++j) {
        if (j + 1 < J) wload(j + 1, nxt);
        const float4 x = *reinterpret_cast<const float4*>(trow + 8 * j + 4 * h);
        const float xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          if (q < nmy) {
#pragma unroll
            for (int i = 0; i < 4; ++i) z[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[i], cur[q][i], z[q], 0, 0, 0);
          }
        }
#pragma unroll
        for (int q = 0; q < QT; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) cur[q][i] = nxt[q][i];
      }
    }
    // Rows of the output this lane holds in a 32 x 32 accumulator tile: 8 * (v / 4) + 4 * h + v % 4, from `targets`.  (The
    // index is opaque because look-ups moved out of the loop hold their registers all the same; those from memory are made
    // all at once, a load between the stores would wait for them.)
    uint32_t t0 = rt * 32 + h * 4;
    asm volatile("" : "+v"(t0));
    if constexpr (FROM == TARGETS_BEHIND) {
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) far[v4] = *reinterpret_cast<const int4*>(targets + t0 + v4 * 8);
    }
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int col = (ct0 + 2 * q) * 32 + r;
      if (q >= nmy || col >= fa.f_out) continue;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        int4 t4;
        if constexpr (FROM != TARGETS_LDS) t4 = far[v4];
        else t4 = *reinterpret_cast<const int4*>(targets + t0 + v4 * 8);
        const int32_t tg[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (tg[v] < 0) continue;               // unused slot, or a piece of a split row
          const float zz = z[q][v4 * 4 + v];
          if (fa.Z) fa.Z[(int64_t)tg[v] * fa.f_out + col] = zz;
          if (fa.Hout) fa.Hout[(int64_t)tg[v] * fa.f_out + col] = fa.act == SAGNN_ACT_RELU ? (zz > 0.f ? zz : 0.f) : zz;
        }
      }
    }
  }
}

template <int FPL, int U, bool BUF, int MODE, bool TURN, Targets FROM = TARGETS_LDS>
__global__ __launch_bounds__(256, FPL == 1 ? 8 : 1) void spmm_sweep_fused_kernel(
    const uint32_t* __restrict__ code, const float* __restrict__ vals,
    const int32_t* __restrict__ wave_base, const int32_t* __restrict__ piece_target,
    const SpmmWsHeader* __restrict__ hdr, const float* __restrict__ B, float* __restrict__ partial,
    const SweepDims d, const SweepFusedArgs fa) {
  using vec = typename Vec<FPL>::T;
  extern __shared__ __attribute__((aligned(16))) float lds_acc[];  // [4 waves][16][kStride], then [4 waves][16] targets
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t loff = lane * (FPL * 4);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t block = run_block(d), w = block * 4 + wave;
  // (the launch has whole workgroups: n_waves is a multiple of 4, checked by the launcher)
  if (hdr->magic != kSpmmMagic || hdr->generation != d.generation || hdr->n_waves != d.n_waves ||
      hdr->groups != 1)
    return;
  constexpr int kRow = 64 * FPL, kStride = kRow + kPadRow;  // floats of an accumulator row (f_in), between two
  const int32_t target = piece_target[w * kSweepSlots + (lane & (kSweepSlots - 1))];
  float* __restrict__ my = lds_acc + (size_t)wave * kSweepSlots * kStride + lane * FPL;
  for (int s = 0; s < kSweepSlots; ++s) *reinterpret_cast<vec*>(my + s * kStride) = vec(0.f);

  const int32_t base = wave_base[w];
  const int32_t len = wave_base[w + 1] - base;  // a multiple of U (padded when built)
  const uint32_t* __restrict__ cw = code + base;
  const float* __restrict__ vw = vals + base;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B, d.b_bytes);

  walk_stream<FPL, U, BUF, false, TURN>(cw, vw, len, rs, B, d, loff, my, kStride);

  int32_t* __restrict__ targets = reinterpret_cast<int32_t*>(lds_acc + 4 * kSweepSlots * kStride);
  if (lane < kSweepSlots) targets[wave * kSweepSlots + lane] = target;
  // pieces of split rows to `partial`; T rows to memory if wanted
#pragma unroll 1
  for (int s = 0; s < kSweepSlots; ++s) {
    const int32_t tgt = piece_target[w * kSweepSlots + s];
    if (tgt == INT32_MIN) continue;
    const vec r = *reinterpret_cast<const vec*>(my + s * kStride);
    if (tgt >= 0) {
      if (fa.T) *reinterpret_cast<vec*>(reinterpret_cast<char*>(fa.T + (int64_t)tgt * kRow) + loff) = r;
    } else {
      const int64_t pi = -(int64_t)tgt - 1;
      *reinterpret_cast<vec*>(reinterpret_cast<char*>(partial + pi * d.f_total + d.col0) + loff) = r;
    }
  }
  __syncthreads();

  // tiles per pass: 4 at f = 256 (the LDS already limits a CU to two workgroups; 2 with three operand
  // terms per tile in registers), 1 below
  sweep_dense_epilogue<kRow, MODE, (FPL == 4 ? (MODE == 2 ? 2 : 4) : 1), FROM>(
      lds_acc, FROM != TARGETS_LDS ? piece_target + block * 4 * kSweepSlots : targets, fa, wave, (int)lane);
}

// W (f_in x f_out, row-major fp32) -> [f_in / 8][NB] vectors of 8 bfloat16 (k fastest), NB = f_out
// rounded up to 32, zero beyond f_out: one 16-byte load then gives a lane its matrix-core operand
// planes = 3: the three bfloat16 terms of every element, one plane of that layout per term
__global__ __launch_bounds__(256) void sweep_pack_w_kernel(const float* __restrict__ W, int32_t f_in, int32_t f_out,
                                                           int32_t NB, __bf16* __restrict__ Wp, int32_t planes) {
  const int idx = blockIdx.x * 256 + threadIdx.x;     // one (k / 8, n) vector per thread
  if (idx >= (f_in / 8) * NB) return;
  const int kg = idx / NB, n = idx - kg * NB;
  const int64_t plane = (int64_t)(f_in / 8) * NB * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float w = n < f_out ? W[(int64_t)(kg * 8 + i) * f_out + n] : 0.f;
    if (planes == 3)
      split3(w, Wp[(int64_t)idx * 8 + i], Wp[plane + (int64_t)idx * 8 + i], Wp[2 * plane + (int64_t)idx * 8 + i]);
    else
      Wp[(int64_t)idx * 8 + i] = (__bf16)w;
  }
}

// Lane-group variant: the wavefront carries R independent streams (zipped in memory), lane
// group g = lanes [g*64/R, (g+1)*64/R) walks stream g.  A group's 64/R lanes move one whole row
// of B with V floats (16 bytes at V = 4) per lane, so one load instruction serves R entries.
// Column ids and values still arrive by scalar loads; a lane picks its group's pair with
// selects (the row offset is multiplied on the scalar side first).  Flushes are per group:
// lanes of other groups are masked off by the divergent branch.
// FUSE: 0 the product alone; 1 / 2 / 3 the layer form: the kernel ends with the dense transform of the
// workgroup's rows (fp32 / bfloat16 / three-term operands, see sweep_dense_epilogue) instead of storing T (C is
// then only written if the caller wants T as a by-product: fa.T).
template <int V, int R, int U, bool BUF, int FUSE = 0, bool ODD = false, bool AHEAD = true, bool TWO = ODD && R == 4>
__global__ __launch_bounds__(256) void spmm_sweep_group_kernel(
    const uint32_t* __restrict__ code, const float* __restrict__ vals,
    const int32_t* __restrict__ wave_base, const int32_t* __restrict__ piece_target,
    const SpmmWsHeader* __restrict__ hdr, const float* __restrict__ B, float* __restrict__ C,
    float* __restrict__ partial, const int32_t* __restrict__ sync_off,
    uint32_t* __restrict__ barrier, const float* __restrict__ sched, const SweepDims d,
    const SweepFusedArgs fa) {
  using vec = typename Vec<V>::T;
  constexpr int LG = 64 / R;             // lanes per group = lanes per row
  const int kRow = ODD ? d.fw : LG * V;  // floats per row of this launch
  const int kStride = FUSE != 0 ? kRow + kPadRow : kRow;
  extern __shared__ __attribute__((aligned(16))) float lds_acc[];  // [4 waves][d.slots][kStride]
  const int SL = d.slots / R;            // slots per group
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t gid = lane / LG, lig = lane % LG;
  const uint32_t el = row_element<ODD>(lig * V, V, d.fw);
  const uint32_t loff = el * 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t w = run_block(d) * 4 + wave;
  if (w >= d.n_waves) return;
  if (hdr->magic != kSpmmMagic || hdr->generation != d.generation || hdr->n_waves != d.n_waves ||
      hdr->groups != R)
    return;
  float* __restrict__ my = lds_acc + (size_t)wave * d.slots * kStride + el;
  for (int ls = 0; ls < SL; ++ls) *reinterpret_cast<vec*>(my + (gid * SL + ls) * kStride) = vec(0.f);

  [[maybe_unused]] int32_t target = 0;
  if constexpr (FUSE != 0) target = piece_target[w * kSweepSlots + (lane & (kSweepSlots - 1))];
  const int32_t base = wave_base[w];
  const int32_t steps = (wave_base[w + 1] - base) / R;   // a multiple of U (padded when built)
  const uint32_t* __restrict__ cw = code + base;
  const float* __restrict__ vw = vals + base;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B, d.b_bytes);
  // interval boundaries of this wavefront's stream (whole batches) and the barrier it shares
  // with the workgroups of its cohort on its XCD
  const bool with_barrier = d.n_intervals > 1;     // negative: same layout, no barriers
  const int n_iv = d.n_intervals < 0 ? -d.n_intervals : d.n_intervals;
  const int32_t* __restrict__ so = sync_off + w * (kSweepMaxIntervals + 1);
  uint32_t expected = 0;
  int bar_slot0 = 0;
  if (with_barrier) {
    const int64_t cohort = (int64_t)blockIdx.x / d.wg_per_cohort;
    const int64_t first = cohort * d.wg_per_cohort;
    int64_t last = first + d.wg_per_cohort;
    if (last > (int64_t)gridDim.x) last = gridDim.x;
    const int xg = (int)(blockIdx.x & 7);
    // workgroups b in [first, last) with b mod 8 == xg (first is a multiple of 8)
    expected = (uint32_t)((last - first - xg + 7) / 8) + (uint32_t)d.sync_test_extra;
    bar_slot0 = (int)((cohort * 8 + xg) * n_iv);
  }

  const bool paced = d.pace_ticks > 0.f && n_iv > 1;
  const uint64_t t_start = paced ? wall_clock64() : 0ull;

  TurnTaking turn(steps, d.turn);
  // Words of H steps in scalar registers, requested while the rows of the steps before are on their way: they come from
  // HBM, and waiting for them at the head of a batch left the address units idle.  With four groups half a batch, a whole
  // one does not fit the scalar registers (1547 and 1947 us for 1723 before: 233 k vertices, 114 M entries, f = 64).
  // f = 128 2313 -> 2102.  (Before the wavefronts took turns this cost more misses
  // than it gave.  One vector load per batch with DPP broadcasts instead, half the vector instructions: 2671, 4196;
  // vector loads return in order, so every row waits for the words before it.)
  // AHEAD false: operands over a size, where this costs more misses than it gives (sweep_launch; with four groups it pays
  // at all sizes but some: 3.5 M vertices of 40, f = 64 2802, 2863 without, 4 M 3773, 3348, 6 M of 30 4632, 4845).
  constexpr int kParts = R == 4 ? 2 : 1, H = U / kParts;
  uint32_t c[H][R];
  float v[H][R];
  auto words = [&](int32_t at) {
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int g = 0; g < R; ++g) {
        c[i][g] = cw[(at + i) * R + g];
        v[i][g] = vw[(at + i) * R + g];
      }
  };
  if (AHEAD && steps > 0) words(0);
  int32_t e = 0;
  for (int iv = 0; iv < n_iv; ++iv) {
    SegmentSum<vec, TWO> sum;   // (what the padding of the interval before left is not summed: see spmm_sweep_perm_kernel)
    const int32_t e_end = iv + 1 < n_iv ? so[iv + 1] : steps;
    for (; e < e_end; e += U) {
      turn.at(e);
      uint32_t mc[U];
      float mv[U];
      vec h[U];
#pragma unroll
      for (int p = 0; p < kParts; ++p) {
        if constexpr (!AHEAD) words(e + p * H);
#pragma unroll
        for (int i = 0; i < H; ++i) {
          const int u = p * H + i;
          mc[u] = c[i][0];
          mv[u] = v[i][0];
          if constexpr (BUF) {
            uint32_t off = (c[i][0] & kColMask) * d.row_bytes;
#pragma unroll
            for (int g = 1; g < R; ++g)
              if (gid == (uint32_t)g) {
                mc[u] = c[i][g];
                mv[u] = v[i][g];
                off = (c[i][g] & kColMask) * d.row_bytes;
              }
            off += loff;
            if constexpr (V == 1) h[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
            else if constexpr (V == 2) h[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
            else h[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
          } else {
            const char* rowp = reinterpret_cast<const char*>(B + (int64_t)(c[i][0] & kColMask) * d.ldb);
#pragma unroll
            for (int g = 1; g < R; ++g)
              if (gid == (uint32_t)g) {
                mc[u] = c[i][g];
                mv[u] = v[i][g];
                rowp = reinterpret_cast<const char*>(B + (int64_t)(c[i][g] & kColMask) * d.ldb);
              }
            h[u] = *reinterpret_cast<const vec*>(rowp + loff);
          }
        }
        // the words after these, while the rows are on their way (the last ones again at the end of the stream)
        __builtin_amdgcn_sched_barrier(0);
        const int32_t en = e + (p + 1) * H;
        if constexpr (AHEAD) words(en < steps ? en : e);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(h[u]));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        sum.add(u, mv[u], h[u]);
        if (mc[u] >> 31) {   // last entry of a (piece, slab) segment of this lane's group
          vec* p = reinterpret_cast<vec*>(my + __mul24((mc[u] >> kSweepColBits) & (kSweepSlots - 1), kStride));
          *p += sum.take();
        }
      }
      sum.batch_ends();
    }
    // between two intervals: wait for the cohort (barrier mode) or hold the wavefront to the
    // schedule (pacing); a wavefront with nothing in an interval still takes part
    if (iv + 1 < n_iv) {
      if (with_barrier) sweep_interval_barrier(barrier, bar_slot0 + iv, expected, d.sync_timeout_ticks);
      else if (paced) sweep_pace_until(t_start, d.pace_ticks * sched[iv + 1]);
    }
  }

#pragma unroll 1
  for (int ls = 0; ls < SL; ++ls) {
    const int slot = (int)gid * SL + ls;
    const int32_t tgt = piece_target[w * kSweepSlots + slot];
    if (tgt == INT32_MIN) continue;
    vec r = *reinterpret_cast<const vec*>(my + slot * kStride);
    if (tgt >= 0) {
      if constexpr (FUSE != 0) {
        if (fa.T) *reinterpret_cast<vec*>(reinterpret_cast<char*>(fa.T + (int64_t)tgt * kRow) + loff) = r;
      } else {
        vec* p = reinterpret_cast<vec*>(reinterpret_cast<char*>(C + (int64_t)tgt * d.ldc) + loff);
        if (d.accumulate) r += *p;
        *p = r;
      }
    } else {
      const int64_t pi = -(int64_t)tgt - 1;
      *reinterpret_cast<vec*>(reinterpret_cast<char*>(partial + pi * d.f_total + d.col0) + loff) = r;
    }
  }
  if constexpr (FUSE != 0) {
    // (whole workgroups: the launcher only takes this form when n_waves is a multiple of 4 and
    // every wavefront owns 16 slots)
    int32_t* __restrict__ targets = reinterpret_cast<int32_t*>(lds_acc + 4 * kSweepSlots * kStride);
    if (lane < kSweepSlots) targets[wave * kSweepSlots + lane] = target;
    __syncthreads();
    sweep_dense_epilogue<LG * V, FUSE - 1, 1>(lds_acc, targets, fa, wave, (int)lane);
  }
}

// Narrow operands (rows of 64 / 128 bytes): R = 16 / 8 lane groups of 4 / 8 lanes.  Too many
// groups for scalar selects, so a batch of 64 stream words (64/R steps x R groups) is fetched with
// one coalesced load per array and a step's group takes its word with a lane permute.  With 16
// groups each group owns a single piece and its register accumulator is the piece's accumulator
// (no LDS at all); with 8 groups two pieces per group share it through LDS as in the wide kernels.
// Padding multiplies row 0 of B by 0, which is no 0 where that row holds an infinity or NaN.  In the LDS forms it
// lands behind the last flush; here it would land in the result, so the steps behind the end of the wavefront's shortest
// stream are masked per lane (no check in the steps before: 1 M vertices, 50 M entries, training at f = 16
// 2281 us without and 2283 with the masks).
// TWO: two sums (SegmentSum), FOLD: the running sum is folded every 32 entries; with 16 groups always both, with 8 by the
// length of the segments (narrow_sums).
template <int R, bool BUF, bool ODD, bool TURN, bool TWO, bool FOLD>
__global__ __launch_bounds__(256) void spmm_sweep_perm_kernel(
    const uint32_t* __restrict__ code, const float* __restrict__ vals,
    const int32_t* __restrict__ wave_base, const int32_t* __restrict__ piece_target,
    const SpmmWsHeader* __restrict__ hdr, const float* __restrict__ B, float* __restrict__ C,
    float* __restrict__ partial, const int32_t* __restrict__ sync_off, const SweepDims d) {
  typedef float vec __attribute__((ext_vector_type(4)));
  constexpr int LG = 64 / R;             // lanes per group = lanes per row
  const int kRow = ODD ? d.fw : LG * 4;  // floats per row
  constexpr int SL = kSweepSlots / R;    // pieces per group
  constexpr int UB = 64 / R;             // steps per batch of 64 stream words
  constexpr int NB = 8 / UB;             // batches per iteration: 8 steps (gathers) in flight
  extern __shared__ __attribute__((aligned(16))) float lds_acc[];  // [4 waves][16 slots][kRow], SL > 1 only
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t gid = lane / LG, lig = lane % LG;
  const uint32_t el = row_element<ODD>(lig * 4, 4, d.fw);
  const uint32_t loff = el * 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t w = run_block(d) * 4 + wave;
  if (w >= d.n_waves) return;
  if (hdr->magic != kSpmmMagic || hdr->generation != d.generation || hdr->n_waves != d.n_waves ||
      hdr->groups != R)
    return;
  float* __restrict__ my = lds_acc + (size_t)wave * kSweepSlots * kRow + el;
  if constexpr (SL > 1) {
#pragma unroll
    for (int ls = 0; ls < SL; ++ls) *reinterpret_cast<vec*>(my + (gid * SL + ls) * kRow) = vec(0.f);
  }
  const int32_t base = wave_base[w];
  const int32_t steps = (wave_base[w + 1] - base) / R;   // a multiple of 8 (padded when built)
  const uint32_t* __restrict__ cw = code + base;
  const float* __restrict__ vw = vals + base;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B, d.b_bytes);

  int32_t own = 0, all_own = 0;          // SL == 1: steps of this group's stream, of the shortest stream
  if constexpr (SL == 1) {
    own = sync_off[w * (kSweepMaxIntervals + 1) + kSweepOwnSteps + gid];
    all_own = own > 0 ? own : steps;     // (a group without a piece: nothing of it is stored)
#pragma unroll
    for (int o = LG; o < 64; o <<= 1) {
      const int32_t t = __shfl_xor(all_own, o, 64);
      all_own = t < all_own ? t : all_own;
    }
    all_own = __builtin_amdgcn_readfirstlane(all_own);
  }

  [[maybe_unused]] vec tot = 0.f;
  auto walk = [&](auto sum, auto folded) {
    constexpr bool kFold = decltype(folded)::value;
    uint32_t cb[NB];
    float vb[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      cb[q] = steps > 0 ? cw[q * 64 + lane] : 0u;
      vb[q] = steps > 0 ? vw[q * 64 + lane] : 0.f;
    }
    [[maybe_unused]] TurnTaking turn(steps, d.turn);
    for (int32_t e = 0; e < steps; e += 8) {
      if constexpr (TURN) turn.at(e);
      // the next iteration's stream words are requested before this one's gathers are waited for
      const bool more = e + 8 < steps;
      uint32_t ncb[NB];
      float nvb[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        ncb[q] = more ? cw[(e + 8) * R + q * 64 + lane] : 0u;
        nvb[q] = more ? vw[(e + 8) * R + q * 64 + lane] : 0.f;
      }
      uint32_t mc[8];
      float mv[8];
      vec h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        mc[u] = (uint32_t)__shfl((int)cb[u / UB], (u % UB) * R + (int)gid, 64);
        mv[u] = __shfl(vb[u / UB], (u % UB) * R + (int)gid, 64);
        const uint32_t col = mc[u] & kColMask;
        if constexpr (BUF) {
          h[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(rs, col * d.row_bytes + loff, 0, 0));
        } else {
          h[u] = *reinterpret_cast<const vec*>(reinterpret_cast<const char*>(B + (int64_t)col * d.ldb) + loff);
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(h[u]));
      if constexpr (SL > 1) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          sum.add(u, mv[u], h[u]);
          if (mc[u] >> 31) {   // last entry of a (piece, slab) segment of this lane's group
            vec* p = reinterpret_cast<vec*>(my + __mul24((mc[u] >> kSweepColBits) & (kSweepSlots - 1), kRow));
            if constexpr (kFold) {
              *p += tot + sum.take();
              tot = 0.f;
            } else {
              *p += sum.take();
            }
          }
        }
      } else {
        if (e + 8 <= all_own) {
#pragma unroll
          for (int u = 0; u < 8; ++u) sum.add(u, mv[u], h[u]);
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (e + u < own) sum.add(u, mv[u], h[u]);
        }
      }
      sum.batch_ends();
      // (folded every 32 entries: with 16 groups there are no slots to flush into; four groups and two would be 1 to 3 % slower
      // for 0.2 to 2 %, what is left there are the entries outside a community)
      if constexpr (kFold)
        if ((e & 31) == 24) tot += sum.take();
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        cb[q] = ncb[q];
        vb[q] = nvb[q];
      }
    }
    if constexpr (SL == 1) tot += sum.take();
  };
  if constexpr (SL > 1) {
    if (w >= d.long_waves) walk(ShortRowSum<vec>{}, std::false_type{});
    else walk(SegmentSum<vec, TWO>{}, std::integral_constant<bool, FOLD>{});
  } else {
    walk(SegmentSum<vec, TWO>{}, std::integral_constant<bool, FOLD>{});
  }

#pragma unroll 1
  for (int ls = 0; ls < SL; ++ls) {
    const int slot = (int)gid * SL + ls;
    const int32_t tgt = piece_target[w * kSweepSlots + slot];
    if (tgt == INT32_MIN) continue;
    vec r = tot;
    if constexpr (SL > 1) r = *reinterpret_cast<const vec*>(my + slot * kRow);
    if (tgt >= 0) {
      vec* p = reinterpret_cast<vec*>(reinterpret_cast<char*>(C + (int64_t)tgt * d.ldc) + loff);
      if (d.accumulate) r += *p;
      *p = r;
    } else {
      const int64_t pi = -(int64_t)tgt - 1;
      *reinterpret_cast<vec*>(reinterpret_cast<char*>(partial + pi * d.f_total + d.col0) + loff) = r;
    }
  }
}

// rows cut into several pieces: C[row] (+)= sum of the pieces' partial rows, fixed order
__global__ __launch_bounds__(256) void sweep_combine_kernel(
    const int32_t* __restrict__ multi_row, const int32_t* __restrict__ multi_first,
    const float* __restrict__ partial, const SpmmWsHeader* __restrict__ hdr, uint64_t generation,
    int64_t n_multi, float* __restrict__ C, int64_t ldc, int32_t f_total, int32_t accumulate) {
  const int lane = threadIdx.x & 63;
  const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
  if (q >= n_multi) return;
  if (hdr->magic != kSpmmMagic || hdr->generation != generation) return;
  const int32_t row = multi_row[q];
  const int32_t a = multi_first[q], b = multi_first[q + 1];
  for (int c4 = lane; c4 * 4 < f_total; c4 += 64) {
    float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0;
    int32_t j = a;
    for (; j + 2 <= b; j += 2) {
      const float4 t0 = *reinterpret_cast<const float4*>(partial + (int64_t)j * f_total + c4 * 4);
      const float4 t1 = *reinterpret_cast<const float4*>(partial + (int64_t)(j + 1) * f_total + c4 * 4);
      s0.x += t0.x; s0.y += t0.y; s0.z += t0.z; s0.w += t0.w;
      s1.x += t1.x; s1.y += t1.y; s1.z += t1.z; s1.w += t1.w;
    }
    if (j < b) {
      const float4 t0 = *reinterpret_cast<const float4*>(partial + (int64_t)j * f_total + c4 * 4);
      s0.x += t0.x; s0.y += t0.y; s0.z += t0.z; s0.w += t0.w;
    }
    float4* p = reinterpret_cast<float4*>(C + (int64_t)row * ldc + c4 * 4);
    float4 o = accumulate ? *p : make_float4(0.f, 0.f, 0.f, 0.f);
    o.x += s0.x + s1.x; o.y += s0.y + s1.y; o.z += s0.z + s1.z; o.w += s0.w + s1.w;
    *p = o;
  }
}

std::atomic<uint64_t> g_generation{1};

// Floats per accumulator row for which LDS is asked.  Rows of 97 to 127 floats would let a fifth workgroup onto a CU;
// four are faster because their wavefronts drift apart less (1 M vertices, 50 M entries, f = 100: 1592 against
// 1943 us; f = 80 with six workgroups 1326 against 1337; above 128 every further wavefront counts: f = 140 2088 against
// 3052 us with the two that rows of 256 allow).
int32_t sweep_lds_width(int32_t fw) { return fw > 96 && fw < 128 ? 128 : fw; }

}  // namespace

// ---------------------------------------------------------------------------------------
// host side of the preparation: the launch shape (lane groups, slots, windows, wavefronts per
// window) is decided here from a handful of totals; classifying rows, cutting long rows into
// pieces, dealing the pieces to the streams of the wavefronts (largest first, each to the
// shortest stream so far, so the streams have nearly equal lengths) and the compacted short-row
// CSR are device work (sweep_plan.hip), as is the layout of the streams (the passes above).
int sweep_prepare(const int32_t* d_rowptr, const int32_t* d_colidx, const float* d_val, int64_t m,
                  int64_t k, int64_t nnz, int32_t f, char* ws, const SpmmWsLayout& L,
                  const sagnn_spmm_options& opt, bool no_hubs, hipStream_t s, SweepPlanResult* out) {
  out->use_sweep = false;
  const int force = opt.schedule == 1 ? 0 : (opt.schedule == 2 ? 1 : -1);
  if (force == 0 || nnz < 4096 || k <= 0 || k >= (1ll << kSweepColBits) || m <= 0) return SAGNN_OK;
  const int64_t b_bytes = k * (int64_t)f * 4;
  // worth it only if B is much larger than an L2 (the long-row share is checked below) and there are enough entries
  // for balanced streams on every CU (2.4 M entries: 129 against 139 us at f = 128, 49 against 67 at f = 16; 4 M: 154
  // against 146 the other way), or if there are no hubs (rows of more than 32 chunks of nonzero splitting; a tenth of the
  // entries at most in rows that are cut into pieces, see below): then 1 M entries are enough, whatever
  // the size of B.  us by nonzero splitting and swept, random columns: 30 k vertices of 48, f = 16, 64, 256 34, 45, 190 and
  // 15, 33, 123; 100 k of 24 47, 91, 352 and 33, 64, 250; 100 k of 64, f = 16 109 and 50; 10 k of 120 28, 29, 115 and 17,
  // 30, 72; in communities: 30 k of 64 42, 44, 162 and 22, 38, 136; a row block of 85 k rows of 30, f = 64, 256 97, 375 and
  // 56, 217.  Under 1 M entries some lose: 30 k of 24 in communities, f = 100, 256 36, 89 and 46, 101.
  if (force != 1 && (no_hubs ? nnz < (1 << 20) : !sweep_size(k, nnz, f))) return SAGNN_OK;

  if (!sweep_plan_fits(L)) return SAGNN_OK;
  int piece_max = opt.piece > 0 ? opt.piece : (force == 1 ? 4096 : sweep_piece_default(nnz, f));
  if (piece_max < sweep_piece_floor(nnz, f)) piece_max = sweep_piece_floor(nnz, f);
  if (piece_max > 32768) piece_max = 32768;
  constexpr int kLocalPermille = 400;   // (between what the two kinds of order measure, see the windows below)
  const bool tree = f > 16 && f < 128 && f != 64;
  SweepRowTotals tot{};
  // Without hubs, small: short rows are swept beside the others above 32 columns only (100 k rows of 16, 55 % of the entries
  // in rows of 16 or more, f = 16 29 us by nonzero splitting, 31 swept); hardly any re-use (a rank's 125 k rows of 15 by
  // 8 M columns, f = 64, 256 85, 298 and 124, 321).  Nonzero splitting adds as a tree at the widths under 128 but 64, and a
  // row's sum here has a term per slab: not swept at these where the slabs that locality needs are more than a row's
  // entries fill (a row block of 85 k rows of 30 in communities, f = 100 6.7e-8 from 64 bits, 7.5e-8 in the slabs of the
  // other widths, 6.8e-8 in so few that nothing is gained), nor long rows in many small communities, whose entries elsewhere
  // are each a term (16 communities, 16 k of 75 f = 48 7.7e-8, 7.9e-8, of 140 f = 48, 100 8.5e-8, 9.0e-8, 9.0e-8, 9.0e-8).
  // And few long rows make few streams, long ones: by nonzero splitting and swept 5 k of 220 f = 48, 64 23, 23 and 32, 33 us, 10 k
  // of 228 f = 32, 48, 64 29, 38, 36 and 36, 41, 43, in communities, where the streams of a window are fewer, f = 48, 64, 128
  // 36, 35, 54 and 57, 59, 59, 15 k of 180 f = 48, 64 44, 41 and 54, 53, 10 k of 228 f = 4 25, 27; but random columns, 10 k of 160, f = 16, 32, 256 30, 27,
  // 148 and 18, 25, 76.
  auto small_refused = [&]() {
    const int64_t long_entries = nnz - tot.short_entries;
    const bool local = tot.locality >= kLocalPermille;
    const double span = (double)k * tot.span / 1000.0, deg = (double)nnz / (double)m;
    const bool few = (double)m < 64.0 * deg;
    return (f <= 32 && long_entries * 10 < nnz * 9) || (double)nnz < 8.0 * span || (tree && !local && 2.0 * span < (double)k) ||
           (tree && f > 32 && local && 8.0 * span < (double)k && deg >= (f < 64 ? 64.0 : 128.0)) ||
           (f > 32 && f <= 64 && (few || (local && (double)m < 128.0 * deg))) || (f <= 32 && few && deg >= 200.0) ||
           (f > 64 && local && few && deg >= 150.0) || long_entries * 10 < nnz * 3 ||
           (opt.groups != 2 && f <= 32 && long_entries < 8 * k);
  };
  // (without hubs every row that may be is long: sixteen short rows of up to 63 entries are several times the stream of a
  // small matrix' other wavefronts.  15 k rows of 80, f = 64, 256 32, 139 us by nonzero splitting, 46, 126 with rows from
  // 64 entries on long, 27, 78 from 16 on)
  const int32_t min_long = no_hubs && opt.min_long <= 0 ? kSweepMinLong : opt.min_long;   // (negative: "where 64 is picked")
  if (no_hubs && opt.groups != 2 && f <= 32 && nnz < 8 * k) return SAGNN_OK;              // (see small_refused)
  {
    // (small matrices that are refused are so by what the sample tells: looking costs them 50 us, with the pass over their
    // rows 90; 100 k rows of 16, f = 16 49 us without, 99)
    int rc = sweep_plan_sample(d_rowptr, d_colidx, m, k, nnz, min_long, ws, L, s, no_hubs ? &tot : nullptr);
    if (rc != SAGNN_OK) return rc;
    if (no_hubs && (tot.bad || small_refused())) return SAGNN_OK;
    // Row classification, the short-row CSR, the list of split rows and one record per piece are
    // made on the device (the long-row threshold is chosen there from the degree distribution);
    // the host gets the totals.
    rc = sweep_plan_rows(d_rowptr, m, piece_max, ws, L, s, &tot, opt.short_rows >= 0);
    if (rc != SAGNN_OK) return rc;
  }
  if (tot.bad) return SAGNN_OK;   // not a CSR row pointer for this nnz: keep the plain schedule
  const int64_t P = tot.pieces, short_rows = tot.short_rows, short_entries = tot.short_entries;
  const int64_t long_entries = nnz - short_entries;
  const bool has_empty = tot.has_empty;

  // Lane groups: at f = 128 half a wavefront, at f = 64 a quarter, moves a whole row of B with
  // 16 bytes per lane, so one load instruction serves 2 / 4 entries (the vector-memory issue
  // rate, not bandwidth, bounds B-in-cache cases).  Other widths keep one row per instruction.
  // They pay when the rows of B are re-used from cache (issue-bound: 233 k-vertex graph
  // 3.38 -> 2.63 ms, 2.45 M-vertex graph 4.85 -> 4.62 ms) and cost ~3 % when almost every gather
  // misses (rank share of the 111 M-vertex graph, 2.6 entries per row of B): decided below by
  // the average number of swept entries per row of B.
  // Narrow operands (f <= 32, 16: 8 / 4 lanes a row) exist only in the grouped form, 8 / 16 rows per load.  Widths
  // between the powers of two take the next wider form (124 M entries, 2.45 M vertices: f = 24 2513 us by nonzero
  // splitting, 1905 swept; f = 48 3599 and 2560, f = 100 8135 and 5407, f = 200 13857 and 8598).
  // Wider operands (multiples of 64 above 128) can be taken as 128-wide slabs by the two-group
  // kernels (a last slab of 64 is served by the same streams): an option, see sagnn_spmm_options.
  const bool narrow_slabs = opt.slab_width == 128 && f > 128 && (f & 63) == 0 && opt.groups != 1;
  // Columns 64 at a time, one row per load and one stream per wavefront, where the product costs what its L2 misses cost
  // and the rows that are resident together want the same rows of B: an XCD holds 16384 rows of A then (256 workgroups of
  // 16 KB), four times as many as at 256 columns, so a row of B is wanted that many times more often while they pass over
  // it; sixteen rows in one stream stand at the same column to within 2 % of the stream where four streams of four rows
  // are 4 % apart; and a load of one float per lane keeps the address units busy for 8.5 clocks (two rows of four 17).
  // us as before (256 columns at once; two streams of 128; four of 64) and so, f = 256, 128, 64: 16 communities of 125 k
  // vertices, 84 M entries 10999, 5557, 2866 -> 7131, 3524, 1837; of 62 k, 30 M 3719, 1834, 893 -> 2818, 1479, 852; one of
  // the former as a row block 590, 279, 134 -> 424, 200, 105; random columns, 250 k vertices of 60 1864, 973, 501 -> 1265,
  // 642, 329; 1 M of 40 5825, 2829, 1461 -> 5200, 2598, 1298.
  // Not where the columns that neighbouring rows choose from fit the L2s anyway (communities of 19 k, f = 256: 1242 as
  // before, 1412 so; of 5 k: 480, 536) or nearly (of 44 k, 36 a row, f = 64, 128, 256 695, 1428, 2828 and 786, 1400, 2539, and
  // inference, whose dense part needs the whole width in one launch, at f = 128 1628 and 1831) or rows are short (of 125 k,
  // 16 a row, f = 64, 256 1129, 4835 and 1180, 4696; 24 a row 1557, 6355 and 1338, 5005), where there are too many for a
  // second use (a rank's rows; random columns, 500 k of 18, f = 128 661 and 653, 1 M of 30 in inference 2278 and 2392), and
  // not with hubs, whose rows hit in any case (233 k vertices of 489: 5627, 7060).  Nor where the columns go along with the
  // rows: resident rows then begin in different slabs, and the more of them there are the more slabs (1 M rows of 40 within
  // 50 k of the diagonal, f = 64, 128, 192, 256 973, 2417, 3276, 5094 and 1304, 2634, 4014, 5084).
  const bool local = tot.locality >= kLocalPermille;
  const double span = (double)k * tot.span / 1000.0;
  // how often the 16384 rows of A that an XCD holds at 64 columns a launch want a row of the columns they choose from
  const double reuse = 16384.0 * (double)nnz / (std::max(span, 1.0) * (double)m);
  const bool hubs = 10 * tot.multi_pieces * (int64_t)piece_max > nnz;   // a tenth of the entries in rows that are cut
  const bool col_groups = f >= 64 && (f & 63) == 0 && opt.groups == 0 && opt.slab_width == 0 && opt.sync_slabs <= 0 &&
                          opt.barriers != 1 && opt.pace_ps_per_step <= 0 && span >= 40000.0 &&
                          reuse >= 0.6 && !hubs &&
                          (!local || (nnz >= 18 * m && span >= 60000.0 && tot.slide < 600));
  int64_t R = narrow_slabs ? 2 : (f > 128 ? 1 : (f > 64 ? 2 : (f > 32 ? 4 : (f > 16 ? 8 : 16))));
  if ((opt.groups == 1 && f > 32) || col_groups) R = 1;
  if (force != 1 && long_entries * 10 < nnz * 3) return SAGNN_OK;   // < 30 % of the entries
  if (no_hubs && (hubs || small_refused())) return SAGNN_OK;
  if (opt.groups != 2 && long_entries < 8 * k) {
    if (f <= 32) return SAGNN_OK;  // one row per instruction would leave most lanes idle: plain schedule
    R = 1;
  }
  if (P <= 0 || P > L.max_pieces) return SAGNN_OK;
  if (tot.multi_rows > L.max_multi_rows || tot.multi_pieces > L.max_multi_pieces) return SAGNN_OK;

  // Accumulator rows per wavefront.  A launch of width 128 with 16 rows per wavefront needs
  // 32768 bytes of LDS per workgroup, of which a CU holds four, not five (measured; the LDS
  // is handed out in units that make 5 x 32768 overshoot 160 KB).  14 rows (lane groups, 7 each)
  // or 15 rows bring the fifth workgroup in, 20 wavefronts and 280 / 300 rows per CU instead
  // of 16 and 256 -- measured slower free-running on the 2.45 M-vertex graph (5.4 against
  // 4.5 ms: more wavefronts drift apart more) and equal under pacing, so it is an option only.
  const bool has_128_slab = narrow_slabs || (f % 256) == 128 || (f % 256) == 192;
  const int64_t slots = has_128_slab && opt.narrow_slots == 1 ? (R == 2 ? 14 : 15) : kSweepSlots;
  // Pieces per wavefront: all slots when there are plenty of pieces; fewer when that would
  // leave the chip short of wavefronts (a row block of a partitioned graph has few long rows).
  int64_t slots_used = ceil_div(P, (int64_t)(opt.min_waves > 0 ? opt.min_waves : 8192));
  if (slots_used < R) slots_used = R;          // every lane group of a wavefront gets a piece
  if (slots_used > slots) slots_used = slots;
  while (slots_used < slots && ceil_div(P, slots_used) + 64 > L.max_waves - 8) ++slots_used;
  // Pieces are dealt window by window.  A window is a run of consecutive long rows holding a
  // few times as many pieces as the chip keeps resident at once (LDS-limited); inside a window
  // the pieces are sorted by size and dealt longest-first, so its wavefronts have nearly equal
  // stream lengths (they pass the slabs in step).  A matrix of up to ~4 generations is one
  // window (measured best on randomly labelled graphs: 4.95 ms against 5.4 ms with one window
  // per generation on the 2.45 M-vertex R-MAT graph).  Where the row order carries locality (row_locality) a
  // window of a quarter of a generation keeps its wavefronts in the part of B that its rows' neighbourhoods share.
  // One generation in four against four generations, 50 entries a row in 16 communities: 1 M vertices f = 16 783 ->
  // 418 us, f = 64 1733 -> 1420, f = 256 6383 -> 5960; 300 k vertices f = 16 208 -> 94, f = 256 1834 -> 1468; 2 M of
  // 42 f = 256 11213 -> 10942.  Random labels lose (1 M R-MAT vertices of 100 entries: f = 32 930 -> 1192 us).
  // The line lies between what the two kinds measure, 50 to 100 permille and 700 to 900.
  const int64_t fw_max = col_groups ? 64 : sweep_widest_launch(f, narrow_slabs ? 128 : 256);
  int64_t wg_per_cu = lds_resident_workgroups((size_t)(4ll * slots * sweep_lds_width(fw_max) * 4));
  if (wg_per_cu < 1) wg_per_cu = 1;
  int n_cus = 256;
  {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n_cus = v;
  }
  const int64_t resident_waves = (int64_t)n_cus * wg_per_cu * 4;
  int64_t window = resident_waves * slots_used;              // pieces per window
  {
    const int pct = opt.window_pct < 0 ? 0 : (opt.window_pct > 0 ? opt.window_pct : (local ? (col_groups ? 12 : 25) : 400));
    window = pct <= 0 ? P : std::max<int64_t>(slots_used, window * pct / 100);
  }
  if (window > P) window = P;
  if (ceil_div(P, window) > kSweepMaxWindows) window = ceil_div(P, kSweepMaxWindows);
  const int64_t nwin = ceil_div(P, window);
  // Wavefronts in all: whole generations of resident wavefronts when there is more than one
  // (the last generation then runs at the same occupancy, and under pacing at the same speed, as
  // the others), else as few as the slots allow.
  int64_t n_target_waves = ceil_div(P, slots_used);
  if (n_target_waves > resident_waves) {
    const int64_t up = round_up((size_t)n_target_waves, (size_t)resident_waves);
    if (up + 64 <= L.max_waves - 8) n_target_waves = up;
  }
  // (column groups without locality: not under 8192 rows a slab, which wide operands would get, 250 k vertices of 60, f = 256
  // 1286 -> 1254 us, a row block of a partitioned graph 445 -> 424; but while a row has at most 16 entries a slab, since the
  // sum of longer segments is further from exact: f = 256, 8192 rows and 4 MB a slab 60 k of 120 9.3e-8, 9.4e-8, of 200
  // 10.9e-8, 10.2e-8, of 489 15.3e-8, 12.8e-8, 120 k of 200 10.3e-8, 11.7e-8, of 489 12.8e-8, 12.9e-8.  Finer slabs than 4 MB
  // of the whole width for narrow operands would be up to 5 % faster, but a row's sum has a term per slab it has entries in,
  // and more terms are further from exact too: f = 64 8.7e-8 with 4 MB, 1.04e-7 with 2.)
  auto slabs_of = [&](int64_t bytes) { return bytes >= (1 << 16) ? 8 * ceil_div(b_bytes, 8 * bytes) : (int64_t)kSweepMaxSlabs; };
  int64_t S = slabs_of(opt.slab_kb < 0 ? 0 : (int64_t)(opt.slab_kb > 0 ? opt.slab_kb : 4096) << 10);
  if (opt.slab_kb == 0 && col_groups && !local && f > 128) {
    const int64_t coarse = std::max<int64_t>(8, slabs_of((int64_t)32 * f << 10));
    if (nnz <= 16 * coarse * m) S = coarse;
  }
  if (S < 8) S = 8;
  // Where the order of the rows carries locality at least four slabs (eight with 64 entries a row) in the columns that
  // neighbouring rows choose from: slabs of 4 MB may hold all of them, and then nothing keeps the wavefronts of a window in
  // step, and a row's entries are one long sum.  Sixteen communities, us and error against 64 bits before and so: 100 k
  // vertices of 40, f = 100, 256 204, 448, 11.4e-8, 8.9e-8 and 179, 378, 7.6e-8, 7.6e-8; 250 k of 100, f = 128, 256 1414,
  // 2441, 13.2e-8, 10.5e-8 and 1273, 2098, 9.5e-8, 9.5e-8; 250 k of 40, f = 64 284, 11.4e-8 and 276, 7.6e-8 (100 k, f = 64
  // 106 and 109, f = 32 48 and 52: not there).
  if (local && opt.slab_kb == 0 && (f > 64 || (f > 32 && b_bytes >= (48ll << 20))))
    S = std::max(S, (int64_t)((nnz >= 64 * m ? 8.0 : 4.0) * (double)k / std::max(span, 1.0) + 0.5));
  // Small matrices: the columns that neighbouring rows choose from in four slabs where the order of the rows carries
  // locality, in eight where all choose from the same; where nonzero splitting would add as a tree three and four; and at 17
  // to 32 columns, where a stream has two rows and longer segments are folded, one per 64 entries of a row in all columns
  // (an entry outside the community is a segment of its own in slabs of its size).  Error against 64 bits by nonzero splitting
  // and so, e-8: random columns, 30 k vertices of 60, f = 16, 32, 64, 100, 256 7.2, 7.4, 12.2, 7.7, 13.1 and 6.9, 6.9, 7.8, 7.0,
  // 7.8; sixteen communities 7.2, 7.4, 12.3, 7.7, 13.1 and 6.9, 6.9, 8.8, 7.64, 8.8, f = 48 7.59 and 7.64; of 110, f = 20, 48
  // 8.2, 8.5 and 7.9, 8.6 (f = 20 in slabs that follow the communities 8.7); 80 k of 31, f = 48, 100 6.82, 6.82 and 6.83,
  // 6.84 (in four slabs 6.90 at both).  In eight slabs for all 13.8e-8 from f = 64, and 131 us for 110 at f = 256.
  if (no_hubs && opt.slab_kb == 0) {
    if (f > 16 && f <= 32) S = ceil_div(nnz, 64 * m);
    else S = (int64_t)((tree ? (local ? 3.0 : 4.0) : (local ? 4.0 : 8.0)) * (double)k / std::max(span, 1.0) + 0.5);
  }
  if (S < 1) S = 1;
  if (S > kSweepMaxSlabs) S = kSweepMaxSlabs;
  const int64_t width = ceil_div(k, S);
  std::vector<int64_t> win_entries(1, long_entries);
  if (nwin > 1) {
    const int rc = sweep_plan_window_entries(ws, L, P, window, (int32_t)nwin, s, &win_entries);
    if (rc != SAGNN_OK) return rc;
  }
  // wavefronts of a window: as many as keep the stream length equal to the global average (equal
  // lengths in ALL windows keep successive generations in step), but never fewer than the slots
  // allow.  With R lane groups a wavefront carries R independent streams (group g owns slots
  // g*SL ..); the unit of dealing is then the group stream.
  const int64_t SL = slots / R;                 // slots per group stream
  std::vector<int32_t> win_unit0((size_t)nwin + 1);   // first stream of every window
  int64_t NW = 0;
  for (int64_t w = 0; w < nwin; ++w) {
    const int64_t a = w * window, b = std::min(P, a + window);
    const double target_len = (double)long_entries / (double)n_target_waves;
    int64_t nw = (int64_t)((double)win_entries[(size_t)w] / target_len + 0.5);
    nw = std::max(nw, ceil_div(b - a, slots));
    nw = std::max<int64_t>(nw, 1);
    nw = std::min(nw, b - a);
    win_unit0[(size_t)w] = (int32_t)(NW * R);
    NW += nw;
  }
  win_unit0[(size_t)nwin] = (int32_t)(NW * R);
  // whole workgroups of four wavefronts (the last ones may own no piece): the kernels' workgroup
  // barriers then never meet a wavefront that has left
  const int64_t NW4 = (NW + 3) / 4 * 4;
  if (NW4 > L.max_waves - 1) return SAGNN_OK;   // cannot happen with the bounds above; plain schedule
  // Option: the short rows are swept too, as whole rows -- 16 per wavefront, behind the wavefronts
  // of the long rows, every row one segment of its wavefront's stream -- instead of going through
  // the nonzero-splitting kernel.  Every row then ends in a wavefront's accumulator rows, which is
  // what the layer form with the dense transform as the sweep's epilogue needs.
  // Measured never slower than the nonzero-splitting kernel on the power-law graphs (233 k vertices:
  // 2.54 -> 2.50 ms, 2.45 M vertices: 2.78 -> 2.62 ms at f = 64, 4.24 -> 4.19 ms at f = 128), also
  // when the short rows are very short (2 M rows of which 92 % hold one entry each: 3.50 -> 3.38 ms).  With eight and sixteen
  // groups us so for in kernels of their own, power-law 1 M vertices of 50 f = 16, 24, 32 472, 588, 522 -> 398, 510, 444, of 14
  // f = 16, 32 199, 250 -> 161, 180, 2.45 M of 51 1232, 1370 -> 1094, 1184, 233 k of 489 815, 900 -> 760, 854; random columns, 100 k of
  // 20 28, 36 -> 22, 30; communities, 500 k of 18 94, 133 -> 79, 117; and the preparation, which does without the tables of
  // nonzero splitting, 1340, 1260 -> 1060, 1110 (1 M of 50).  A row of theirs is padded by up to seven steps: where the streams
  // have room for twice that.
  const bool roomy = 7 * (short_rows + kSweepSlots) + 4096 <= (L.stream_cap - nnz) / 2;
  bool whole_rows = opt.short_rows >= 0 &&
                    short_rows > 0 && tot.min_long <= 255 && slots == kSweepSlots && (R <= 4 || roomy) &&
                    P + short_rows <= L.max_pieces && opt.sync_slabs <= 0 && opt.barriers != 1 &&
                    opt.pace_ps_per_step <= 0;
  int64_t NWT4 = NW4;
  if (whole_rows) {
    NWT4 = NW4 + (ceil_div(short_rows, (int64_t)kSweepSlots) + 3) / 4 * 4;
    if (NWT4 > L.max_waves - 1) {
      whole_rows = false;
      NWT4 = NW4;
    }
  }
  const int64_t short_entries_csr = whole_rows ? 0 : short_entries;   // entries of the compacted short-row CSR
  // Inside a window: largest piece first, each to the stream that is shortest so far and still
  // has a free slot.  Streams come out equal to within a piece of the smallest size class, which
  // keeps the wavefronts in step from slab to slab.  A piece at a time to half of the streams; to all of them in column groups,
  // which have no hubs and sixteen pieces a stream at every width: the longest stream is as long, the product as fast, and of
  // the launches of the dealing, which take most of such a preparation, half are left (300 k random rows of 20, f = 64, 256
  // 1395, 1420 -> 937, 960 us; 1.5 M of 42 in communities 4250 -> 3498).
  {
    const bool snake = R == 1 && opt.snake == 1;
    int rc = sweep_plan_deal(ws, L, P, window, win_unit0.data(), (int32_t)nwin, NWT4, (int32_t)R,
                             (int32_t)SL, piece_max, snake, col_groups, s);
    if (rc != SAGNN_OK) return rc;
    if (whole_rows) {
      rc = sweep_plan_deal_short(ws, L, P, short_rows, NW4, s);
      if (rc != SAGNN_OK) return rc;
    }
  }

  // Interval barriers (lane-group kernels only): every `sync_slabs` slabs the workgroups of an
  // XCD that run together wait for each other.  Decided here, laid out by the device passes.
  // (the interval layout costs ~3 % of padding, so it is only made when something will use it)
  int64_t sync_slabs = opt.sync_slabs < 0 ? 0 : (opt.sync_slabs > 0 ? opt.sync_slabs : 16);
  if (opt.barriers != 1 && opt.pace_ps_per_step <= 0 && opt.sync_slabs <= 0) sync_slabs = 0;
  if ((R != 2 && R != 4) || whole_rows) sync_slabs = 0;   // (whole-row wavefronts have no slab intervals)
  if (sync_slabs > 0 && ceil_div(S, sync_slabs) > kSweepMaxIntervals) sync_slabs = ceil_div(S, kSweepMaxIntervals);
  int64_t NI = sync_slabs > 0 ? ceil_div(S, sync_slabs) : 1;
  if (NI <= 1) { NI = 1; sync_slabs = 0; }

  // long rows must be column-sorted for the slab segmentation (the counting pass looks)
  int32_t* d_flag = reinterpret_cast<int32_t*>(ws + L.carry);  // scratch until the first product; zeroed by the row pass
  struct { int32_t unsorted; SweepScanRecord scan; } rec{};
  static_assert(sizeof(rec) == 24, "one copy brings both");
  const uint32_t kmax = (uint32_t)(k - 1);
  const int32_t* d_info = reinterpret_cast<const int32_t*>(ws + L.piece_info);
  int32_t* d_wave_base = reinterpret_cast<int32_t*>(ws + L.wave_base);
  int32_t* d_wave_steps = reinterpret_cast<int32_t*>(ws + L.wave_steps);
  int32_t* d_sync_off = reinterpret_cast<int32_t*>(ws + L.sync_off);
  const size_t count_lds = sweep_count_lds_bytes(S), build_lds = sweep_build_lds_bytes(S);
  SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(sweep_count_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)count_lds));
  const auto build = R >= 4 && !local ? sweep_build_kernel<true> : sweep_build_kernel<false>;
  SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(build),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)build_lds));
  KeptTables kept{reinterpret_cast<int32_t*>(ws + L.code), reinterpret_cast<int32_t*>(ws + L.vals),
                  (L.stream_cap - ceil_div(NW4, 2) * kSweepSlots * (S + 1)) / 64 * 64};
  if (L.stream_cap < ceil_div(NW4, 2) * kSweepSlots * (S + 1)) kept.from = -1;
  int64_t stream_len = 0, short_base = 0;
  for (int attempt = 0; attempt < 2; ++attempt) {
    hipLaunchKernelGGL(sweep_count_kernel, dim3((unsigned)NW4), dim3(kBuildThreads), count_lds, s, d_rowptr,
                       d_colidx, d_info, (int32_t)S, (int32_t)width, kmax, (int32_t)R, (int32_t)SL, (int32_t)NI,
                       (int32_t)sync_slabs, d_sync_off, d_wave_steps, d_flag, kept);
    SAGNN_LAUNCH_CHECK();
    if (NWT4 > NW4) {
      hipLaunchKernelGGL(sweep_short_count_kernel, dim3((unsigned)ceil_div(NWT4 - NW4, kBuildThreads / kSweepSlots)),
                         dim3(kBuildThreads), 0, s, d_rowptr, d_info, NW4, NWT4, (int32_t)SL, d_sync_off, d_wave_steps);
      SAGNN_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(sweep_scan_kernel, dim3((unsigned)std::max<int64_t>(1, ceil_div(NWT4, kScanTile))), dim3(1024), 0, s,
                       d_wave_steps, NWT4, (int32_t)R, d_wave_base, reinterpret_cast<SweepScanRecord*>(d_flag + 1));
    SAGNN_LAUNCH_CHECK();
    SAGNN_HIP(hipMemcpyAsync(&rec, d_flag, sizeof(rec), hipMemcpyDeviceToHost, s));
    SAGNN_HIP(hipStreamSynchronize(s));    // also: win_unit0 has been consumed
    if (rec.unsorted || rec.scan.left) return SAGNN_OK;   // unsorted long row, column out of range, pieces left over: plain schedule
    stream_len = rec.scan.total;
    short_base = (int64_t)round_up((size_t)stream_len + 64, 256);
    const bool fits = !rec.scan.overflow && short_base + short_entries_csr + 256 <= L.stream_cap;
    if (fits) break;
    if (whole_rows && R > 4) {             // (their streams' padding did not fit: with the short rows beside the sweep)
      sagnn_spmm_options apart = opt;
      apart.short_rows = -1;
      return sweep_prepare(d_rowptr, d_colidx, d_val, m, k, nnz, f, ws, L, apart, no_hubs, s, out);
    }
    if (attempt == 1 || NI == 1) return SAGNN_OK;
    NI = 1;                                // the interval padding did not fit: lay out without it
    sync_slabs = 0;
  }

  if (NI > 1) {   // (the schedule of paced intervals; without intervals nothing reads it)
    hipLaunchKernelGGL(sweep_sched_kernel, dim3((unsigned)(NI + 1)), dim3(256), 0, s, d_sync_off, NWT4, (int32_t)NI,
                       reinterpret_cast<float*>(ws + L.sched));
    SAGNN_LAUNCH_CHECK();
  }
  if (stream_len > kept.from) kept.from = -1;   // (the streams take the place of the tables)
  hipLaunchKernelGGL(build, dim3((unsigned)NW4), dim3(kBuildThreads), build_lds, s, d_rowptr,
                     d_colidx, d_val, d_info, d_wave_base, d_sync_off, (int32_t)S, (int32_t)width, kmax,
                     (int32_t)R, (int32_t)SL, (int32_t)NI, (int32_t)sync_slabs, reinterpret_cast<uint32_t*>(ws + L.code),
                     reinterpret_cast<float*>(ws + L.vals), kept);
  SAGNN_LAUNCH_CHECK();
  if (NWT4 > NW4) {
    hipLaunchKernelGGL(sweep_short_build_kernel, dim3((unsigned)ceil_div(NWT4 - NW4, kBuildThreads / 64)), dim3(kBuildThreads), 0,
                       s, d_rowptr, d_colidx, d_val, d_info, d_wave_base, NW4, NWT4, kmax, (int32_t)R, (int32_t)SL,
                       reinterpret_cast<uint32_t*>(ws + L.code), reinterpret_cast<float*>(ws + L.vals));
    SAGNN_LAUNCH_CHECK();
  }
  // zero the gap between the long stream and the short entries (tail batches read into it)
  hipLaunchKernelGGL(sweep_zero_gap_kernel, dim3(1), dim3(256), 0, s,
                     reinterpret_cast<uint32_t*>(ws + L.code) + stream_len,
                     reinterpret_cast<float*>(ws + L.vals) + stream_len, (int32_t)(short_base - stream_len));
  SAGNN_LAUNCH_CHECK();
  if (short_rows > 0 && !whole_rows) {
    hipLaunchKernelGGL(sweep_short_copy_kernel, dim3((unsigned)ceil_div(short_rows, 256)), dim3(256), 0, s,
                       d_rowptr, d_colidx, d_val, reinterpret_cast<const int32_t*>(ws + L.rowptr_s),
                       reinterpret_cast<const int32_t*>(ws + L.rowmap_s), short_rows,
                       reinterpret_cast<int32_t*>(ws + L.code) + short_base,
                       reinterpret_cast<float*>(ws + L.vals) + short_base);
    SAGNN_LAUNCH_CHECK();
  }

  SpmmWsHeader& h = out->hdr;
  h = SpmmWsHeader{};
  h.magic = kSpmmMagic;
  h.has_empty_rows = has_empty ? 1 : 0;
  h.m = m; h.nnz = nnz; h.f = f; h.mode = 1;
  h.generation = g_generation.fetch_add(1);
  h.c_rows = whole_rows ? 0 : short_rows; h.c_nnz = short_entries_csr; h.c_nchunks = spmm_nchunks(short_entries_csr, spmm_chunk_entries(short_entries_csr, f));
  h.n_waves = NWT4; h.n_long_entries = stream_len;   // padded length of the sweep streams
  h.n_multi_rows = tot.multi_rows; h.n_multi_pieces = tot.multi_pieces;
  h.n_slabs = (int32_t)S; h.slab_width = (int32_t)width;
  h.groups = (int32_t)R;
  h.n_intervals = (int32_t)NI; h.sync_slabs = (int32_t)sync_slabs;
  h.sync_timeout_ticks = (opt.sync_timeout_us > 0 ? opt.sync_timeout_us : 200) * 100;
  h.sync_test_extra = opt.sync_test_extra > 0 ? opt.sync_test_extra : 0;
  h.slots = (int32_t)slots;
  h.barriers = opt.barriers == 1 && sync_slabs > 0 ? 1 : 0;
  h.pace_ps_per_step = sync_slabs > 0 && !h.barriers ? opt.pace_ps_per_step : 0;
  h.max_slab = narrow_slabs && R == 2 ? 128 : 256;
  h.col_slab = col_groups ? 64 : 0;
  h.launch_waves = col_groups ? (int32_t)(2 * resident_waves) : 0;
  h.fused_waves = local ? h.launch_waves / 2 : 0;
  out->reuse = (float)reuse;
  out->long_waves = (int32_t)NW4;
  out->run_blocks = local && NI == 1 ? (int32_t)std::min<int64_t>(resident_waves / 4, 1 << 20) : 0;
  // Rows of a generation from which runs pay (sweep_run): 1.3 times the rows of a neighbourhood, three times where the columns
  // go along with the rows, since the runs then begin in different slabs.  us without and with runs: 16 communities, 1 M of 42
  // (62 k rows) f = 64, 128, 256 (131 k rows a generation) 1074, 1803, 3498 and 802, 1572, 3274; 300 k of 20 f = 64, 128, 256
  // 183, 351, 702 and 157, 310, 589; 100 k of 42 f = 32, 100, 256 44, 179, 420 and 37, 111, 238; a layer 64 to 64 1084 and 893,
  // 200 k of 50, 128 to 128 489 and 402; of 125 k rows 1772, 3414, 7041 and 1773, 3416, 7036, the layer 64 to 64 2125 and 2174.
  // Columns within 3000 of the diagonal, 500 k of 30, f = 32, 64, 128 154, 292, 649 and 107, 205, 486; within 20000, 1 M of 24,
  // f = 32 (131 k rows for 40 k) 249 and 237, but f = 64, 128 551, 1180 and 609, 1285; within 50000, 1 M of 40, f = 64 932 and 1125.
  out->run_rows = (float)((tot.slide >= 600 ? 3.0 : 1.3) * span * (double)m / (double)k);
  // Sums of eight groups by the entries a segment has on average, as many of a row's as lie in one of the slabs that it
  // chooses from.  At 32 columns plain of short ones, two from 6 on, between the kernel's widths, which nonzero splitting added
  // as a tree, two at least; folded from 36 on, without locality with the two.  Error against 64 bits plain, with two
  // sums, folded, e-8: random columns, 300 k of 20 (1.3 a segment) 7.17, 7.34, 7.34, of 60 (3.8) 8.69, 8.81, 8.81, 200 k of 60
  // (7.5) 7.84, 7.57, 7.57; communities, 500 k of 16 7.02, 6.02, 6.02, of 32 10.2, 6.92, 6.91, of 42 11.7, 7.42, 7.16, 150 k of
  // 110 18.5, 9.47, 8.42; rows within 3000 of the diagonal, of 30 9.72, 6.43, 6.52.  Folding takes random columns, 200 k of 120, 150 k of 200
  // from 248, 291 to 241, 285 us, power-law matrices, as near every way, 500 k of 30, take 199 plain, 207, 212.
  const double segment = (double)nnz / (double)m / std::max(1.0, (double)S * span / (double)k);
  out->narrow_sums = segment >= 36.0 || (segment >= 6.0 && !local) ? 2 : (segment >= 6.0 ? 1 : 0);
  // Turns (TurnTaking; column groups have them always, one row per load up to 128 columns by the size of B, sweep_launch).  us
  // without and with:
  // Where the order of the rows carries locality not if the columns that neighbouring rows choose from are few megabytes of
  // B, which the L2s hold for all that are near each other in their streams: 16 communities, two groups, 200 k of 50 (6 MB at
  // 128 columns) f = 72, 96, 128 336, 370, 501 and 354, 388, 513, 300 k of 24 264, 314, 401 and 275, 326, 425, 500 k of 42 f =
  // 72, 100 784, 1010 and 807, 992, 700 k of 60 f = 100, 128 (25 MB) 2244, 2428 and 2031, 2377; four, 500 k of 42 f = 36, 48, 64
  // (9 MB) 400, 462, 548 and 438, 491, 561, 1 M of 40 f = 48 (13 MB) 1003, 991; eight, f = 32, 500 k of 42 249, 268, 700 k of 60
  // 503, 513, but 2 M of 35 (18 MB) 1066, 1040 and 150 k of 110 136, 123; four floats a lane only short rows, f = 160, 200,
  // 300 k of 24 516, 714 and 531, 738, 500 k of 16 (22 MB) 713, 960 and 748, 997, of 42 1515, 2036 and 1453, 1874, 1 M of 24
  // (45 MB) 1890, 2661 and 1797, 2506, 700 k of 20 (31, 39 MB) 1112, 1557 and 1071, 1436.  Rows within 3000 of the diagonal,
  // 300 k of 60, f = 32, 48, 96 184, 281, 577 and 205, 305, 621, 500 k of 30, f = 200 1343 and 1257; within 20000, 500 k of 24,
  // f = 128, 160 582, 805 and 645, 908.
  // In the layer with two groups not with locality at any size: 128 to 128 in fp32 200 k of 50 507, 558, 500 k of 42 1126,
  // 1185, 700 k of 20 940, 1010, of 60 (25 MB) 2392, 2386.
  // With hubs and eight groups where resident rows use a row of B often, f = 20, 32: 300 k of 200 566, 535 and 539, 510, 233 k
  // of 489 961, 930 and 934, 904, but 300 k of 30 (1.6 uses) 140, 122 and 143, 125, 1.5 M of 51 930, 824 and 976, 874; with four
  // floats a lane not at 160 and 192 columns, whose rows are whole lines, if they do and rows are not long: 60 k of 200 366, 588
  // and 396, 609, 100 k of 100 316, 494 and 338, 509, 233 k of 100 790, 1100 and 796, 1132, but of 489 f = 192 5032, 4801, 1 M of
  // 50 (0.8 uses) 2195, 2674 and 2116, 2664; f = 200 in all of them 2 to 20 % faster with.
  const double near = span * (double)f * 4.0;
  bool turns = true;
  if (local && !col_groups) {
    if (R > 1) turns = near >= 12e6 || (R == 8 && nnz >= 80 * m);
    else if (f > 128) turns = near >= 28e6 || nnz >= 28 * m;
  } else if (hubs && R == 8) {
    turns = reuse >= 4.0;
  } else if (hubs && R == 1 && f > 128 && f <= 192 && (f & 31) == 0) {
    turns = reuse < 2.0 || nnz >= 300 * m;
  }
  out->turns = turns;
  out->layer_turns = R == 2 ? !local : turns;
  out->mean_steps = rec.scan.mean_steps;
  out->max_steps = rec.scan.max_steps;
  out->use_sweep = true;
  return SAGNN_OK;
}

uint64_t spmm_next_generation() { return g_generation.fetch_add(1); }

namespace {
// workgroups of a kernel that are resident at once on the whole device, for the cohort size of
// the interval barriers: CUs x workgroups per CU as the runtime reports them for this kernel
// and its LDS size, rounded down to a multiple of 8 (one share per XCD).  0 if unknown.
int resident_workgroups(const void* kern, size_t lds) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds) != hipSuccess) return 0;
  // the runtime's figure is too high where the LDS is what limits (see lds_resident_workgroups):
  // assuming too few resident workgroups only makes a cohort smaller, assuming too many would
  // make every barrier run into its time limit
  const int by_lds = lds_resident_workgroups(lds);
  if (per_cu > by_lds) per_cu = by_lds;
  const int64_t n = (int64_t)cus * per_cu / 8 * 8;
  return n > 0 && n < (1 << 30) ? (int)n : 0;
}
}  // namespace

namespace {
// Strides of 32, 64 and 128 steps on three matrices in turn: 233 k vertices f = 128 (119 MB) 1992, 2057, 2101 us; 1 M f = 64
// (256 MB) 710, 716, 711, f = 128 1320, 1329, 1299; 1.2 M f = 128 1740, 1751, 1765; 2.45 M f = 64 (627 MB) 2230, 2249, 2156,
// f = 128 4155, 4240, 4127.
int64_t operand_bytes(uint32_t kmax, int32_t fw) { return ((int64_t)kmax + 1) * fw * 4; }
int32_t turn_steps(uint32_t kmax, int32_t fw) { return operand_bytes(kmax, fw) > (256ll << 20) ? 128 : 32; }

// Workgroups that are shared out among the XCDs in runs (run_block): those of two generations, where the order of the rows
// carries locality and one generation has the rows of more than one neighbourhood (run_rows); otherwise all XCDs want the same
// rows of B in any case, and what one has fetched the others read from the memory-side cache.  (With one and four generations
// 1 M of 42 in communities, f = 64 519 and 531 for 533 us, 500 k, f = 256 2052 and 1939 for 1971.)  Above 128 columns from one
// neighbourhood on, 500 k of 42 (31 k rows), f = 256 product 2146, 1975, bfloat16 layer 2190, 1846; of 125 k the fp32 layer
// 11456, 11775.  The layer holds the whole width in the LDS where the product goes in column groups.
int32_t sweep_run(const SpmmHostDesc& d, int32_t fw, bool layer) {
  if (d.run_blocks < 8) return 0;
  const float rows = (float)d.run_blocks * 4 * kSweepSlots * (layer && d.col_slab > 0 ? (float)d.col_slab / (float)fw : 1.f);
  return rows >= d.run_rows / (fw > 128 ? 1.3f : 1.f) ? 2 * d.run_blocks / 8 * 8 : 0;
}
}  // namespace

namespace {
// lane-group kernels: fuse = 0 product, 1 / 2 / 3 layer form with fp32 / bfloat16 / three-term operands
template <int V, int R, bool BUF, bool AHEAD>
auto group_kernel_of(int fuse) {
  if (fuse == 1) return &spmm_sweep_group_kernel<V, R, 8, BUF, 1, false, AHEAD>;
  if (fuse == 2) return &spmm_sweep_group_kernel<V, R, 8, BUF, 2, false, AHEAD>;
  if (fuse == 3) return &spmm_sweep_group_kernel<V, R, 8, BUF, 3, false, AHEAD>;
  return &spmm_sweep_group_kernel<V, R, 8, BUF, 0, false, AHEAD>;
}
}  // namespace

int sweep_launch(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, const float* B,
                 int64_t ldb, int32_t col0, int32_t fw, uint32_t kmax, float* C, int64_t ldc,
                 int32_t accumulate, int32_t f_total, hipStream_t s, const SweepFusedArgs* fused, int32_t fuse) {
  if (d.n_waves <= 0) return SAGNN_OK;
  const SweepFusedArgs fa = fused ? *fused : SweepFusedArgs{};
  if (!fused) fuse = 0;
  SweepDims sd{};
  sd.n_waves = d.n_waves; sd.ldb = ldb; sd.ldc = ldc; sd.f_total = f_total;
  sd.generation = d.generation; sd.col0 = col0; sd.accumulate = accumulate;
  // bytes of B reachable from B + col0: rows 0..kmax, fw columns each (columns were clamped to
  // kmax when the stream was built)
  sd.b_bytes = 0;
  const bool buf = buffer_addressable(kmax, ldb, fw, &sd.b_bytes);
  sd.row_bytes = (uint32_t)(ldb * 4);
  const unsigned blocks = (unsigned)ceil_div(d.n_waves, 4);
  sd.slots = d.slots > 0 && d.slots <= kSweepSlots ? d.slots : kSweepSlots;
  sd.fw = fw;
  sd.run = sweep_run(d, fw, false);
  sd.long_waves = d.long_waves;
  sd.turn = (fuse != 0 ? d.layer_turns : d.turns) ? turn_steps(kmax, fw) : 0;
  size_t lds = (size_t)4 * sd.slots * (sweep_lds_width(fw) + (fuse != 0 ? kPadRow : 0)) * sizeof(float);
  // (the layer: the targets behind the rows, and no more than five workgroups a CU, which 64 columns would allow: a sixth
  // only drives the others' rows out of the L2, 233 k vertices of 489, 64 to 64 columns 1480 us, with five 1410, 300 k of 60 in
  // communities 460, 447; but in fp32, whose dense part is longest, not where rows are short, 500 k of 18 in communities 319,
  // 334, power-law of 30 314, 337)
  if (fuse != 0) lds = std::max(lds + 4 * kSweepSlots * sizeof(int32_t), (size_t)(fuse == 1 && d.nnz < 40 * d.m ? 0 : 28) << 10);
  auto go = [&](auto kern) -> int {
    if (lds > 48 * 1024)
      SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    // Column groups: two generations of wavefronts a launch, so that those that pass over B together begin together
    // (2 M vertices in communities, f = 256: 8.45 ms in one launch per group, 7.1 so; as good as one generation each).
    const unsigned per = d.col_slab > 0 && fw == d.col_slab && d.launch_waves >= 4 ? (unsigned)(d.launch_waves / 4) : blocks;
    for (unsigned b0 = 0; b0 < blocks; b0 += per) {
      sd.block0 = (int32_t)b0;
      hipLaunchKernelGGL(kern, dim3(blocks - b0 < per ? blocks - b0 : per), dim3(256), lds, s,
                         reinterpret_cast<const uint32_t*>(ws + L.code),
                         reinterpret_cast<const float*>(ws + L.vals),
                         reinterpret_cast<const int32_t*>(ws + L.wave_base),
                         reinterpret_cast<const int32_t*>(ws + L.piece_target),
                         reinterpret_cast<const SpmmWsHeader*>(ws + L.header), B + col0, C + col0,
                         reinterpret_cast<float*>(ws + L.partial), sd);
      SAGNN_LAUNCH_CHECK();
    }
    return SAGNN_OK;
  };
  auto go_perm = [&](auto kern) -> int {   // (at most 32 KB of LDS)
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, s,
                       reinterpret_cast<const uint32_t*>(ws + L.code),
                       reinterpret_cast<const float*>(ws + L.vals),
                       reinterpret_cast<const int32_t*>(ws + L.wave_base),
                       reinterpret_cast<const int32_t*>(ws + L.piece_target),
                       reinterpret_cast<const SpmmWsHeader*>(ws + L.header), B + col0, C + col0,
                       reinterpret_cast<float*>(ws + L.partial),
                       reinterpret_cast<const int32_t*>(ws + L.sync_off), sd);
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  };
  // lane-group kernels: walk the stream interval by interval, with a barrier of the XCD's
  // resident workgroups in between when the schedule was laid out for it
  auto go_group = [&](auto kern) -> int {
    if (lds > 48 * 1024)
      SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    uint32_t* barrier = reinterpret_cast<uint32_t*>(ws + L.barrier);
    sd.n_intervals = d.n_intervals > 0 ? d.n_intervals : 1;
    sd.sync_timeout_ticks = d.sync_timeout_ticks;
    sd.sync_test_extra = d.sync_test_extra;
    sd.wg_per_cohort = 0;
    sd.pace_ticks = d.barriers ? 0.f : (float)d.pace_ps_per_step * 1e-4f;    // ps -> 10 ns ticks
    if (d.barriers && d.sync_slabs > 0 && sd.n_intervals > 1 && (d.n_waves & 3) == 0) {
      const int wpc = resident_workgroups(reinterpret_cast<const void*>(kern), lds);
      const int64_t cohorts = wpc > 0 ? ceil_div((int64_t)blocks, wpc) : 0;
      if (wpc >= 8 && cohorts * 8 * sd.n_intervals <= kSweepBarrierSlots) {
        sd.wg_per_cohort = wpc;
        const int n_ctr = (int)(cohorts * 8 * sd.n_intervals);
        hipLaunchKernelGGL(sweep_barrier_clear_kernel, dim3((unsigned)ceil_div(n_ctr, 256)), dim3(256), 0, s,
                           barrier, n_ctr);
        SAGNN_LAUNCH_CHECK();
      }
    }
    if (sd.wg_per_cohort == 0) sd.n_intervals = sd.n_intervals > 1 ? -sd.n_intervals : sd.n_intervals;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, s,
                       reinterpret_cast<const uint32_t*>(ws + L.code),
                       reinterpret_cast<const float*>(ws + L.vals),
                       reinterpret_cast<const int32_t*>(ws + L.wave_base),
                       reinterpret_cast<const int32_t*>(ws + L.piece_target),
                       reinterpret_cast<const SpmmWsHeader*>(ws + L.header), B + col0, C + col0,
                       reinterpret_cast<float*>(ws + L.partial),
                       reinterpret_cast<const int32_t*>(ws + L.sync_off), barrier,
                       reinterpret_cast<const float*>(ws + L.sched), sd, fa);
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  };
  if (fuse != 0 && d.groups != 2 && d.groups != 4) return SAGNN_EINVAL;   // (groups == 1: sweep_launch_fused)
  if (fw <= 0 || (fw & 3)) return SAGNN_EINVAL;
  if (d.groups == 16) {  // four lanes per row
    if (fw > 16) return SAGNN_EINVAL;
#define SAGNN_SIXTEEN(ODD_) \
  (buf ? go_perm(spmm_sweep_perm_kernel<16, true, ODD_, false, true, true>) : go_perm(spmm_sweep_perm_kernel<16, false, ODD_, false, true, true>))
    return fw == 16 ? SAGNN_SIXTEEN(false) : SAGNN_SIXTEEN(true);
#undef SAGNN_SIXTEEN
  }
  if (d.groups == 8) {   // eight lanes per row
    if (fw > 32) return SAGNN_EINVAL;
#define SAGNN_EIGHT(ODD_, TURN_, TWO_, FOLD_)                                      \
  (buf ? go_perm(spmm_sweep_perm_kernel<8, true, ODD_, TURN_, TWO_, FOLD_>) \
       : go_perm(spmm_sweep_perm_kernel<8, false, ODD_, TURN_, TWO_, FOLD_>))
    if (d.narrow_sums == 2 && fw == 32) return d.turns ? SAGNN_EIGHT(false, true, true, true) : SAGNN_EIGHT(false, false, true, true);
    if (d.narrow_sums == 2) return d.turns ? SAGNN_EIGHT(true, true, true, true) : SAGNN_EIGHT(true, false, true, true);
    if (fw != 32) return d.turns ? SAGNN_EIGHT(true, true, true, false) : SAGNN_EIGHT(true, false, true, false);
    if (d.narrow_sums == 1) return d.turns ? SAGNN_EIGHT(false, true, true, false) : SAGNN_EIGHT(false, false, true, false);
    return d.turns ? SAGNN_EIGHT(false, true, false, false) : SAGNN_EIGHT(false, false, false, false);
#undef SAGNN_EIGHT
  }
  if (d.groups == 2) {   // half a wavefront per row
    // Words ahead (see the kernel) up to a size of the operand, whatever its addressing, in the product and in the layer:
    // beyond it wavefronts that run ahead only cost misses.  us with and without, products of power-law matrices at 128
    // columns: 300 k vertices of 30 278, 320, 600 k of 51 849, 892, 1.1 M of 51 (563 MB) 1639, 1704, 1.2 M of 51 (614 MB) 1785,
    // 1873, 1.3 M of 30, 51, 80 (666 MB) 1392, 2148, 3279 and 1386, 2101, 2979, 1.6 M of 51 2880, 2729, 2.1 M 4109, 3521, 2.45 M
    // 4179, 4135, of 30 3303, 3050, 3.3 M of 45 6927, 5538, 5 M of 40 10328, 8921, 9 M of 30 (4.6 GB) 16867, 15440 (at the line
    // itself either may win: 1.24 M of 20, 42 1087, 1580 and 1042, 1652, 1.29 M of 42 1673, 1767, 1.32 M 1997, 1862); its layer
    // in fp32 1.2 M of 51 2173, 2293, 1.6 M 3315, 3201, 2.45 M 4833, 4740.  Between the kernels' own widths, whose rows begin
    // inside lines, from the memory-side cache's size on: 233 k of 489, f = 100 1975, 2286, 600 k of 60 (240 MB) 970, 1005, 1 M
    // of 51, f = 72 (288 MB) 1345, 1205, 2 M of 51, f = 72, 100, 112 3604, 3942, 3934 and 2637, 3739, 3739, 2.45 M of 40, f = 96
    // 3261, 2686; and where rows are whole lines (96), in smaller and shorter ones, with and without: 100 k of 60 152, 172, 200 k
    // of 30, 120 164, 436 and 171, 452, 300 k of 70 408, 425, 400 k of 30 (154 MB) 301, 322, but of 70, 120 664, 1084 and 576,
    // 884, 233 k of 200 868, 766, 500 k of 30, 60 (192 MB) 442, 778 and 397, 647.
    const int64_t b = operand_bytes(kmax, fw);
    if (fw == 128) {
      if (b <= (600ll << 20)) return buf ? go_group(group_kernel_of<4, 2, true, true>(fuse)) : go_group(group_kernel_of<4, 2, false, true>(fuse));
      return buf ? go_group(group_kernel_of<4, 2, true, false>(fuse)) : go_group(group_kernel_of<4, 2, false, false>(fuse));
    }
    if (fw == 64) return buf ? go_group(group_kernel_of<2, 2, true, true>(fuse)) : go_group(group_kernel_of<2, 2, false, true>(fuse));
    if (fw > 128 || fuse) return SAGNN_EINVAL;
    // (two sums where nonzero splitting would be the alternative, with its tree: communities, 30 k vertices of 60, f = 100
    // 7.7e-8 from 64 bits by the tree, 13.8e-8 by one sum; elsewhere they cost up to 2 %)
    if (d.apart)
      return buf ? go_group(&spmm_sweep_group_kernel<4, 2, 8, true, 0, true, true, true>)
                 : go_group(&spmm_sweep_group_kernel<4, 2, 8, false, 0, true, true, true>);
    if ((fw & 31) == 0 ? b <= (160ll << 20) && d.nnz <= 25000000 : b <= (256ll << 20))
      return buf ? go_group(&spmm_sweep_group_kernel<4, 2, 8, true, 0, true>) : go_group(&spmm_sweep_group_kernel<4, 2, 8, false, 0, true>);
    return buf ? go_group(&spmm_sweep_group_kernel<4, 2, 8, true, 0, true, false>)
               : go_group(&spmm_sweep_group_kernel<4, 2, 8, false, 0, true, false>);
  }
  if (d.groups == 4) {   // a quarter wavefront per row
    if (fw == 64) return buf ? go_group(group_kernel_of<4, 4, true, true>(fuse)) : go_group(group_kernel_of<4, 4, false, true>(fuse));
    if (fw > 64 || fuse) return SAGNN_EINVAL;
    return buf ? go_group(&spmm_sweep_group_kernel<4, 4, 8, true, 0, true>) : go_group(&spmm_sweep_group_kernel<4, 4, 8, false, 0, true>);
  }
  if (fw > 256) return SAGNN_EINVAL;
  // At up to 128 columns, where one row per load is for matrices whose rows of B are hardly used twice (but for column
  // groups), turns pay by the size of the operand, whatever its width.  us without and with, over the line: a rank's rows
  // f = 64 638, 618 (1.25 GB), f = 96 753, 747 (1.5), f = 112 909, 888 (1.7), 1315, 1265 (2.2), f = 128 548, 545 (1.3),
  // 588, 584 (1.4), 792, 758 (1.6), 927, 902 (2.0), 1351, 1288 (2.5), 1553, 1502 (3.4); under it: f = 128 485, 493 (1.03),
  // f = 96 446, 453 (0.95), f = 128 370, 371 (0.7), random columns of 9 to 19, f = 128 1037, 1065 (0.5), 1316, 1337 (0.6),
  // f = 64 and 96 the same.
  const bool turns = d.col_slab > 0 || d.f > 128 || operand_bytes(kmax, fw) > (1100ll << 20);
#define SAGNN_ONE(FPL_, ODD_, TURN_) \
  (buf ? go(spmm_sweep_kernel<FPL_, 8, true, ODD_, TURN_>) : go(spmm_sweep_kernel<FPL_, 8, false, ODD_, TURN_>))
  if (fw == 256) return SAGNN_ONE(4, false, true);
  if (fw == 128) return turns ? SAGNN_ONE(2, false, true) : SAGNN_ONE(2, false, false);
  if (fw == 64) return turns ? SAGNN_ONE(1, false, true) : SAGNN_ONE(1, false, false);
  if (fw > 128) return SAGNN_ONE(4, true, true);
  if (fw > 64) return turns ? SAGNN_ONE(2, true, true) : SAGNN_ONE(2, true, false);
  return turns ? SAGNN_ONE(1, true, true) : SAGNN_ONE(1, true, false);
#undef SAGNN_ONE
}

int sweep_launch_fused(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, const float* B, int64_t ldb,
                       int32_t f_in, uint32_t kmax, const SweepFusedArgs& fa, int32_t mode, hipStream_t s) {
  if (d.n_waves <= 0 || (d.n_waves & 3) || d.slots != kSweepSlots) return SAGNN_EINVAL;
  if (mode < 0 || mode > 2) return SAGNN_EINVAL;
  if (!(f_in == 64 || f_in == 128 || f_in == 256) || fa.f_out <= 0 || fa.f_out > 256 || !fa.W) return SAGNN_EINVAL;
  if (d.groups == 2 || d.groups == 4) {
    // lane-group schedules: the same kernels as the product, with the dense transform compiled in
    SweepFusedArgs fg = fa;
    fg.Wp = nullptr;
    if (mode != 0) {
      const int32_t NB = (fa.f_out + 31) / 32 * 32;
      __bf16* wp = reinterpret_cast<__bf16*>(ws + L.wpack);
      hipLaunchKernelGGL(sweep_pack_w_kernel, dim3((unsigned)ceil_div((int64_t)(f_in / 8) * NB, 256)), dim3(256), 0, s,
                         fa.W, f_in, fa.f_out, NB, wp, mode == 2 ? 3 : 1);
      SAGNN_LAUNCH_CHECK();
      fg.Wp = wp;
    }
    return sweep_launch(d, L, ws, B, ldb, 0, f_in, kmax, nullptr, f_in, 0, f_in, s, &fg, mode + 1);
  }
  if (d.groups != 1) return SAGNN_EINVAL;
  SweepDims sd{};
  sd.n_waves = d.n_waves; sd.ldb = ldb; sd.ldc = f_in; sd.f_total = f_in;
  sd.generation = d.generation; sd.col0 = 0; sd.accumulate = 0; sd.slots = kSweepSlots;
  sd.turn = turn_steps(kmax, f_in);
  sd.run = sweep_run(d, f_in, true);
  sd.b_bytes = 0;
  const bool buf = buffer_addressable(kmax, ldb, f_in, &sd.b_bytes);
  sd.row_bytes = (uint32_t)(ldb * 4);
  const unsigned blocks = (unsigned)(d.n_waves / 4);
  const size_t lds = (size_t)4 * kSweepSlots * (f_in + kPadRow + 1) * sizeof(float);   // (rows and their targets)
  SweepFusedArgs fb = fa;
  fb.Wp = nullptr;
  if (mode != 0) {
    const int32_t NB = (fa.f_out + 31) / 32 * 32;
    __bf16* wp = reinterpret_cast<__bf16*>(ws + L.wpack);
    hipLaunchKernelGGL(sweep_pack_w_kernel, dim3((unsigned)ceil_div((int64_t)(f_in / 8) * NB, 256)), dim3(256), 0, s,
                       fa.W, f_in, fa.f_out, NB, wp, mode == 2 ? 3 : 1);
    SAGNN_LAUNCH_CHECK();
    fb.Wp = wp;
  }
  // At 128 columns turns pay in the layer where rows of B are used often by rows that are resident together, and those are
  // not short.  us without and with, random columns, 200 k vertices of 30 (2.5 uses) to 40 columns 404, 400, 200 k of 60 (4.9)
  // 709, 663, 100 k of 40 (6.6) 205, 188, 350 k of 60 (2.8) to 128 1369, 1342; 300 k of 20 (1.1) to 128 526, 545, 275 k of 40
  // (2.4) 791, 804, 150 k of 24 (2.6) 311, 318; 1 M of 15 1341, 1381; communities, 1.6 M of 31 in bfloat16 3069, 2906, 700 k of
  // 21 to 40 1024, 995, but to 128 1061, 1110.  Over 1100 MB as in the product.
  const bool brief = mode != 0 || fa.f_out <= 64;
  const bool turns = (d.reuse >= 2.4f && (d.nnz >= 28 * d.m || (brief && d.fused_waves > 0))) || operand_bytes(kmax, f_in) > (1100ll << 20);
  auto go = [&](auto kern) -> int {
    if (lds > 48 * 1024)
      SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    // (two generations a launch for column groups, as sweep_launch, but at 128 columns only, where the order of the rows
    // carries locality and the dense part is not long: 1.6 M vertices of 40 in communities to 40 columns in fp32 3950 -> 3718
    // us, to 128 in bfloat16 4042 -> 3795, in fp32 4086 -> 4132; random columns, 500 k of 24, 976 -> 1096.  At 64 and 256 the
    // dense parts of workgroups that end together are left without gathers beside them: 803 -> 822, 3862 -> 4120.)
    const unsigned per = f_in == 128 && brief && d.fused_waves >= 4 ? (unsigned)(d.fused_waves / 4) : blocks;
    for (unsigned b0 = 0; b0 < blocks; b0 += per) {
      sd.block0 = (int32_t)b0;
      hipLaunchKernelGGL(kern, dim3(blocks - b0 < per ? blocks - b0 : per), dim3(256), lds, s,
                         reinterpret_cast<const uint32_t*>(ws + L.code),
                         reinterpret_cast<const float*>(ws + L.vals),
                         reinterpret_cast<const int32_t*>(ws + L.wave_base),
                         reinterpret_cast<const int32_t*>(ws + L.piece_target),
                         reinterpret_cast<const SpmmWsHeader*>(ws + L.header), B,
                         reinterpret_cast<float*>(ws + L.partial), sd, fb);
      SAGNN_LAUNCH_CHECK();
    }
    return SAGNN_OK;
  };
#define SAGNN_SWF(FPL_, TURN_)                                                                               \
  (mode == 2 ? (buf ? go(spmm_sweep_fused_kernel<FPL_, 8, true, 2, TURN_>) : go(spmm_sweep_fused_kernel<FPL_, 8, false, 2, TURN_>))   \
   : mode == 1 ? (buf ? go(spmm_sweep_fused_kernel<FPL_, 8, true, 1, TURN_>) : go(spmm_sweep_fused_kernel<FPL_, 8, false, 1, TURN_>)) \
               : (buf ? go(spmm_sweep_fused_kernel<FPL_, 8, true, 0, TURN_>) : go(spmm_sweep_fused_kernel<FPL_, 8, false, 0, TURN_>)))
  if (f_in == 256 && mode == 0) {   // (see Targets)
    const int64_t b = operand_bytes(kmax, f_in);
    if (d.reuse >= 2.f && (b <= (256ll << 20) || (b <= (768ll << 20) && d.nnz >= 36 * d.m)))
      return buf ? go(spmm_sweep_fused_kernel<4, 8, true, 0, false, TARGETS_BEFORE>) : go(spmm_sweep_fused_kernel<4, 8, false, 0, false, TARGETS_BEFORE>);
    return buf ? go(spmm_sweep_fused_kernel<4, 8, true, 0, false, TARGETS_BEHIND>) : go(spmm_sweep_fused_kernel<4, 8, false, 0, false, TARGETS_BEHIND>);
  }
  if (f_in == 256) return SAGNN_SWF(4, false);   // (only two wavefronts share a SIMD)
  if (f_in == 128) return turns ? SAGNN_SWF(2, true) : SAGNN_SWF(2, false);
  return SAGNN_SWF(1, true);
#undef SAGNN_SWF
}

int sweep_combine(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, float* C, int64_t ldc,
                  int32_t f_total, int32_t accumulate, hipStream_t s) {
  if (d.n_multi_rows <= 0) return SAGNN_OK;
  hipLaunchKernelGGL(sweep_combine_kernel, dim3((unsigned)ceil_div(d.n_multi_rows, 4)), dim3(256), 0, s,
                     reinterpret_cast<const int32_t*>(ws + L.multi_row),
                     reinterpret_cast<const int32_t*>(ws + L.multi_first),
                     reinterpret_cast<const float*>(ws + L.partial),
                     reinterpret_cast<const SpmmWsHeader*>(ws + L.header), d.generation, d.n_multi_rows,
                     C, ldc, f_total, accumulate);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

}  // namespace sagnn
