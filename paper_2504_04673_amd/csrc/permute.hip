// Locality reordering of a row block's graph: symmetric permutation of a square CSR matrix by
// partition labels (Sec. 5 and Sec. 6.1: the vertices are renumbered so that every part owns a
// contiguous block of rows; A is permuted symmetrically and the rows of H follow).
//
//   perm / inv from labels   stable sort of the vertices by label (the order inside a part is
//                            the original order), done with the library's stable radix sort:
//                            the labels are the "column ids" of an n x n_parts pattern with one
//                            entry per row, whose transpose lists the vertices of every part
//   B = P A P^T              B[inv[r], inv[c]] = A[r, c].  Where every row has at most 512 entries
//                            a row of A becomes a row of B by itself: a wavefront relabels its
//                            columns, ranks them in registers and writes them to the row's new
//                            place.  With longer rows: two stable transposes with a
//                            relabelling before each: relabel columns, transpose (rows are now
//                            new column ids, ascending, entries by old row), relabel those old
//                            row ids, transpose again (rows are new row ids, entries ascending
//                            by new column id, repeated entries in stored order).  Unique result.
// The dense side is moved with spmm_pack_rows: H_new = H[perm, :], Z_old = Z_new[inv, :].
// Integer work only: bit-exact.
#include "common.h"

namespace sagnn {
namespace {

constexpr int kThreads = 256;

inline dim3 grid_for(int64_t items) {
  int64_t b = ceil_div(items > 0 ? items : 1, kThreads);
  if (b > 256 * 32) b = 256 * 32;
  return dim3((unsigned)b);
}

// out[i] = map[in[i]]; an id outside [0, n) sets err[0] and maps to 0
__global__ __launch_bounds__(kThreads) void relabel_kernel(const int32_t* __restrict__ in, int64_t cnt,
                                                           const int32_t* __restrict__ map, int64_t n,
                                                           int32_t* __restrict__ out,
                                                           int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < cnt; i += stride) {
    const int32_t c = in[i];
    if (c < 0 || c >= n) {
      err[0] = 1;
      out[i] = 0;
    } else {
      out[i] = map[c];
    }
  }
}

// perm[i] = order[i], inv[order[i]] = i
__global__ __launch_bounds__(kThreads) void order_kernel(const uint32_t* __restrict__ order, int64_t n,
                                                         int32_t* __restrict__ perm, int32_t* __restrict__ inv) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
    const int32_t p = (int32_t)order[i];   // a payload of the sort: always in [0, n)
    perm[i] = p;
    inv[p] = (int32_t)i;
  }
}

// Checks of the two maps, the row lengths of B, and the inverse map: seen[p] = 1 + the row of A that becomes row p.
// err[1] = 1 unless map is a permutation of [0, n) (every value in range and seen exactly once); err[2] = 1 if the rows of A cannot be permuted one by one (a row longer than
// kRowSortMax, or rowptr is no CSR row pointer).
constexpr int kRowSortMax = 512;
__global__ __launch_bounds__(kThreads) void check_perm_kernel(const int32_t* __restrict__ map,
                                                              const int32_t* __restrict__ rowptr, int64_t n,
                                                              int64_t nnz, int32_t* __restrict__ seen,
                                                              int32_t* __restrict__ len, int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
    const int32_t p = map[i];
    const int64_t b = rowptr[i], e = rowptr[i + 1];
    if (b < 0 || e < b || e > nnz || e - b > kRowSortMax || (i == 0 && b != 0) || (i == n - 1 && e != nnz)) err[2] = 1;
    if (p < 0 || p >= n) {
      err[1] = 1;
    } else {
      if (atomicExch(&seen[p], (int32_t)i + 1) != 0) err[1] = 1;
      len[p] = (int32_t)(e - b);
    }
  }
}

// Exclusive scan of the n row lengths into rowptr[0..n]: tiles of 2048, their sums, the sums added back.
constexpr int kScanTile = 8 * kThreads;
__device__ __forceinline__ int32_t scan_block(int32_t v, int32_t* total) {
  __shared__ int32_t wsum[kThreads / 64];
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
  for (int w = 0; w < kThreads / 64; ++w) {
    if (w < wave) before += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return before + inc - v;
}

__global__ __launch_bounds__(kThreads) void scan_tiles_kernel(const int32_t* __restrict__ len, int64_t n,
                                                              int32_t* __restrict__ rowptr,
                                                              int32_t* __restrict__ tilesum) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
  int32_t x[8], sum = 0, tot;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = i0 + i < n ? len[i0 + i] : 0;
    sum += x[i];
  }
  int32_t run = scan_block(sum, &tot);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (i0 + i < n) rowptr[i0 + i] = run;
    run += x[i];
  }
  if (threadIdx.x == 0) tilesum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kThreads) void scan_sums_kernel(int32_t* __restrict__ tilesum, int64_t ntiles) {
  int32_t carry = 0;
  for (int64_t base = 0; base < ntiles; base += kThreads) {
    const int64_t i = base + threadIdx.x;
    int32_t tot;
    const int32_t ex = scan_block(i < ntiles ? tilesum[i] : 0, &tot);
    if (i < ntiles) tilesum[i] = carry + ex;
    carry += tot;
  }
}

// SUMMED: tilesum has been scanned.  Up to kFewSums tiles every workgroup adds up the tiles before its own by itself instead:
// they are in cache, and the scan is one of three launches.
constexpr int64_t kFewSums = 1024;
template <bool SUMMED>
__global__ __launch_bounds__(kThreads) void scan_add_kernel(const int32_t* __restrict__ tilesum, int64_t n, int64_t nnz,
                                                            int32_t* __restrict__ rowptr) {
  int32_t before = 0;
  if constexpr (SUMMED) {
    before = tilesum[blockIdx.x];
  } else {
    int32_t part = 0;
    for (int64_t t = threadIdx.x; t < blockIdx.x; t += kThreads) part += tilesum[t];
    scan_block(part, &before);
  }
  for (int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x; i < ((int64_t)blockIdx.x + 1) * kScanTile && i <= n; i += kThreads) {
    if (i < n) rowptr[i] += before;
    else rowptr[n] = (int32_t)nnz;
  }
}

// Ascending bitonic sort over the 64 lanes.  Partners at 1, 2, 4 and 8 lanes come by DPP (two steps for 4), at 16 and 32
// by the row swaps, so no step goes through the LDS: about 75 instructions, where counting the smaller keys takes three
// for every entry of the row.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int J>
__device__ __forceinline__ void sort_step(uint32_t& x, bool keep_smaller) {
  uint32_t lo, hi;
  if constexpr (J <= 8) {
    uint32_t y;
    if constexpr (J == 1) y = dpp_move<0xB1>(x);                          // quad_perm:[1,0,3,2]
    else if constexpr (J == 2) y = dpp_move<0x4E>(x);                     // quad_perm:[2,3,0,1]
    else if constexpr (J == 4) y = dpp_move<0x1B>(dpp_move<0x141>(x));    // lane 7 - i of eight, then 3 - i of four
    else y = dpp_move<0x128>(x);                                          // row_ror:8
    lo = x < y ? x : y;
    hi = x < y ? y : x;
  } else {
    // both rows (halves) of a pair get the keys of the lower one in `a`, of the upper one in `b`
    const auto ab = J == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false) : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const uint32_t a = ab[0], b = ab[1];
    lo = a < b ? a : b;
    hi = a < b ? b : a;
  }
  x = keep_smaller ? lo : hi;
}
template <int K, int J>
__device__ __forceinline__ void sort_merge(uint32_t& x, int lane) {
  if constexpr (J > 0) {
    sort_step<J>(x, ((lane & J) == 0) == ((lane & K) == 0));
    sort_merge<K, J / 2>(x, lane);
  }
}
__device__ __forceinline__ void sort_lanes(uint32_t& x, int lane) {
  sort_merge<2, 1>(x, lane);
  sort_merge<4, 2>(x, lane);
  sort_merge<8, 4>(x, lane);
  sort_merge<16, 8>(x, lane);
  sort_merge<32, 16>(x, lane);
  sort_merge<64, 32>(x, lane);
}

// Rows of B from rows of A, in the order of B: rows that lie together are written together (rows of A are read where
// they are; the other way round every row's ends were partly written lines).  A wavefront relabels a row's columns and
// sorts them (a row of up to 64) or ranks them by counting the smaller ones, equal ones the earlier ones first.  Bound by
// the latency of its dependent loads (old row, row pointer, columns, new ids), so a wavefront has four rows in flight
// while they fit 64 lanes each.  There the key carries the lane in its low bits (n <= 2^26), which makes equal columns
// different and finds the value.  21 M entries in 500 k rows: 300 us by ranks and in the order of A, 265 so, 236 with eight
// wavefronts per SIMD (25 of the registers that rows of 257 to 512 entries would like are spilled there: 20 k rows of 300
// 348 -> 336, 60 k of 200 414 -> 386); in the
// order of A 245.  27 M requests to the L2s, most of them the new ids of random columns, at 85 % of the rate gathers reach.
// Relabelling and sorting the entries twice through memory took 1.4 ms.
// Nothing is done where check_perm_kernel found a reason against it (the host looks afterwards).
template <int K>
__device__ __forceinline__ void permute_row(const int32_t* __restrict__ colidx, const float* __restrict__ val,
                                            const int32_t* __restrict__ inv, int64_t n, int64_t b, int d, int64_t out,
                                            int32_t* __restrict__ colidx_p, float* __restrict__ val_p,
                                            int32_t* __restrict__ err) {
  const int lane = threadIdx.x & 63;
  uint32_t key[K];
  float v[K];
  int rank[K];
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const int i = q * 64 + lane;
    key[q] = 0xFFFFFFFFu;
    v[q] = 0.f;
    rank[q] = 0;
    if (i < d) {
      const int32_t c = colidx[b + i];
      v[q] = val[b + i];
      if (c >= 0 && c < n) key[q] = (uint32_t)inv[c];
      else err[0] = 1;
    }
  }
#pragma unroll
  for (int qj = 0; qj < K; ++qj) {
    const int left = d - qj * 64;
    for (int l = 0; l < (left < 64 ? left : 64); ++l) {
      const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key[qj], l);
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const bool earlier = qj < q || (qj == q && l < lane);
        rank[q] += earlier ? (kj <= key[q]) : (kj < key[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < K; ++q)
    if (q * 64 + lane < d) {
      colidx_p[out + rank[q]] = (int32_t)key[q];
      val_p[out + rank[q]] = v[q];
    }
}

__global__ __launch_bounds__(kThreads, 8) void permute_rows_kernel(const int32_t* __restrict__ rowptr,
                                                                const int32_t* __restrict__ colidx,
                                                                const float* __restrict__ val, int64_t n,
                                                                const int32_t* __restrict__ inv,
                                                                const int32_t* __restrict__ seen,
                                                                const int32_t* __restrict__ rowptr_p,
                                                                int32_t* __restrict__ colidx_p,
                                                                float* __restrict__ val_p, int32_t* __restrict__ err) {
  constexpr int R = 4;
  if (err[1] | err[2]) return;
  const int lane = threadIdx.x & 63;
  const int64_t wave = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6));
  const int64_t p0 = wave * R;
  int64_t b[R], out[R];
  int d[R], longest = 0;
#pragma unroll
  for (int t = 0; t < R; ++t) {
    const int64_t p = p0 + t < n ? p0 + t : n - 1;
    const int64_t r = (int64_t)seen[p] - 1;      // (in [0, n): check_perm_kernel found a permutation)
    b[t] = rowptr[r];
    d[t] = p0 + t < n ? (int)(rowptr[r + 1] - b[t]) : 0;
    longest = d[t] > longest ? d[t] : longest;
    out[t] = rowptr_p[p];
  }
  if (longest <= 64 && n <= (1 << 26)) {
    uint32_t key[R];
    float v[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
      key[t] = 0xFFFFFFC0u | (uint32_t)lane;     // (lanes past the end of a row: behind all keys)
      v[t] = 0.f;
      if (lane < d[t]) {
        const int32_t c = colidx[b[t] + lane];
        v[t] = val[b[t] + lane];
        if (c >= 0 && c < n) key[t] = ((uint32_t)inv[c] << 6) | (uint32_t)lane;
        else err[0] = 1;
      }
    }
#pragma unroll
    for (int t = 0; t < R; ++t) sort_lanes(key[t], lane);
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const float moved = __shfl(v[t], (int)(key[t] & 63u), 64);
      if (lane < d[t]) {
        colidx_p[out[t] + lane] = (int32_t)(key[t] >> 6);
        val_p[out[t] + lane] = moved;
      }
    }
    return;
  }
#pragma unroll 1
  for (int t = 0; t < R; ++t) {
    if (d[t] <= 64) permute_row<1>(colidx, val, inv, n, b[t], d[t], out[t], colidx_p, val_p, err);
    else if (d[t] <= 128) permute_row<2>(colidx, val, inv, n, b[t], d[t], out[t], colidx_p, val_p, err);
    else if (d[t] <= 256) permute_row<4>(colidx, val, inv, n, b[t], d[t], out[t], colidx_p, val_p, err);
    else permute_row<8>(colidx, val, inv, n, b[t], d[t], out[t], colidx_p, val_p, err);
  }
}

__global__ __launch_bounds__(kThreads) void zero_i32_kernel(int32_t* __restrict__ a, int64_t n, int32_t* __restrict__ b, int m) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) a[i] = 0;
  if (blockIdx.x == 0 && (int)threadIdx.x < m) b[threadIdx.x] = 0;
}

struct PermuteWs {
  int32_t *ci_a, *rp_b, *ci_b, *seen, *tilesum, *err;
  float* va_b;
  char* tws;
  size_t tws_bytes, bytes;
};

int carve_permute(void* base, int64_t n, int64_t nnz, PermuteWs* w) {
  if (nnz < 0 || nnz > 0x7FFFFFFFll) return SAGNN_EINVAL;
  const size_t tb = transpose_ws_bytes(nnz);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? static_cast<char*>(base) + off : nullptr;
    off += round_up(bytes > 0 ? bytes : 4, 256);
    return p;
  };
  const size_t e = (size_t)(nnz > 0 ? nnz : 1);
  w->ci_a = reinterpret_cast<int32_t*>(take(4 * e));
  w->rp_b = reinterpret_cast<int32_t*>(take(4 * (size_t)(n + 2)));
  w->ci_b = reinterpret_cast<int32_t*>(take(4 * e));
  w->va_b = reinterpret_cast<float*>(take(4 * e));
  w->seen = reinterpret_cast<int32_t*>(take(4 * (size_t)(n > 0 ? n : 1)));
  w->tilesum = reinterpret_cast<int32_t*>(take(4 * (size_t)(ceil_div(n > 0 ? n : 1, kScanTile) + 1)));
  w->err = reinterpret_cast<int32_t*>(take(16));
  w->tws = take(tb);
  w->tws_bytes = tb;
  w->bytes = off;
  return SAGNN_OK;
}

}  // namespace
}  // namespace sagnn

SAGNN_EXPORT int spmm_permute_workspace_bytes(int64_t n, int64_t nnz, size_t* bytes) {
  using namespace sagnn;
  if (!bytes || n < 0 || nnz < 0 || n > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll) return SAGNN_EINVAL;
  PermuteWs w{};
  // the label sort transposes an n-entry pattern, the matrix permutation an nnz-entry one
  int rc = carve_permute(nullptr, n, nnz > n ? nnz : n, &w);
  if (rc != SAGNN_OK) return rc;
  *bytes = w.bytes;
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_perm_from_labels(const int32_t* d_labels, int64_t n, int32_t n_parts,
                                       int32_t* d_perm, int32_t* d_inv, int64_t* h_part_off,
                                       void* d_ws, size_t ws_bytes, void* stream) {
  using namespace sagnn;
  if (n < 0 || n > 0x7FFFFFFFll || n_parts < 1) return SAGNN_EINVAL;
  if (!d_perm || !d_inv || !h_part_off || !d_ws || (n > 0 && !d_labels)) return SAGNN_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ws) & 255u) return SAGNN_EINVAL;
  PermuteWs w{};
  int rc = carve_permute(d_ws, n, n, &w);
  if (rc != SAGNN_OK) return rc;
  if (ws_bytes < w.bytes) return SAGNN_ECAPACITY;
  hipStream_t s = (hipStream_t)stream;
  if (n_parts > 1024 || (int64_t)n_parts > (n > 0 ? n : 1)) return SAGNN_EINVAL;
  for (int32_t q = 0; q <= n_parts; ++q) h_part_off[q] = 0;
  if (n == 0) return SAGNN_OK;
  // stable sort of the vertices by label; the part offsets come from the sorted labels.  The error flag lies
  // behind the offsets so that one copy brings both to the host.
  const RadixWs rw = carve_radix(w.tws, n);
  int bits = 1;
  while ((1 << bits) < n_parts) ++bits;
  int32_t h[1026];
  auto apart = [&](const int32_t* out) { return out + n <= d_labels || d_labels + n <= out; };
  if (bits <= 8 && apart(d_perm) && apart(d_inv)) {
    // one pass, which writes both orders; the offsets are sums of its totals (500 k labels of 16: sorted pairs, offsets and
    // orders by kernels of their own 26 us, now 18).  Its tiles are written while others still read their labels: an order
    // that takes the labels' place is written behind the sort.
    SAGNN_HIP(hipMemsetAsync(rw.totals + 256, 0, sizeof(int32_t), s));
    rc = radix_order(reinterpret_cast<const uint32_t*>(d_labels), n, bits, rw, d_perm, d_inv, s, n_parts);
    if (rc != SAGNN_OK) return rc;
    SAGNN_HIP(hipMemcpyAsync(h, rw.totals, sizeof(int32_t) * 257, hipMemcpyDeviceToHost, s));
    SAGNN_HIP(hipStreamSynchronize(s));
    if (h[256]) return SAGNN_EFORMAT;   // a label outside [0, n_parts)
    for (int32_t q = 0; q < n_parts; ++q) h_part_off[q + 1] = h_part_off[q] + h[q];
    return SAGNN_OK;
  }
  int32_t* d_off = w.rp_b;
  int32_t* d_err = w.rp_b + n_parts + 1;
  SAGNN_HIP(hipMemsetAsync(d_err, 0, sizeof(int32_t), s));
  int res = 0;
  rc = radix_sort_pairs(reinterpret_cast<const uint32_t*>(d_labels), nullptr, n, bits, rw, s, &res, n_parts, d_err);
  if (rc != SAGNN_OK) return rc;
  rc = launch_sorted_rowptr(rw.keys[res], n, n_parts, d_off, s);
  if (rc != SAGNN_OK) return rc;
  hipLaunchKernelGGL(order_kernel, grid_for(n), dim3(kThreads), 0, s, rw.pay[res], n, d_perm, d_inv);
  SAGNN_LAUNCH_CHECK();
  SAGNN_HIP(hipMemcpyAsync(h, d_off, sizeof(int32_t) * (size_t)(n_parts + 2), hipMemcpyDeviceToHost, s));
  SAGNN_HIP(hipStreamSynchronize(s));
  if (h[n_parts + 1]) return SAGNN_EFORMAT;   // a label outside [0, n_parts)
  for (int32_t q = 0; q <= n_parts; ++q) h_part_off[q] = h[q];
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_permute_symmetric(const int32_t* d_rowptr, const int32_t* d_colidx,
                                            const float* d_val, int64_t n, int64_t nnz,
                                            const int32_t* d_inv, int32_t* d_rowptr_p,
                                            int32_t* d_colidx_p, float* d_val_p, void* d_ws,
                                            size_t ws_bytes, void* stream) {
  using namespace sagnn;
  if (n < 0 || nnz < 0 || n > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll) return SAGNN_EINVAL;
  if (!d_rowptr || !d_rowptr_p || !d_ws || (n > 0 && !d_inv)) return SAGNN_EINVAL;
  if (nnz > 0 && (!d_colidx || !d_val || !d_colidx_p || !d_val_p)) return SAGNN_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ws) & 255u) return SAGNN_EINVAL;
  PermuteWs w{};
  int rc = carve_permute(d_ws, n, nnz, &w);
  if (rc != SAGNN_OK) return rc;
  if (ws_bytes < w.bytes) return SAGNN_ECAPACITY;
  if (n == 0 && nnz > 0) return SAGNN_EFORMAT;   // no column is in range
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(zero_i32_kernel, grid_for(n), dim3(kThreads), 0, s, w.seen, n, w.err, 4);
  SAGNN_LAUNCH_CHECK();
  if (n > 0) {
    hipLaunchKernelGGL(check_perm_kernel, grid_for(n), dim3(kThreads), 0, s, d_inv, d_rowptr, n, nnz, w.seen, w.rp_b, w.err);
    SAGNN_LAUNCH_CHECK();
  }
  int32_t h_err[4] = {0, 0, 0, 0};
  {
    const int64_t ntiles = ceil_div(n > 0 ? n : 1, kScanTile);
    hipLaunchKernelGGL(scan_tiles_kernel, dim3((unsigned)ntiles), dim3(kThreads), 0, s, w.rp_b, n, d_rowptr_p, w.tilesum);
    SAGNN_LAUNCH_CHECK();
    if (ntiles > kFewSums) {
      hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kThreads), 0, s, w.tilesum, ntiles);
      SAGNN_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(ntiles > kFewSums ? scan_add_kernel<true> : scan_add_kernel<false>, dim3((unsigned)ceil_div(n + 1, kScanTile)),
                       dim3(kThreads), 0, s, w.tilesum, n, nnz, d_rowptr_p);
    SAGNN_LAUNCH_CHECK();
    if (nnz > 0 && n > 0) {
      hipLaunchKernelGGL(permute_rows_kernel, dim3((unsigned)ceil_div(n, 4 * (kThreads / 64))), dim3(kThreads), 0, s,
                         d_rowptr, d_colidx, d_val, n, d_inv, w.seen, d_rowptr_p, d_colidx_p, d_val_p, w.err);
      SAGNN_LAUNCH_CHECK();
    }
    SAGNN_HIP(hipMemcpyAsync(h_err, w.err, sizeof(h_err), hipMemcpyDeviceToHost, s));
    SAGNN_HIP(hipStreamSynchronize(s));
    if (h_err[0] || h_err[1]) return SAGNN_EFORMAT;   // a column index outside [0, n), or d_inv is not a permutation
    if (!h_err[2]) return SAGNN_OK;
  }
  // rows that are too long (or overlap): through two sorts
  SAGNN_HIP(hipMemsetAsync(w.err, 0, sizeof(h_err), s));   // (the flags of the two sorts are among them)
  if (nnz > 0) {
    hipLaunchKernelGGL(relabel_kernel, grid_for(nnz), dim3(kThreads), 0, s, d_colidx, nnz, d_inv, n,
                       w.ci_a, w.err);
    SAGNN_LAUNCH_CHECK();
  }
  rc = launch_transpose(d_rowptr, w.ci_a, d_val, n, n, nnz, w.rp_b, w.ci_b, w.va_b, w.tws, w.err + 2, s);
  if (rc != SAGNN_OK) return rc;
  if (nnz > 0) {
    // ci_b holds old row ids (always in range); relabel them in place into ci_a
    hipLaunchKernelGGL(relabel_kernel, grid_for(nnz), dim3(kThreads), 0, s, w.ci_b, nnz, d_inv, n,
                       w.ci_a, w.err);
    SAGNN_LAUNCH_CHECK();
  }
  rc = launch_transpose(w.rp_b, w.ci_a, w.va_b, n, n, nnz, d_rowptr_p, d_colidx_p, d_val_p, w.tws, w.err + 3, s);
  if (rc != SAGNN_OK) return rc;
  SAGNN_HIP(hipMemcpyAsync(h_err, w.err, sizeof(h_err), hipMemcpyDeviceToHost, s));
  SAGNN_HIP(hipStreamSynchronize(s));
  if (h_err[0] || h_err[2] || h_err[3]) return SAGNN_EFORMAT;   // a column index outside [0, n)
  return SAGNN_OK;
}
