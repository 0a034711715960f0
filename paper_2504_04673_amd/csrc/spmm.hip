// Local CSR x tall-skinny dense product  C (+)= A * B  (Alg. 1 / Alg. 2, the statement
// "Z <- Z + SpMM(A_iq, H^)"; Sec. 4.1 block-sum equation).  fp32 FMA on the vector ALUs.
//
// This file holds the entry points, the preparation, the dispatch between the schedules (nonzero splitting:
// spmm_flat.hip; slab sweep: spmm_sweep.hip; dense tiles: tiles.hip), the kernel of accumulating calls over
// chunks, the kernel without a workspace and the layer's rows that the sweep leaves over.
// Operands wider than 256 are processed as column slabs.
#include <stdlib.h>


#include "common.h"
#include "rowload.h"

namespace sagnn {
namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWavesPerBlock * 64;

// Scalars of a launch.  Pointers are passed as separate __restrict__ kernel parameters: that
// is what lets the compiler prove the index/value streams are never written by the kernel and
// fetch them with scalar loads.
struct SpmmDims {
  int64_t m, nnz, nchunks, ldb, ldc, carry_ld;  // m, nnz, nchunks: of the CSR being walked
  uint64_t generation;
  uint32_t b_bytes;    // bytes addressable from B (buffer-load variant)
  uint32_t row_bytes;  // ldb * 4
  uint32_t kmax;  // k - 1: largest valid column index
  int32_t f;      // columns handled by this launch (slab width)
  int32_t accumulate;
};

__device__ __forceinline__ bool ws_matches(const SpmmWsHeader* __restrict__ hdr, const SpmmDims& d) {
  return hdr->magic == kSpmmMagic && hdr->generation == d.generation && hdr->c_rows == d.m &&
         hdr->c_nnz == d.nnz && hdr->c_nchunks == d.nchunks;
}

#define SPMM_PTR_PARAMS                                                                     \
  const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,                   \
      const float *__restrict__ val, const float *__restrict__ B, float *__restrict__ C,    \
      const SpmmWsHeader *__restrict__ hdr, const int4 *__restrict__ chunks,                \
      const uint32_t *__restrict__ flags, float *__restrict__ carry_base,                   \
      const int32_t *__restrict__ rowmap

// ------------------------------------------------------------------------------------------
// Accumulating calls (the per-stage sums of Alg. 2) at f == 64 * FPL: one chunk per wavefront, one entry per load.
// They read the old row of C at every row end; with short rows that read would sit on the critical path once per row,
// so the rows that end inside a batch of U entries are fetched together with the batch's rows of B.  (Column ids and
// values of a batch are wavefront-uniform: scalar loads.)
template <int FPL, int U, bool BUF>
__global__ __launch_bounds__(kBlock) void spmm_wide_accumulate_kernel(SPMM_PTR_PARAMS, const SpmmDims d) {
  using vec = typename Vec<FPL>::T;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t loff = lane * (FPL * 4);  // byte offset of this lane's columns inside a row
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t k = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  if (k >= d.nchunks) return;
  if (!ws_matches(hdr, d)) return;
  const int4 ch = chunks[k];
  const int32_t e0 = ch.x < 0 ? 0 : ch.x;
  const int32_t e1 = ch.y > d.nnz ? (int32_t)d.nnz : ch.y;
  if (e0 >= e1) return;
  int r = ch.z;
  bool head = ch.w & 1;  // first row began in an earlier chunk -> carry slot
  char* __restrict__ carry = reinterpret_cast<char*>(carry_base + k * d.carry_ld) + loff;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B, d.b_bytes);
  auto c_row = [&](int rr) -> vec* {
    const int rc = rr < 0 ? 0 : (rr < d.m ? rr : (int)(d.m - 1));
    const int64_t ro = rowmap ? rowmap[rc] : rc;
    return reinterpret_cast<vec*>(reinterpret_cast<char*>(C + ro * d.ldc) + loff);
  };

  vec acc = 0.f;
  auto flush = [&](const vec old) {
    if (r < d.m) {
      if (head) *reinterpret_cast<vec*>(carry) = acc;
      else *c_row(r) = acc + old;
    }
    head = false;
    acc = 0.f;
    ++r;
  };
  // entry e of the chunk, clamped so that the last batch never reads past the chunk
  auto fetch = [&](int32_t e, int32_t (&c)[U], float (&v)[U]) {
    if (e + U <= e1) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c[u] = colidx[e + u];
        v[u] = val[e + u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t ee = (e + u < e1) ? e + u : e1 - 1;
        c[u] = colidx[ee];
        v[u] = (e + u < e1) ? val[ee] : 0.f;
      }
    }
  };

  int32_t c[U];
  float v[U];
  fetch(e0, c, v);
  for (int32_t e = e0; e < e1; e += U) {
    const uint64_t two = (uint64_t)flags[e >> 5] | ((uint64_t)flags[(e >> 5) + 1] << 32);
    uint32_t fbits = (uint32_t)(two >> (e & 31)) & ((1u << U) - 1u);
    // (the chunk's last entry hands over the sum in any case: a row that continues in the next chunk before the steps
    // that fill up the batch, which multiply the last column's row by 0 whatever it holds)
    if (e + U >= e1) fbits = (fbits & ((1u << (e1 - e)) - 1u)) | (1u << (e1 - e - 1));
    vec h[U];
    float vc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t cc = (uint32_t)c[u] > d.kmax ? d.kmax : (uint32_t)c[u];
      h[u] = load_row<FPL, BUF>(rs, B, cc, loff, d.row_bytes, d.ldb);
      vc[u] = v[u];
    }
    vec cold[U];
#pragma unroll
    for (int u = 0; u < U; ++u) cold[u] = 0.f;
    if (fbits) {
      int rr = r;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if ((fbits >> u) & 1u) cold[u] = *c_row(rr++);
    }
    if (e + U < e1) fetch(e + U, c, v);
    // keep the U loads above together (the compiler would otherwise sink each one next to its use)
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" : "+v"(h[u]));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc += vc[u] * h[u];
      if ((fbits >> u) & 1u) flush(cold[u]);
    }
  }
}

// header of a prepared workspace; empty: its has_empty_rows where the host does not know it yet
__global__ void spmm_header_kernel(SpmmWsHeader h, const int32_t* __restrict__ empty, SpmmWsHeader* __restrict__ out) {
  if (threadIdx.x != 0) return;
  if (empty) h.has_empty_rows = *empty;
  *out = h;
}

// rows without entries: C[r,:] = 0 when overwriting (no chunk ever visits them).  A lane looks at a row, the wavefront
// zeroes the empty ones together (a wavefront per row for the look as well: 72 us for 1 M rows, now 26).
__global__ __launch_bounds__(kBlock) void spmm_zero_empty_kernel(SPMM_PTR_PARAMS, const SpmmDims d,
                                                                 int32_t f_total) {
  if (hdr->magic != kSpmmMagic || hdr->generation != d.generation || hdr->has_empty_rows == 0) return;
  const int lane = threadIdx.x & 63;
  const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
  const int f4 = f_total >> 2;
  for (int64_t r0 = wave0 * 64; r0 < d.m; r0 += nwaves * 64) {
    const int64_t r = r0 + lane;
    uint64_t empty = __ballot(r < d.m && rowptr[r + 1] == rowptr[r]);
    if (f4 <= 16) {
      // several rows per store: lane l takes quad l % f4 of the (l / f4)-th empty row
      const int per = 64 / f4, mine = lane / f4, q = lane - mine * f4;
      while (empty) {
        uint64_t rest = empty;
        for (int i = 0; i < mine && rest; ++i) rest &= rest - 1;
        if (mine < per && rest)
          *reinterpret_cast<float4*>(C + (r0 + __builtin_ctzll(rest)) * d.ldc + q * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i = 0; i < per && empty; ++i) empty &= empty - 1;
      }
    } else {
      for (; empty; empty &= empty - 1) {
        float* __restrict__ row = C + (r0 + __builtin_ctzll(empty)) * d.ldc;
        for (int c4 = lane; c4 < f4; c4 += 64) *reinterpret_cast<float4*>(row + c4 * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
}

// Rows of B moved to rows that begin on a cache line (see spmm_pad_pays): a row of 96 bytes touches one line instead of
// one and a half.  1 M rows, 50 M entries, f = 24: 677 -> 585 us with the copy, f = 60: 1323 -> 1023.
__global__ __launch_bounds__(kBlock) void spmm_pad_kernel(const float* __restrict__ B, int64_t ldb, int32_t f4,
                                                          int64_t quads, float* __restrict__ out, int32_t ld_out) {
  const int64_t q0 = (int64_t)blockIdx.x * (4 * kBlock) + threadIdx.x;
  float4 v[4];
  int64_t r[4];
  int32_t c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t q = q0 + j * kBlock;
    if (q >= quads) break;
    r[j] = (uint64_t)q < 0x80000000ull ? (uint32_t)q / (uint32_t)f4 : q / f4;
    c[j] = (int32_t)(q - r[j] * f4) * 4;
    v[j] = *reinterpret_cast<const float4*>(B + r[j] * ldb + c[j]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (q0 + j * kBlock < quads) *reinterpret_cast<float4*>(out + r[j] * ld_out + c[j]) = v[j];
}

// ------------------------------------------------------------------------------------------
// fallback without a prepared workspace: one wavefront per row, float4 pieces along f
__global__ __launch_bounds__(kBlock) void spmm_row_kernel(SPMM_PTR_PARAMS, const SpmmDims d,
                                                          int32_t f_total) {
  const int lane = threadIdx.x & 63;
  const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
  for (int64_t r = wave0; r < d.m; r += nwaves) {
    int32_t lo = rowptr[r], hi = rowptr[r + 1];
    lo = lo < 0 ? 0 : lo;
    hi = hi > d.nnz ? (int32_t)d.nnz : hi;
    for (int c4 = lane; c4 * 4 < f_total; c4 += 64) {
      // two-level sum: runs of 128 entries, then the runs (keeps the rounding error of a long
      // row of equal terms from growing with the row length)
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), tot = acc;
      for (int32_t e = lo; e < hi; ++e) {
        const uint32_t c = (uint32_t)colidx[e];
        const uint32_t cc = c > d.kmax ? d.kmax : c;
        const float v = val[e];
        const float4 h = *reinterpret_cast<const float4*>(B + (int64_t)cc * d.ldb + c4 * 4);
        acc.x += v * h.x; acc.y += v * h.y; acc.z += v * h.z; acc.w += v * h.w;
        if (((e - lo) & 127) == 127) {
          tot.x += acc.x; tot.y += acc.y; tot.z += acc.z; tot.w += acc.w;
          acc = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
      acc.x += tot.x; acc.y += tot.y; acc.z += tot.z; acc.w += tot.w;
      float4* p = reinterpret_cast<float4*>(C + r * d.ldc + c4 * 4);
      if (d.accumulate) {
        const float4 o = *p;
        acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
      }
      *p = acc;
    }
  }
}

inline unsigned capped_grid(int64_t blocks) {
  const int64_t cap = 256 * 64;
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  return (unsigned)blocks;
}

struct SpmmPtrs {
  const int32_t* rowptr; const int32_t* colidx; const float* val; const float* B; float* C;
  const SpmmWsHeader* hdr; const int4* chunks; const uint32_t* flags; float* carry;
  const int32_t* rowmap;
};

template <typename Kern, typename... Extra>
inline void launch_waves(Kern kern, int64_t blocks, const SpmmPtrs& p, const SpmmDims& d,
                         hipStream_t s, Extra... extra) {
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kBlock), 0, s, p.rowptr, p.colidx, p.val,
                     p.B, p.C, p.hdr, p.chunks, p.flags, p.carry, p.rowmap, d, extra...);
}

}  // namespace

uint64_t spmm_next_generation();
int sweep_combine(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, float* C, int64_t ldc,
                  int32_t f_total, int32_t accumulate, hipStream_t s);

namespace {
int launch_spmm_body(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                     int64_t k, int64_t nnz, const float* B, int64_t ldb, int32_t f, float* C,
                     int64_t ldc, int32_t accumulate, void* ws, size_t ws_bytes, hipStream_t s, bool inner);
}
int launch_spmm(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                int64_t k, int64_t nnz, const float* B, int64_t ldb, int32_t f, float* C,
                int64_t ldc, int32_t accumulate, void* ws, size_t ws_bytes, hipStream_t s) {
  return launch_spmm_body(rowptr, colidx, val, m, k, nnz, B, ldb, f, C, ldc, accumulate, ws, ws_bytes, s, false);
}
namespace {
// inner: the call is the rest-CSR part of a workspace prepared with dense tiles
int launch_spmm_body(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                     int64_t k, int64_t nnz, const float* B, int64_t ldb, int32_t f, float* C,
                     int64_t ldc, int32_t accumulate, void* ws, size_t ws_bytes, hipStream_t s, bool inner) {
  if (m < 0 || k < 0 || nnz < 0 || f <= 0 || (f & 3) || ldb < f || ldc < f || (ldb & 3) ||
      (ldc & 3) || m > 0x7FFFFFFFll || k > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  if (accumulate != 0 && accumulate != 1) return SAGNN_EINVAL;
  if (m == 0) return SAGNN_OK;
  if (!rowptr || !C || !aligned16(C)) return SAGNN_EINVAL;
  if (nnz > 0 && (!colidx || !val || !B || !aligned16(B) || k == 0)) return SAGNN_EINVAL;
  if (ws && (reinterpret_cast<uintptr_t>(ws) & 255u)) return SAGNN_EINVAL;

  SpmmPtrs p{};
  p.rowptr = rowptr; p.colidx = colidx; p.val = val; p.B = B; p.C = C;
  SpmmDims d{};
  d.m = m; d.nnz = nnz; d.ldb = ldb; d.ldc = ldc;
  d.kmax = k > 0 ? (uint32_t)(k - 1) : 0u;
  d.f = f; d.accumulate = accumulate;
  d.carry_ld = f;

  if (!ws) {
    launch_waves(spmm_row_kernel, capped_grid(ceil_div(m, kWavesPerBlock)), p, d, s, f);
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  }

  SpmmHostDesc desc{};
  if (!spmm_desc_get(ws, &desc)) return SAGNN_EINVAL;        // never prepared in this process
  if (desc.tiles && !inner) {
    // dense tiles: the rest CSR (stored behind the plain workspace) through the schedule prepared
    // for it, then C += tiles * B out of LDS
    if (desc.m != m || desc.full_nnz != nnz || desc.f != f || k < desc.k) return SAGNN_EINVAL;
    const size_t plain = spmm_ws_layout(m, desc.full_nnz, desc.f).need;
    const TileWsLayout TL = tile_ws_layout(m, desc.k, desc.full_nnz, desc.f);
    if (ws_bytes < plain + TL.total) return SAGNN_ECAPACITY;
    char* tb = reinterpret_cast<char*>(ws) + plain;
    int rc = launch_spmm_body(reinterpret_cast<const int32_t*>(tb + TL.rest_rowptr),
                              reinterpret_cast<const int32_t*>(tb + TL.rest_col),
                              reinterpret_cast<const float*>(tb + TL.rest_val), m, k, desc.nnz, B, ldb, f, C, ldc,
                              accumulate, ws, plain, s, true);
    if (rc != SAGNN_OK) return rc;
    TilePlan tp{};
    tp.n_ts = desc.tile_count; tp.n_items = desc.tile_items; tp.entries = desc.tile_entries;
    tp.rest_nnz = desc.nnz; tp.rows = desc.tile_rows;
    return tile_launch(tp, desc.tile_generation, tb, TL, B, ldb, d.kmax, f, m, C, ldc, s);
  }
  if (desc.m != m || desc.nnz != nnz || desc.f < f) return SAGNN_EINVAL;
  // the re-ordered entry streams hold column ids checked against the k of the preparation: an
  // operand with fewer rows would be read out of range
  if (nnz > 0 && k < desc.k) return SAGNN_EINVAL;
  const SpmmWsLayout L = spmm_ws_layout(m, nnz, desc.f);
  if (ws_bytes < L.need) return SAGNN_ECAPACITY;
  char* base = reinterpret_cast<char*>(ws);
  p.hdr = reinterpret_cast<const SpmmWsHeader*>(base + L.header);
  p.chunks = reinterpret_cast<const int4*>(base + L.chunks);
  p.flags = reinterpret_cast<const uint32_t*>(base + L.flags);
  p.carry = reinterpret_cast<float*>(base + L.carry);
  d.generation = desc.generation;
  d.nchunks = desc.c_nchunks;

  if (k <= L.padded_rows && ws_bytes >= L.total && f <= desc.f && spmm_padded_width(f) <= spmm_padded_width(desc.f) && spmm_pad_pays(k, nnz, f, ldb)) {
    float* padded = reinterpret_cast<float*>(base + L.padded);
    const int32_t fp = spmm_padded_width(f);
    const int64_t quads = k * (f / 4);
    hipLaunchKernelGGL(spmm_pad_kernel, dim3((unsigned)ceil_div(quads, 4 * kBlock)), dim3(kBlock), 0, s, B, ldb, f / 4,
                       quads, padded, fp);
    SAGNN_LAUNCH_CHECK();
    B = p.B = padded;
    ldb = d.ldb = fp;
  }
  if (!accumulate && desc.has_empty_rows) {
    launch_waves(spmm_zero_empty_kernel, capped_grid(ceil_div(m, kBlock)), p, d, s, f);
    SAGNN_LAUNCH_CHECK();
  }
  if (desc.mode == 1) {
    // the chunk kernels walk the compacted short-row CSR stored in the workspace
    const int64_t short_base = (int64_t)round_up((size_t)desc.sweep_stream_len + 64, 256);
    p.rowptr = reinterpret_cast<const int32_t*>(base + L.rowptr_s);
    p.rowmap = reinterpret_cast<const int32_t*>(base + L.rowmap_s);
    p.colidx = reinterpret_cast<const int32_t*>(base + L.code) + short_base;
    p.val = reinterpret_cast<const float*>(base + L.vals) + short_base;
    d.m = desc.c_rows; d.nnz = desc.c_nnz;
  } else if (desc.c_rows != m) {
    // empty rows were taken out of the row list when the workspace was prepared
    p.rowptr = reinterpret_cast<const int32_t*>(base + L.rowptr_s);
    p.rowmap = reinterpret_cast<const int32_t*>(base + L.rowmap_s);
    d.m = desc.c_rows;
  }

  FlatArgs fl{};
  fl.rows = d.m; fl.nnz = d.nnz; fl.nchunks = d.nchunks; fl.colidx = p.colidx; fl.val = p.val; fl.B = B; fl.ldb = ldb;
  fl.kmax = d.kmax; fl.C = C; fl.ldc = ldc; fl.accumulate = accumulate; fl.hdr = p.hdr; fl.generation = d.generation;
  fl.chunks = p.chunks; fl.flags = p.flags; fl.carry = p.carry; fl.carry_ld = f; fl.rowmap = p.rowmap;
  fl.hubs = desc.n_fix_big > 0;
  if (desc.mode == 1) {
    const int32_t max_slab = desc.max_slab == 128 ? 128 : 256;
    const bool narrow = desc.col_slab > 0 && f % desc.col_slab == 0;
    for (int32_t col0 = 0, fw = 0; col0 < f; col0 += fw) {
      fw = narrow ? desc.col_slab : sweep_slab(f - col0, max_slab);
      int rc = sweep_launch(desc, L, base, B, ldb, col0, fw, d.kmax, C, ldc, accumulate, f, s);
      if (rc != SAGNN_OK) return rc;
    }
  }
  // column slabs of at most 256
  if (d.nchunks > 0) {
    for (int32_t col0 = 0, fw = 0; col0 < f; col0 += fw) {
      fw = f - col0 >= 256 ? 256 : f - col0;
      if (accumulate && (fw == 64 || fw == 128 || fw == 256)) {
        SpmmPtrs sp = p;
        SpmmDims sd = d;
        sp.B = B + col0; sp.C = C + col0; sp.carry = p.carry + col0;
        sd.f = fw;
        sd.row_bytes = (uint32_t)(ldb * 4);
        const bool buf = buffer_addressable(d.kmax, ldb, fw, &sd.b_bytes);
        const int64_t blocks = ceil_div(d.nchunks, kWavesPerBlock);
#define SAGNN_WIDE(FPL_)                                                                        \
  (buf ? launch_waves(spmm_wide_accumulate_kernel<FPL_, 8, true>, blocks, sp, sd, s)            \
       : launch_waves(spmm_wide_accumulate_kernel<FPL_, 8, false>, blocks, sp, sd, s))
        if (fw == 256) SAGNN_WIDE(4);
        else if (fw == 128) SAGNN_WIDE(2);
        else SAGNN_WIDE(1);
#undef SAGNN_WIDE
        SAGNN_LAUNCH_CHECK();
      } else {
        int rc = flat_launch(fl, col0, fw, s);
        if (rc != SAGNN_OK) return rc;
      }
    }
  }
  {
    int rc = flat_fixup(fl, reinterpret_cast<const int2*>(base + L.fix_list), L.max_chunks, desc.n_fix, desc.n_fix_big, f, s);
    if (rc != SAGNN_OK) return rc;
  }
  if (desc.mode == 1) {
    int rc = sweep_combine(desc, L, base, C, ldc, f, accumulate, s);
    if (rc != SAGNN_OK) return rc;
  }
  return SAGNN_OK;
}
}  // namespace

// ------------------------------------------------------------------------------------------
// The layer with the dense transform as the epilogue of the slab sweep (spmm_sweep_fused_kernel)
// covers the rows that one wavefront of the sweep finishes.  The others -- rows outside the sweep
// (short rows) and rows cut into several pieces -- are few where this form is used and go
// through this kernel: one wavefront per row computes the row of T (a gather over the row's
// entries, or the sum of the row's partial rows in a fixed order), puts it into LDS and
// multiplies it by W, 64 output columns at a time.
namespace {
constexpr int64_t kFusedLeftoverMax = 65536;   // rows; above that the row-range kernel serves the layer

template <int FPL, bool BF16>
__global__ __launch_bounds__(256) void layer_leftover_kernel(
    const int32_t* __restrict__ rowptr_s, const int32_t* __restrict__ rowmap_s,
    const int32_t* __restrict__ colidx_s, const float* __restrict__ val_s, int64_t n_short, int64_t nnz_s,
    const int32_t* __restrict__ multi_row, const int32_t* __restrict__ multi_first, int64_t n_multi,
    const float* __restrict__ partial, const SpmmWsHeader* __restrict__ hdr, uint64_t generation,
    const float* __restrict__ B, int64_t ldb, uint32_t kmax, const SweepFusedArgs fa) {
  using vec = typename Vec<FPL>::T;
  constexpr int kRow = 64 * FPL;
  __shared__ float trow[4][kRow];
  if (hdr->magic != kSpmmMagic || hdr->generation != generation) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 4 + wave;
  int64_t row = -1;
  vec t = 0.f;
  if (i < n_short) {
    row = rowmap_s[i];
    int32_t b = rowptr_s[i], e = rowptr_s[i + 1];
    b = b < 0 ? 0 : b;
    e = e > nnz_s ? (int32_t)nnz_s : e;
    for (int32_t q = b; q < e; ++q) {
      const uint32_t cc = (uint32_t)colidx_s[q];
      const uint32_t c = cc > kmax ? kmax : cc;
      t += val_s[q] * *reinterpret_cast<const vec*>(B + (int64_t)c * ldb + lane * FPL);
    }
  } else if (i < n_short + n_multi) {
    const int64_t q = i - n_short;
    row = multi_row[q];
    for (int32_t j = multi_first[q]; j < multi_first[q + 1]; ++j)
      t += *reinterpret_cast<const vec*>(partial + (int64_t)j * kRow + lane * FPL);
  }
  if (row >= 0 && fa.T) *reinterpret_cast<vec*>(fa.T + row * kRow + lane * FPL) = t;
  if constexpr (FPL == 1) {
    trow[wave][lane] = BF16 ? (float)(__bf16)t : t;
  } else {
#pragma unroll
    for (int c = 0; c < FPL; ++c) trow[wave][lane * FPL + c] = BF16 ? (float)(__bf16)t[c] : t[c];
  }
  __syncthreads();
  if (row < 0) return;
  for (int col = lane; col < fa.f_out; col += 64) {
    float z = 0.f;
    for (int k = 0; k < kRow; ++k) {
      const float w = fa.W[(int64_t)k * fa.f_out + col];
      z += trow[wave][k] * (BF16 ? (float)(__bf16)w : w);
    }
    if (fa.Z) fa.Z[row * fa.f_out + col] = z;
    if (fa.Hout) fa.Hout[row * fa.f_out + col] = fa.act == SAGNN_ACT_RELU ? (z > 0.f ? z : 0.f) : z;
  }
}
}  // namespace

bool fused_sweep_layer_applicable(const void* ws, int32_t f_in, int32_t f_out) {
  SpmmHostDesc desc{};
  if (!ws || !spmm_desc_get(ws, &desc)) return false;
  if (desc.apart) return false;
  if (desc.tiles) return false;   // rows with entries in dense tiles are not finished by the sweep
  if (desc.mode != 1 || desc.slots != kSweepSlots || desc.n_waves <= 0 || (desc.n_waves & 3)) return false;
  if (!(f_in == 64 || f_in == 128 || f_in == 256) || f_in > desc.f || f_in > desc.max_slab) return false;
  // the launch must cover the whole width of T with one kernel of the prepared schedule
  if (desc.groups == 2 ? f_in > 128 : (desc.groups == 4 ? f_in != 64 : desc.groups != 1)) return false;
  if (f_out <= 0 || (f_out & 3) || f_out > 256) return false;
  return desc.c_rows + desc.n_multi_rows <= kFusedLeftoverMax;
}

int launch_fused_sweep_layer(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                             int64_t k, int64_t nnz, const float* H, int64_t ldh, int32_t f_in,
                             const float* W, int32_t f_out, int32_t act, int32_t prec, float* T, float* Z,
                             float* Hout, void* ws, size_t ws_bytes, hipStream_t s) {
  (void)colidx; (void)val;   // the prepared workspace holds its own copy of the entries
  SpmmHostDesc desc{};
  if (!fused_sweep_layer_applicable(ws, f_in, f_out) || !spmm_desc_get(ws, &desc)) return 1;
  if (desc.m != m || desc.nnz != nnz) return SAGNN_EINVAL;
  if (prec != SAGNN_GEMM_FP32 && prec != SAGNN_GEMM_BF16 && prec != SAGNN_GEMM_FP32_BF16X3) return SAGNN_EINVAL;
  if (act != SAGNN_ACT_IDENTITY && act != SAGNN_ACT_RELU) return SAGNN_EINVAL;
  if (nnz > 0 && k < desc.k) return SAGNN_EINVAL;
  if (!rowptr || !H || !W || (!Z && !Hout) || ldh < f_in || (ldh & 3) || !aligned16(H)) return SAGNN_EINVAL;
  const SpmmWsLayout L = spmm_ws_layout(m, nnz, desc.f);
  if (ws_bytes < L.need) return SAGNN_ECAPACITY;
  char* base = reinterpret_cast<char*>(ws);
  const SpmmWsHeader* hdr = reinterpret_cast<const SpmmWsHeader*>(base + L.header);
  const uint32_t kmax = k > 0 ? (uint32_t)(k - 1) : 0u;
  const bool bf16 = prec == SAGNN_GEMM_BF16;   // (the few rows left to the small kernel: three-term mode uses fp32 there)

  if (desc.has_empty_rows) {   // a row without entries: T = 0, so Z = 0 and sigma(0) = 0
    SpmmPtrs p{};
    p.rowptr = rowptr; p.hdr = hdr;
    SpmmDims d{};
    d.m = m; d.generation = desc.generation;
    float* outs[3] = {Z, Hout, T};
    const int32_t widths[3] = {f_out, f_out, f_in};
    for (int o = 0; o < 3; ++o) {
      if (!outs[o]) continue;
      p.C = outs[o];
      d.ldc = widths[o];
      launch_waves(spmm_zero_empty_kernel, capped_grid(ceil_div(m, kBlock)), p, d, s, widths[o]);
      SAGNN_LAUNCH_CHECK();
    }
  }
  SweepFusedArgs fa{};
  fa.W = W; fa.Z = Z; fa.Hout = Hout; fa.T = T; fa.f_out = f_out; fa.act = act;
  int rc = sweep_launch_fused(desc, L, base, H, ldh, f_in, kmax, fa, prec, s);   // (operand modes are numbered like prec)
  if (rc != SAGNN_OK) return rc;
  const int64_t left = desc.c_rows + desc.n_multi_rows;
  if (left > 0) {
    const int64_t short_base = (int64_t)round_up((size_t)desc.sweep_stream_len + 64, 256);
    auto go = [&](auto kern) -> int {
      hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(left, 4)), dim3(256), 0, s,
                         reinterpret_cast<const int32_t*>(base + L.rowptr_s),
                         reinterpret_cast<const int32_t*>(base + L.rowmap_s),
                         reinterpret_cast<const int32_t*>(base + L.code) + short_base,
                         reinterpret_cast<const float*>(base + L.vals) + short_base, desc.c_rows, desc.c_nnz,
                         reinterpret_cast<const int32_t*>(base + L.multi_row),
                         reinterpret_cast<const int32_t*>(base + L.multi_first), desc.n_multi_rows,
                         reinterpret_cast<const float*>(base + L.partial), hdr, desc.generation, H, ldh, kmax, fa);
      SAGNN_LAUNCH_CHECK();
      return SAGNN_OK;
    };
    if (f_in == 256) rc = bf16 ? go(layer_leftover_kernel<4, true>) : go(layer_leftover_kernel<4, false>);
    else if (f_in == 128) rc = bf16 ? go(layer_leftover_kernel<2, true>) : go(layer_leftover_kernel<2, false>);
    else rc = bf16 ? go(layer_leftover_kernel<1, true>) : go(layer_leftover_kernel<1, false>);
    if (rc != SAGNN_OK) return rc;
  }
  return SAGNN_OK;
}

}  // namespace sagnn

SAGNN_EXPORT int spmm_csr_workspace_bytes(int64_t m, int64_t nnz, int32_t f, size_t* bytes) {
  using namespace sagnn;
  if (!bytes || m < 0 || nnz < 0 || f <= 0 || (f & 3) || nnz > 0x7FFFFFFFll || m > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  *bytes = spmm_ws_bytes(m, nnz, f);
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_workspace_bytes_opt(int64_t m, int64_t k, int64_t nnz, int32_t f,
                                              const sagnn_spmm_options* h_opt, size_t* bytes) {
  using namespace sagnn;
  if (!bytes || m < 0 || k < 0 || nnz < 0 || f <= 0 || (f & 3) || nnz > 0x7FFFFFFFll || m > 0x7FFFFFFFll ||
      k > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  size_t b = spmm_ws_bytes(m, nnz, f);
  TileGeom g{};
  if (h_opt && h_opt->dense_tiles == 1 && tile_geom(f, &g)) b += tile_ws_layout(m, k, nnz, f).total;
  *bytes = b;
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_tile_info(const void* d_ws, int64_t* h_info) {
  using namespace sagnn;
  if (!d_ws || !h_info) return SAGNN_EINVAL;
  SpmmHostDesc d{};
  if (!spmm_desc_get(d_ws, &d)) return SAGNN_EINVAL;
  h_info[0] = d.tiles;
  h_info[1] = d.tiles ? d.tile_entries : 0;
  h_info[2] = d.tiles ? d.tile_count : 0;
  h_info[3] = d.tiles ? d.tile_items : 0;
  h_info[4] = d.tiles ? d.tile_rows : 0;
  h_info[5] = d.tiles ? d.nnz : 0;
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_prepare_opt(const int32_t* d_rowptr, const int32_t* d_colidx,
                                      const float* d_val, int64_t m, int64_t k, int64_t nnz, int32_t f,
                                      void* d_ws, size_t ws_bytes, const sagnn_spmm_options* h_opt,
                                      void* stream) {
  using namespace sagnn;
  sagnn_spmm_options opt{};
  if (h_opt) opt = *h_opt;
  if (opt.short_rows < -1 || opt.short_rows > 1 ||
      (opt.slab_width != 0 && opt.slab_width != 128 && opt.slab_width != 256))
    return SAGNN_EINVAL;
  if (m < 0 || k < 0 || nnz < 0 || f <= 0 || (f & 3) || m > 0x7FFFFFFFll || nnz > 0x7FFFFFFFll ||
      k > 0x7FFFFFFFll)
    return SAGNN_EINVAL;
  if (!d_rowptr || !d_ws || (reinterpret_cast<uintptr_t>(d_ws) & 255u)) return SAGNN_EINVAL;
  if (nnz > 0 && (!d_colidx || !d_val)) return SAGNN_EINVAL;
  const SpmmWsLayout L = spmm_ws_layout(m, nnz, f);
  if (ws_bytes < L.need) return SAGNN_ECAPACITY;
  hipStream_t s = (hipStream_t)stream;
  char* base = reinterpret_cast<char*>(d_ws);
  if (opt.dense_tiles < -1 || opt.dense_tiles > 1 || opt.tile_reuse_x10 < 0) return SAGNN_EINVAL;
  TileGeom tg{};
  if (opt.dense_tiles == 1 && tile_geom(f, &tg) && m > 0 && k > 0 && nnz > 0) {
    // dense tiles: split A into the kept tiles and a rest CSR (both in the tile region behind the
    // plain workspace), then prepare the rest like any other matrix
    const size_t plain = L.need;
    const TileWsLayout TL = tile_ws_layout(m, k, nnz, f);
    if (ws_bytes < plain + TL.total) return SAGNN_ECAPACITY;
    TilePlan tp{};
    const uint64_t gen = spmm_next_generation();
    int rc = tile_prepare(d_rowptr, d_colidx, d_val, m, k, nnz, f, base + plain, TL, opt.tile_reuse_x10, gen, s, &tp);
    if (rc != SAGNN_OK) return rc;
    if (tp.n_ts > 0) {
      sagnn_spmm_options inner_opt = opt;
      inner_opt.dense_tiles = -1;
      char* tb = base + plain;
      rc = spmm_csr_prepare_opt(reinterpret_cast<const int32_t*>(tb + TL.rest_rowptr),
                                reinterpret_cast<const int32_t*>(tb + TL.rest_col),
                                reinterpret_cast<const float*>(tb + TL.rest_val), m, k, tp.rest_nnz, f, d_ws, plain,
                                &inner_opt, stream);
      if (rc != SAGNN_OK) return rc;
      SpmmHostDesc desc{};
      if (!spmm_desc_get(d_ws, &desc)) return SAGNN_EINVAL;
      desc.tiles = 1;
      desc.full_nnz = nnz;
      desc.tile_count = tp.n_ts; desc.tile_items = tp.n_items; desc.tile_entries = tp.entries;
      desc.tile_rows = tp.rows; desc.tile_generation = gen;
      spmm_desc_put(d_ws, desc);
      return SAGNN_OK;
    }
    // no tile is dense enough: the plain preparation below
  }
  int32_t* d_stat = reinterpret_cast<int32_t*>(base + L.carry);  // scratch until the first product
  int32_t stat[4] = {0, 0, 0, 0};    // of flat_build_tables
  auto read_stat = [&]() -> int {
    SAGNN_HIP(hipMemcpyAsync(stat, d_stat, sizeof(stat), hipMemcpyDeviceToHost, s));
    SAGNN_HIP(hipStreamSynchronize(s));
    return SAGNN_OK;
  };
  // (the header travels as a kernel argument: a copy from the host's stack cost a wait of its own)
  bool header_there = false;
  auto put_header = [&](const SpmmWsHeader& hd, const int32_t* d_empty) -> int {
    hipLaunchKernelGGL(spmm_header_kernel, dim3(1), dim3(64), 0, s, hd, d_empty, reinterpret_cast<SpmmWsHeader*>(base + L.header));
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  };

  SweepPlanResult plan{};
  {
    int rc = sweep_prepare(d_rowptr, d_colidx, d_val, m, k, nnz, f, base, L, opt, false, s, &plan);
    if (rc != SAGNN_OK) return rc;
  }
  SpmmWsHeader h{};
  const int64_t T = spmm_chunk_entries(nnz, f);
  if (!plan.use_sweep) {
    h.magic = kSpmmMagic;
    h.m = m; h.nnz = nnz; h.f = f; h.mode = 0;
    h.generation = spmm_next_generation();
    h.c_rows = m; h.c_nnz = nnz; h.c_nchunks = spmm_nchunks(nnz, T);
    int rc = flat_build_tables(d_rowptr, m, nnz, T, base, L, d_stat, s);
    if (rc == SAGNN_OK) rc = put_header(h, d_stat);
    if (rc == SAGNN_OK) rc = read_stat();
    if (rc != SAGNN_OK) return rc;
    // The tables tell, at no cost to a matrix with hubs, that there is none: then the sweep is looked at again (its own
    // sample and wait take about 0.05 ms, the whole plan 0.3 to 1.3).
    if (opt.schedule == 0 && stat[2] == 0 && !sweep_size(k, nnz, f)) {
      rc = sweep_prepare(d_rowptr, d_colidx, d_val, m, k, nnz, f, base, L, opt, true, s, &plan);
      if (rc != SAGNN_OK) return rc;
    }
  }
  if (plan.use_sweep) {
    h = plan.hdr;
    stat[1] = stat[2] = 0;
    if (h.c_nchunks > 0) {
      int rc = flat_build_tables(reinterpret_cast<const int32_t*>(base + L.rowptr_s), h.c_rows, h.c_nnz,
                                 spmm_chunk_entries(h.c_nnz, f), base, L, d_stat, s);
      if (rc == SAGNN_OK) rc = read_stat();
      if (rc != SAGNN_OK) return rc;
    }
  } else {
    h.has_empty_rows = stat[0];
    header_there = true;
    if (stat[0] && nnz > 0) {
      // Rows without entries (e.g. one column block of a row block, Alg. 2) would have to be stepped over one
      // dependent load at a time.  Walk a row list without them instead: the same compacted-CSR form the short rows
      // of the sweep schedule use.
      // The row pass of the sweep planner with a threshold no row reaches makes exactly that list
      // (every row with entries is "short").
      SweepRowTotals t{};
      int rc = sweep_plan_sample(d_rowptr, nullptr, m, k, nnz, 0x7FFFFFFF, base, L, s, nullptr);
      if (rc == SAGNN_OK) rc = sweep_plan_rows(d_rowptr, m, 1024, base, L, s, &t);
      if (rc != SAGNN_OK) return rc;
      if (!t.bad && t.short_entries == nnz) {   // (a malformed row pointer keeps the plain walk, which clamps everything)
        rc = flat_build_tables(reinterpret_cast<const int32_t*>(base + L.rowptr_s), t.short_rows, nnz, T, base, L, d_stat, s);
        if (rc == SAGNN_OK) rc = read_stat();
        if (rc != SAGNN_OK) return rc;
        h.c_rows = t.short_rows;
        header_there = false;
      }
    }
  }
  if (stat[1] < 0 || stat[2] < 0 || (int64_t)stat[1] + stat[2] > L.max_chunks) return SAGNN_EFORMAT;   // (overlapping rows)
  if (!header_there) {
    const int rc = put_header(h, nullptr);
    if (rc != SAGNN_OK) return rc;
    SAGNN_HIP(hipStreamSynchronize(s));
  }
  SpmmHostDesc desc{};
  desc.generation = h.generation; desc.m = m; desc.nnz = nnz; desc.f = f; desc.mode = h.mode;
  desc.c_rows = h.c_rows; desc.c_nnz = h.c_nnz; desc.c_nchunks = h.c_nchunks;
  desc.n_fix = stat[1]; desc.n_fix_big = stat[2];
  desc.n_waves = h.n_waves; desc.n_multi_rows = h.n_multi_rows; desc.has_empty_rows = h.has_empty_rows;
  desc.sweep_stream_len = h.n_long_entries;
  desc.groups = h.groups > 0 ? h.groups : 1;
  desc.k = k;
  desc.n_intervals = h.n_intervals; desc.sync_slabs = h.sync_slabs; desc.wg_per_cohort = h.wg_per_cohort;
  desc.sync_timeout_ticks = h.sync_timeout_ticks; desc.sync_test_extra = h.sync_test_extra;
  desc.slots = h.slots;
  desc.max_slab = h.max_slab > 0 ? h.max_slab : 256;
  desc.n_slabs = h.n_slabs;
  desc.col_slab = h.col_slab; desc.launch_waves = h.launch_waves; desc.fused_waves = h.fused_waves;
  desc.apart = plan.use_sweep && !sweep_size(k, nnz, f) && opt.schedule != 2;
  desc.barriers = h.barriers; desc.pace_ps_per_step = h.pace_ps_per_step > 0 ? h.pace_ps_per_step : 0;
  desc.reuse = plan.reuse; desc.turns = plan.turns; desc.layer_turns = plan.layer_turns; desc.narrow_sums = plan.narrow_sums;
  desc.run_blocks = plan.run_blocks; desc.long_waves = plan.long_waves; desc.run_rows = plan.run_rows;
  desc.mean_steps = plan.mean_steps;
  desc.max_steps = plan.max_steps;
  spmm_desc_put(d_ws, desc);
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_prepare(const int32_t* d_rowptr, const int32_t* d_colidx,
                                  const float* d_val, int64_t m, int64_t k, int64_t nnz, int32_t f,
                                  void* d_ws, size_t ws_bytes, void* stream) {
  return spmm_csr_prepare_opt(d_rowptr, d_colidx, d_val, m, k, nnz, f, d_ws, ws_bytes, nullptr, stream);
}

SAGNN_EXPORT int spmm_csr_prepare_tuned(const int32_t* d_rowptr, const int32_t* d_colidx,
                                        const float* d_val, int64_t m, int64_t k, int64_t nnz,
                                        int32_t f, void* d_ws, size_t ws_bytes, const float* d_B,
                                        int64_t ldb, float* d_C, int64_t ldc, int32_t* h_choice,
                                        const sagnn_spmm_options* h_opt, void* stream) {
  using namespace sagnn;
  if (!d_B || !d_C || ldb < f || ldc < f) return SAGNN_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  // (piece, long-row threshold) variants of the slab-sweep plan; {0, 0} is spmm_csr_prepare's own
  struct Cand { int piece, min_long, slab; };
  static const Cand cand[] = {{0, 0, 0}, {4608, 0, 0}, {3584, 0, 0}, {0, 96, 0}, {4608, 96, 0},
                              {0, 0, 128}, {4608, 0, 128}};
  // the 128-wide-slab variants only exist for operands wider than 128
  const int n_cand = (f > 128 && (f & 63) == 0 && !(h_opt && h_opt->slab_width != 0)) ? 7 : 5;
  // a variant only replaces choices the planner would make by itself: where it picks the
  // lower long-row threshold (near-regular matrices) the candidate threshold is not forced
  auto options_of = [&](int c) {
    sagnn_spmm_options o{};
    if (h_opt) o = *h_opt;
    if (cand[c].piece > 0) o.piece = cand[c].piece;
    if (cand[c].min_long > 0) o.min_long = -cand[c].min_long;   // negative: "where you would pick 64"
    if (cand[c].slab > 0) o.slab_width = cand[c].slab;
    return o;
  };
  int best = -1, last = -1;
  float best_ms = 0.f;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto cleanup = [&]() {
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  };
  for (int c = 0; c < n_cand; ++c) {
    const sagnn_spmm_options o = options_of(c);
    int rc = spmm_csr_prepare_opt(d_rowptr, d_colidx, d_val, m, k, nnz, f, d_ws, ws_bytes, &o, stream);
    if (rc != SAGNN_OK) { cleanup(); return rc; }
    last = c;
    SpmmHostDesc desc{};
    if (!spmm_desc_get(d_ws, &desc) || desc.mode != 1) {
      if (c > 0) continue;   // (a higher threshold may leave too few long rows; the plans timed so far stay)
      best = c;              // nothing to tune
      break;
    }
    if (!e0) {
      hipError_t e = hipEventCreate(&e0);
      if (e == hipSuccess) e = hipEventCreate(&e1);
      if (e != hipSuccess) { set_hip_error(e); cleanup(); return SAGNN_EHIP; }
    }
    float ms_min = 0.f;
    for (int rep = 0; rep < 6; ++rep) {   // the first run warms the caches and is not counted
      hipError_t e = hipEventRecord(e0, s);
      if (e != hipSuccess) { set_hip_error(e); cleanup(); return SAGNN_EHIP; }
      rc = launch_spmm(d_rowptr, d_colidx, d_val, m, k, nnz, d_B, ldb, f, d_C, ldc, 0, d_ws, ws_bytes, s);
      if (rc != SAGNN_OK) { cleanup(); return rc; }
      float ms = 0.f;
      e = hipEventRecord(e1, s);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (e != hipSuccess) { set_hip_error(e); cleanup(); return SAGNN_EHIP; }
      if (rep == 1 || (rep > 1 && ms < ms_min)) ms_min = ms;
    }
    // a variant has to beat the default plan by more than the run-to-run noise of the timing
    if (best < 0 || ms_min < (best == 0 ? 0.985f * best_ms : best_ms)) { best = c; best_ms = ms_min; }
  }
  if (best != last) {
    const sagnn_spmm_options o = options_of(best);
    int rc = spmm_csr_prepare_opt(d_rowptr, d_colidx, d_val, m, k, nnz, f, d_ws, ws_bytes, &o, stream);
    if (rc != SAGNN_OK) { cleanup(); return rc; }
  }
  // Pacing of the sweep (see sweep_pace_until): lay the kept plan out with intervals and search
  // the time per stream step that makes the product fastest.  Upper end: the whole free-running
  // call time spread over the schedule of the generations of wavefronts; the useful values lie
  // below it, because a paced sweep misses less in L2.  Below some value the wavefronts cannot
  // keep to the schedule and the product falls back to its free-running time, so the search
  // walks down and stops there.  If pacing does not pay, the plain layout is restored.
  {
    SpmmHostDesc desc{};
    // only on request (pace_ps_per_step = -2): on the configurations measured so far the search costs
    // seventy products and has found at most 1.5 %
    const bool wanted = h_opt && h_opt->pace_ps_per_step == -2 && h_opt->barriers != 1 && h_opt->sync_slabs >= 0;
    if (wanted && spmm_desc_get(d_ws, &desc) && desc.mode == 1 && (desc.groups == 2 || desc.groups == 4) &&
        best_ms > 0.f) {
      sagnn_spmm_options o = options_of(best);
      if (o.sync_slabs == 0) o.sync_slabs = 16;
      int rc = spmm_csr_prepare_opt(d_rowptr, d_colidx, d_val, m, k, nnz, f, d_ws, ws_bytes, &o, stream);
      if (rc != SAGNN_OK) { cleanup(); return rc; }
      int32_t best_pace = 0;
      if (spmm_desc_get(d_ws, &desc) && desc.mode == 1 && desc.n_intervals > 1 && desc.mean_steps > 0.f) {
        int dev = 0, cus = 256;
        if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        const int32_t fw = sweep_widest_launch(f, desc.max_slab);
        const int64_t resident = (int64_t)cus * lds_resident_workgroups((size_t)4 * desc.slots * fw * 4) * 4;
        const double gens = (double)ceil_div(desc.n_waves, resident > 0 ? resident : 1);
        const double ps_hi = (double)best_ms * 1e9 / (gens * (double)desc.mean_steps);
        float paced_best = 0.f, prev = 0.f;
        for (int step = 0; step < 14; ++step) {
          desc.pace_ps_per_step = (int32_t)(ps_hi * (0.96 - 0.04 * step));
          spmm_desc_put(d_ws, desc);
          float ms_min = 0.f;
          for (int rep = 0; rep < 5; ++rep) {
            hipError_t e = hipEventRecord(e0, s);
            if (e != hipSuccess) { set_hip_error(e); cleanup(); return SAGNN_EHIP; }
            rc = launch_spmm(d_rowptr, d_colidx, d_val, m, k, nnz, d_B, ldb, f, d_C, ldc, 0, d_ws, ws_bytes, s);
            if (rc != SAGNN_OK) { cleanup(); return rc; }
            float ms = 0.f;
            e = hipEventRecord(e1, s);
            if (e == hipSuccess) e = hipEventSynchronize(e1);
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
            if (e != hipSuccess) { set_hip_error(e); cleanup(); return SAGNN_EHIP; }
            if (rep == 1 || (rep > 1 && ms < ms_min)) ms_min = ms;
          }
          if (paced_best == 0.f || ms_min < paced_best) { paced_best = ms_min; best_pace = desc.pace_ps_per_step; }
          if (prev > 0.f && ms_min > 1.08f * prev) break;    // fell off the schedule: slower again
          prev = ms_min;
        }
        if (paced_best > 0.f && paced_best < 0.985f * best_ms) {
          best_ms = paced_best;
          // one step above the fastest value: a margin against run-to-run variation of the point
          // where the wavefronts stop keeping up
          desc.pace_ps_per_step = best_pace + (int32_t)(ps_hi * 0.02);
          spmm_desc_put(d_ws, desc);
        } else {
          best_pace = 0;
        }
      }
      if (best_pace == 0) {   // restore the layout without intervals
        const sagnn_spmm_options o2 = options_of(best);
        rc = spmm_csr_prepare_opt(d_rowptr, d_colidx, d_val, m, k, nnz, f, d_ws, ws_bytes, &o2, stream);
        if (rc != SAGNN_OK) { cleanup(); return rc; }
      }
    }
  }
  cleanup();
  if (h_choice) {
    h_choice[0] = cand[best].piece;
    h_choice[1] = cand[best].min_long;
    h_choice[2] = (int32_t)(best_ms * 1000.f);
    h_choice[3] = best;
  }
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_schedule_info(const void* d_ws, int64_t* h_info) {
  using namespace sagnn;
  if (!d_ws || !h_info) return SAGNN_EINVAL;
  SpmmHostDesc d{};
  if (!spmm_desc_get(d_ws, &d)) return SAGNN_EINVAL;
  h_info[0] = d.mode;
  h_info[1] = d.n_waves;
  h_info[2] = d.nnz - (d.mode == 1 ? d.c_nnz : d.nnz);   // entries in the slab-sweep streams
  h_info[3] = d.c_rows;
  h_info[4] = d.c_nnz;
  h_info[5] = d.c_nchunks;
  h_info[6] = d.n_multi_rows;
  h_info[7] = d.has_empty_rows;
  h_info[8] = d.mode == 1 ? d.n_intervals : 0;
  h_info[9] = d.mode == 1 ? d.sync_slabs : 0;
  // byte offset, inside the workspace, of the 32-bit flag the sweep kernels set when a barrier
  // wait ran into its time limit during the most recent product (0 = all barriers were met)
  h_info[10] = (int64_t)(spmm_ws_layout(d.m, d.nnz, d.f).barrier + sizeof(uint32_t) * kSweepBarrierSlots);
  h_info[11] = d.groups;
  h_info[12] = d.mode == 1 ? d.pace_ps_per_step : 0;
  h_info[13] = d.mode == 1 ? d.barriers : 0;
  h_info[14] = d.mode == 1 ? d.slots : 0;
  h_info[15] = d.mode == 1 ? (int64_t)d.max_steps : 0;
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_launch_info(const void* d_ws, int64_t* h_info) {
  using namespace sagnn;
  if (!d_ws || !h_info) return SAGNN_EINVAL;
  SpmmHostDesc d{};
  if (!spmm_desc_get(d_ws, &d)) return SAGNN_EINVAL;
  const bool swept = d.mode == 1;
  h_info[0] = swept ? d.col_slab : 0;
  h_info[1] = swept ? d.launch_waves : 0;
  h_info[2] = swept ? d.fused_waves : 0;
  h_info[3] = swept ? d.n_slabs : 0;
  return SAGNN_OK;
}

SAGNN_EXPORT int spmm_csr_tallskinny(const int32_t* d_rowptr, const int32_t* d_colidx,
                                     const float* d_val, int64_t m, int64_t k, int64_t nnz,
                                     const float* d_B, int64_t ldb, int32_t f, float* d_C,
                                     int64_t ldc, int32_t accumulate, void* d_ws, size_t ws_bytes,
                                     void* stream) {
  return sagnn::launch_spmm(d_rowptr, d_colidx, d_val, m, k, nnz, d_B, ldb, f, d_C, ldc,
                            accumulate, d_ws, ws_bytes, (hipStream_t)stream);
}
