// Nonzero-splitting schedule of the local SpMM, C (+)= A * B (Alg. 1 / Alg. 2, "Z <- Z + SpMM(A_iq, H^)"):
// chunk tables (built once per matrix), product kernel, carry fix-up.
//
// The entries are cut into chunks of about T consecutive entries, T = 16 .. 128 chosen so that the chip is full
// (spmm_chunk_entries).  A chunk ends at the row end nearest behind the multiple of T where there is one within 16
// entries (32 where T is 16), so that only rows that are long against T are shared by several chunks; the shares of such
// a row go to carry slots that a second kernel adds in chunk order (reproducible, no floating-point atomics), and a
// matrix without such rows needs no second kernel.
//
// Product kernel.  A group of LPE lanes (4, 8, .. 64: as many as hold a row of up to 4 LPE floats, 16 bytes a lane)
// walks one chunk, so one load instruction serves 64 / LPE entries.  Column ids and values of 16 or 32 entries arrive
// with one load each, spread over the lanes of a DPP unit (a quad below 16 lanes per entry, a row of 16 above), and are
// handed to the whole group by DPP broadcasts that ride on the instructions that use them: per entry and
// group one add for the address, one load, four multiply-adds (and at narrow widths four adds per batch: see FOLD).
// Bound by: the latency of its dependent loads on small matrices (chunk, columns, rows of B: hence the short
// chunks), by what the L2s do not hold of B on large ones (7.5 TB/s behind the L2s whatever the row length).
// The kernels it replaces took 256 entries per wavefront, eight at a time: 30 k rows x 12 entries, f = 100: 64 -> 28 us;
// 4 k x 8, f = 256: 29 -> 15 us.
#include "common.h"
#include "rowload.h"

namespace sagnn {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
typedef float vec4 __attribute__((ext_vector_type(4)));

struct FlatDims {
  int64_t m, nnz, nchunks, ldb, ldc, carry_ld;   // m, nnz: of the CSR being walked
  uint64_t generation;
  uint32_t b_bytes, row_bytes, kmax;
  int32_t f, accumulate;
  int32_t blocks, window;             // workgroups (of a part), those that are shared out among the XCDs at a time (0: in turn)
  int32_t parts, part_cols;           // PARTS: column parts, a share of the XCDs each, and their columns
};

// (no short cuts: all fields are read at once instead of one after the other)
__device__ __forceinline__ bool ws_matches(const SpmmWsHeader* __restrict__ hdr, const FlatDims& d) {
  const uint32_t magic = hdr->magic;
  const uint64_t generation = hdr->generation;
  const int64_t rows = hdr->c_rows, nnz = hdr->c_nnz, nchunks = hdr->c_nchunks;
  return (magic == kSpmmMagic) & (generation == d.generation) & (rows == d.m) & (nnz == d.nnz) & (nchunks == d.nchunks);
}

// value of lane S of the DPP unit (quad or row of 16) in all its lanes
template <bool QUAD, int S>
__device__ __forceinline__ uint32_t unit_bcast(uint32_t x) {
  constexpr int ctrl = QUAD ? S * 0x55 : 0x150 + S;   // quad_perm:[S,S,S,S] / row_newbcast:S
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, true);
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

#define FLAT_PTR_PARAMS                                                                                          \
  const int32_t *__restrict__ colidx, const float *__restrict__ val, const float *__restrict__ B,                \
      float *__restrict__ C, const SpmmWsHeader *__restrict__ hdr, const int4 *__restrict__ chunks,              \
      const uint32_t *__restrict__ flags, float *__restrict__ carry, const int32_t *__restrict__ rowmap

// NC: entries a lane holds of a span (2 above quads; 8 in quads, so that whole lines of the entry arrays are used up
// at once -- with 4 the lines are out of the L1 again before their second half is needed, 670 against 587 us on
// 50 M entries at f = 16 -- or 4 where the chunks are shorter than such a span)
// FOLD > 0: two-level sums, the entries of a batch of eight in FOLD sums of their own, then the batches.  For the widths
// at which a row's entries used to be spread over several lane groups and added as a tree: one sum in stored order was
// further from exact there, by 50 % at f = 16 and rows of 60 entries (1.09e-7 against 7.2e-8 in the 2-norm, now 7.3e-8), by
// 11 % at f = 48 and rows of 12 (6.4e-8, 5.8e-8, 5.7e-8).  Costs registers and four additions per batch; the widths of whole
// lane groups were always one sum and stay one (folded at f = 128: stage loop of a rank 431 -> 440 us, six wavefronts
// per SIMD instead of seven).  30 k rows x 12, training 140.0 -> 140.3 us; 1 M x 50, f = 16, training 2278 -> 2286;
// 4 k rows x 8, f = 16, this kernel 10.5 -> 11.2.  One sum per batch at f <= 16: 10.8 us, but 7.6e-8 on the rows of 60; four
// sums through the whole row: 11.4 us and 7.5e-8.
// PARTS: column parts (see flat_launch; in kernels of their own, the others' were 2 to 4 % slower with them, 30 k x 12, f = 64
// 14.9 and 15.3 us).
template <int LPE, int NC, int FOLD, bool PARTS, bool BUF>
__global__ __launch_bounds__(kBlock) void spmm_flat_kernel(FLAT_PTR_PARAMS, const FlatDims d) {
  constexpr bool QUAD = LPE < 16;
  constexpr int R = 64 / LPE;                // groups (chunks) per wavefront
  constexpr int UNIT = QUAD ? 4 : 16;        // lanes of a DPP unit
  constexpr int SPAN = UNIT * NC;            // entries per fetch of column ids and values
  constexpr int U = 8;                       // rows of B in flight
  const int lane = threadIdx.x & 63;
  const int lig = lane % LPE, sub = lane % UNIT;
  // (workgroups go to the eight XCDs in turn; of each window of them an XCD takes a run of the chunks, see flat_launch)
  int32_t col0 = 0, width = d.f, first = 0, block;
  if constexpr (PARTS) {
    const int32_t xcd = blockIdx.x & 7, i = blockIdx.x >> 3, each = 8 / d.parts, rounds = d.window / each;   // each: XCDs of a part
    col0 = xcd / each * d.part_cols;
    width = d.f - col0 < d.part_cols ? d.f - col0 : d.part_cols;
    const int32_t all = (d.blocks + each - 1) / each;
    if (rounds < all) first = i / rounds * rounds;
    const int32_t n = all - first < rounds ? all - first : rounds;
    block = first * each + xcd % each * n + (i - first);
    if (block >= d.blocks) return;
  } else {
    block = blockIdx.x;
    if (d.window > 0) {
      if (d.window < d.blocks) first = block / d.window * d.window;
      const int32_t n = d.blocks - first < d.window ? d.blocks - first : d.window, i = block - first, xcd = i & 7;
      block = first + xcd * (n >> 3) + (xcd < (n & 7) ? xcd : n & 7) + (i >> 3);
    }
  }
  const bool active = lig * 4 < width;
  const uint32_t loff = active ? lig * 16 : 0;     // (idle lanes read the row's first piece again)
  const int64_t wave = __builtin_amdgcn_readfirstlane((int)(((int64_t)block * kBlock + threadIdx.x) >> 6));
  if (wave * R >= d.nchunks) return;
  const int32_t k = (int32_t)(wave * R) + lane / LPE;
  // (the header is looked at beside the chunk, not before it: a trip to memory less in a chain of four)
  const int4 ch = chunks[k < d.nchunks ? k : d.nchunks - 1];
  const bool ours = ws_matches(hdr, d) & (k < d.nchunks);
  int32_t e0 = ch.x, e1 = ours ? ch.y : ch.x, r = ch.z;
  bool head = ch.w & 1;
  // (nothing below trusts the tables: entries stay inside [0, nnz), rows inside [0, m))
  e0 = e0 < 0 ? 0 : e0;
  e1 = e1 > d.nnz ? (int32_t)d.nnz : e1;
  const int32_t len = e1 > e0 ? e1 - e0 : 0;
  int longest = len;
#pragma unroll
  for (int o = LPE; o < 64; o <<= 1) {
    const int t = __shfl_xor(longest, o, 64);
    longest = t > longest ? t : longest;
  }
  longest = __builtin_amdgcn_readfirstlane(longest);
  const int32_t elast = len > 0 ? e1 - 1 : 0;
  const int32_t rmax = (int32_t)(d.m - 1);
  auto row_at = [&](int32_t i) {
    const int32_t ii = i < 0 ? 0 : (i > rmax ? rmax : i);
    return rowmap ? rowmap[ii] : ii;
  };
  int32_t rid = row_at(r);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(B + col0, d.b_bytes - (PARTS ? (uint32_t)col0 * 4u : 0u));
  const float* __restrict__ Bl = B + col0 + (active ? lig * 4 : 0);

  vec4 acc = 0.f, part[2] = {0.f, 0.f};   // the row's sum up to this batch, and in this batch
  auto fold = [&]() {
    if constexpr (FOLD == 1) acc += part[0];
    if constexpr (FOLD == 2) acc += part[0] + part[1];
    part[0] = part[1] = 0.f;
  };
  auto emit = [&]() {   // the row that ends (or is cut) here
    fold();
    if (active && r <= rmax) {
      if (head) {
        *reinterpret_cast<vec4*>(carry + (k * d.carry_ld + col0 + lig * 4)) = acc;
      } else {
        vec4* p = reinterpret_cast<vec4*>(C + (rid * d.ldc + col0 + lig * 4));
        if (d.accumulate) acc += *p;
        *p = acc;
      }
    }
    head = false;
    acc = 0.f;
    ++r;
    rid = row_at(r);
  };

  // column ids, values and row ends of a span; those of the next one are requested before this one is worked on
  uint32_t c[NC], cn[NC];
  float v[NC], vn[NC];
  uint64_t f2 = 0, f2n = 0;
  auto fetch = [&](int base, uint32_t (&ci)[NC], float (&vi)[NC], uint64_t& fw) {
    const int32_t mine = e0 + base + sub * NC;
    // all groups have a whole span left: vector loads
    if (__ballot(base + SPAN <= len) == ~0ull) {
      constexpr int W = NC < 4 ? NC : 4;
      struct __attribute__((packed, aligned(4))) iv { int32_t x[W]; };
      struct __attribute__((packed, aligned(4))) fv { float x[W]; };
#pragma unroll
      for (int q = 0; q < NC / W; ++q) {
        const iv ii = *reinterpret_cast<const iv*>(colidx + mine + q * W);
        const fv ff = *reinterpret_cast<const fv*>(val + mine + q * W);
#pragma unroll
        for (int i = 0; i < W; ++i) {
          ci[q * W + i] = (uint32_t)ii.x[i];
          vi[q * W + i] = ff.x[i];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const bool in = mine + i < e1 && len > 0;
        const int32_t ee = in ? mine + i : elast;
        ci[i] = (uint32_t)colidx[ee];
        vi[i] = in ? val[ee] : 0.f;
      }
    }
    const int32_t fb = e0 + base < elast ? e0 + base : elast;   // (the flags array has two words of slack behind it)
    fw = (uint64_t)flags[fb >> 5] | ((uint64_t)flags[(fb >> 5) + 1] << 32);
  };
  if (longest > 0) fetch(0, c, v, f2);

  for (int base = 0; base < longest; base += SPAN) {
    if (base + SPAN < longest) fetch(base + SPAN, cn, vn, f2n);
    // row ends among the span's entries of this group.  The chunk's last entry counts as one: a row that continues in
    // the next chunk hands over its share there, before the steps that only longer groups need (they multiply the last
    // column's row by 0, which is no 0 where that row holds an infinity or NaN)
    const int32_t fb = e0 + base < elast ? e0 + base : elast;
    uint32_t fl = (uint32_t)(f2 >> (fb & 31));
    const int left = len - base;
    if (left <= 32) fl = left > 0 ? (fl & ((2u << (left - 1)) - 1u)) | (1u << (left - 1)) : 0u;
    uint32_t off[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      c[i] = c[i] > d.kmax ? d.kmax : c[i];
      off[i] = BUF ? c[i] * d.row_bytes : 0u;
    }
    // bit s of `any`: some group's row ends at step s (lane j of a unit stands for its entries NC j .. NC j + NC - 1)
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      uint64_t b = __ballot((fl >> (sub * NC + i)) & 1u);
      b |= b >> 32;
      b |= b >> 16;
      if constexpr (QUAD) {
        b |= b >> 8;
        b |= b >> 4;
        // four bits, one per lane of the quad: spread to steps 0, NC, 2 NC, 3 NC
        const uint32_t q = (uint32_t)b & 0xFu;
        any |= ((q & 1u) | ((q & 2u) << (NC - 1)) | ((q & 4u) << (2 * NC - 2)) | ((q & 8u) << (3 * NC - 3))) << i;
      } else {
        uint32_t q = (uint32_t)b & 0xFFFFu;               // sixteen bits, spread to every other step
        q = (q | (q << 8)) & 0x00FF00FFu;
        q = (q | (q << 4)) & 0x0F0F0F0Fu;
        q = (q | (q << 2)) & 0x33333333u;
        q = (q | (q << 1)) & 0x55555555u;
        any |= q << i;
      }
    }
    any = (uint32_t)__builtin_amdgcn_readfirstlane((int)any);
    const int steps = longest - base;
    static_for<0, SPAN / U>([&](auto ib) {
      constexpr int s0 = decltype(ib)::value * U;
      if (s0 >= steps) return;
      vec4 h[U];
      static_for<0, U>([&](auto iu) {
        constexpr int s = s0 + decltype(iu)::value;
        if constexpr (BUF) {
          const uint32_t o = unit_bcast<QUAD, s / NC>(off[s % NC]) + loff;
          h[s - s0] = __builtin_bit_cast(vec4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
        } else {
          const uint32_t col = unit_bcast<QUAD, s / NC>(c[s % NC]);
          h[s - s0] = *reinterpret_cast<const vec4*>(Bl + (int64_t)col * d.ldb);
        }
      });
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(h[u]));
      static_for<0, U>([&](auto iu) {
        constexpr int s = s0 + decltype(iu)::value;
        const float vs = __builtin_bit_cast(float, unit_bcast<QUAD, s / NC>(__builtin_bit_cast(uint32_t, v[s % NC])));
        if constexpr (FOLD == 0) acc += vs * h[s - s0];
        else part[s % FOLD] += vs * h[s - s0];
        if ((any >> s) & 1u) {
          asm volatile("");   // (a scalar branch first: the two tests are not to be merged)
          if ((fl >> s) & 1u) emit();
        }
      });
      fold();
    });
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      c[i] = cn[i];
      v[i] = vn[i];
    }
    f2 = f2n;
  }
}

// Carries: a chunk that starts inside a row leaves its share of that row in its carry slot.  The chunks of a row
// that do so follow each other; the list holds the first one of every such row.  Up to kFixWave chunks are added by
// one wavefront, more (hub rows) by a workgroup; fixed order either way.
constexpr int kFixWave = 32;

struct FixDims {
  int64_t nchunks, m, ldc, carry_ld;
  uint64_t generation;
  int32_t f_total;
};

template <bool WG>
__device__ __forceinline__ void fix_row(bool ours, const int4* __restrict__ chunks, const int2* __restrict__ list, int64_t q, int64_t n_list,
                                        const float* __restrict__ carry, const int32_t* __restrict__ rowmap, float* __restrict__ C,
                                        const FixDims& d, float4 (*part)[64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (q >= n_list) return;                                   // (WG: the whole workgroup)
  const int2 it = list[q];                                   // first chunk, number of chunks
  const int64_t k = it.x;
  int64_t cnt = it.y;
  if (!ours || k < 0 || cnt <= 0 || k + cnt > d.nchunks) return;
  const int32_t R = chunks[k].z;
  if (R < 0 || R >= d.m) return;
  const int64_t ro = rowmap ? rowmap[R] : R;
  // share of this wavefront
  const int64_t per = WG ? (cnt + kWaves - 1) / kWaves : cnt;
  const int64_t a = WG ? wave * per : 0, b = a + per < cnt ? a + per : cnt;
  for (int c0 = 0; c0 < d.f_total; c0 += 256) {
    const int c4 = c0 + lane * 4;
    const bool on = c4 < d.f_total;
    float4 s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (on) {
      const float* p = carry + (k + a) * d.carry_ld + c4;
      int64_t j = a;
      for (; j + 8 <= b; j += 8, p += 8 * d.carry_ld) {
        float4 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = *reinterpret_cast<const float4*>(p + u * d.carry_ld);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          s[u & 3].x += t[u].x; s[u & 3].y += t[u].y; s[u & 3].z += t[u].z; s[u & 3].w += t[u].w;
        }
      }
      for (; j < b; ++j, p += d.carry_ld) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        s[0].x += t.x; s[0].y += t.y; s[0].z += t.z; s[0].w += t.w;
      }
    }
    float4 t;
    t.x = (s[0].x + s[1].x) + (s[2].x + s[3].x);
    t.y = (s[0].y + s[1].y) + (s[2].y + s[3].y);
    t.z = (s[0].z + s[1].z) + (s[2].z + s[3].z);
    t.w = (s[0].w + s[1].w) + (s[2].w + s[3].w);
    if constexpr (WG) {
      __syncthreads();
      part[wave][lane] = t;
      __syncthreads();
      if (wave != 0) continue;
      for (int w = 1; w < kWaves; ++w) {
        const float4 o = part[w][lane];
        t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
      }
    }
    if (on) {
      float4* p = reinterpret_cast<float4*>(C + ro * d.ldc + c4);
      float4 o = *p;
      o.x += t.x; o.y += t.y; o.z += t.z; o.w += t.w;
      *p = o;
    }
  }
}

// one launch: the hub rows' workgroups come first, their chain is the longest (two launches before: 2.4 M entries,
// 170 k rows, f = 256: 9.2 + 5.6 us, now 9.2)
__global__ __launch_bounds__(kBlock) void flat_fixup_kernel(const SpmmWsHeader* __restrict__ hdr, const int4* __restrict__ chunks,
                                                            const int2* __restrict__ list, int64_t n_list,
                                                            const int2* __restrict__ big, int64_t n_big,
                                                            const float* __restrict__ carry, const int32_t* __restrict__ rowmap,
                                                            float* __restrict__ C, const FixDims d) {
  __shared__ float4 part[kWaves][64];
  const uint32_t magic = hdr->magic;
  const uint64_t generation = hdr->generation;
  const int64_t nchunks = hdr->c_nchunks;
  const bool ours = (magic == kSpmmMagic) & (generation == d.generation) & (nchunks == d.nchunks);
  const int64_t b = blockIdx.x;
  if (b < n_big) fix_row<true>(ours, chunks, big, b, n_big, carry, rowmap, C, d, part);
  else fix_row<false>(ours, chunks, list, (b - n_big) * kWaves + (threadIdx.x >> 6), n_list, carry, rowmap, C, d, part);
}

// ------------------------------------------------------------------------------------------
// tables
__global__ __launch_bounds__(kBlock) void flat_clear_kernel(uint32_t* __restrict__ flags, int64_t words,
                                                            int32_t* __restrict__ stat) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < words; i += stride) flags[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 4) stat[threadIdx.x] = 0;
}

// flags: one bit per entry that ends a row; stat[0] = 1 if some row has no entries
__global__ __launch_bounds__(kBlock) void flat_rowend_kernel(const int32_t* __restrict__ rowptr, int64_t m, int64_t nnz,
                                                             uint32_t* __restrict__ flags, int32_t* __restrict__ stat) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < m; r += stride) {
    const int64_t b = rowptr[r], e = rowptr[r + 1];
    if (e > b && e <= nnz && e >= 1) atomicOr(&flags[(e - 1) >> 5], 1u << ((e - 1) & 31));
    else if (e == b) stat[0] = 1;
  }
}

// How far a boundary may move: the longest chunk of a wavefront's groups decides when it is done, so long chunks are
// not allowed to differ by much (T / 2 at T = 128 cost 20 % at f = 16).  On small matrices (T = 16) the second kernel that
// a cut row asks for weighs more, and rows of up to 33 entries
// stay whole (30 k rows x 12, training step with four products: 151 -> 141 us; 4 k rows, step: 44 -> 41; slack 8 before).
__device__ __forceinline__ int64_t cut_slack(int64_t T) { return T <= 16 ? 32 : 16; }

struct Cut { int64_t at, row; bool head; };   // a chunk boundary: entry, row it lies in, whether it cuts that row

__device__ __forceinline__ Cut chunk_cut(const int32_t* __restrict__ rowptr, int64_t m, int64_t nnz, int64_t T, int64_t k) {
  Cut c{};
  const int64_t target = k * T;
  if (target >= nnz) return Cut{nnz, m, false};
  int64_t lo = 0, hi = m;                     // last row r with rowptr[r] <= target (the row that holds it)
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)rowptr[mid] <= target) lo = mid; else hi = mid;
  }
  const int64_t b = rowptr[lo], e = rowptr[lo + 1];
  if (b == target) return Cut{target, lo, false};
  if (e > target && e <= nnz && e - target <= cut_slack(T)) {   // the row ends soon: the boundary moves behind it
    // (the next row with entries starts there; rows without entries in between are stepped over)
    int64_t r = lo + 1;
    while (r < m - 1 && rowptr[r + 1] == rowptr[r]) ++r;
    return Cut{e, r, false};
  }
  return Cut{target, lo, b < target};
}

// chunks[k] = {first entry, end, first row, 1 if the chunk starts inside a row}; rows whose later shares are carries
// are appended to the lists (list order does not matter: every row has one writer)
__global__ __launch_bounds__(kBlock) void flat_chunks_kernel(const int32_t* __restrict__ rowptr, int64_t m, int64_t nnz,
                                                             int64_t T, int64_t nchunks, int4* __restrict__ chunks,
                                                             int2* __restrict__ list, int64_t list_cap,
                                                             int32_t* __restrict__ stat) {
  const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (k >= nchunks) return;
  const Cut a = chunk_cut(rowptr, m, nnz, T, k), b = chunk_cut(rowptr, m, nnz, T, k + 1);
  chunks[k] = make_int4((int32_t)a.at, (int32_t)b.at, (int32_t)a.row, a.head ? 1 : 0);
  if (!a.head) return;
  // the first carry of its row?
  if (k > 0) {
    const Cut p = chunk_cut(rowptr, m, nnz, T, k - 1);
    if (p.head && p.row == a.row) return;
  }
  int64_t cnt = 1;                            // chunks that start inside the row: multiples of T below its end
  const int64_t e = rowptr[a.row + 1];
  // the last cut inside the row is the largest multiple of T more than the slack before its end
  const int64_t last = (e - cut_slack(T) - 1) / T;
  if (last > k) cnt = last - k + 1;
  if (k + cnt > nchunks) cnt = nchunks - k;
  const bool big = cnt > kFixWave;
  const int32_t at = atomicAdd(&stat[big ? 2 : 1], 1);
  // small ones from the front, big ones from the back
  const int64_t pos = big ? list_cap - 1 - at : at;
  if (pos >= 0 && pos < list_cap) list[pos] = make_int2((int32_t)k, (int32_t)cnt);
}

inline unsigned capped_grid(int64_t blocks) {
  const int64_t cap = 256 * 64;
  return (unsigned)(blocks > cap ? cap : (blocks < 1 ? 1 : blocks));
}

}  // namespace

int flat_build_tables(const int32_t* d_rowptr, int64_t rows, int64_t nnz, int64_t T, char* ws, const SpmmWsLayout& L,
                      int32_t* d_stat, hipStream_t s) {
  const int64_t nchunks = spmm_nchunks(nnz, T);
  uint32_t* flags = reinterpret_cast<uint32_t*>(ws + L.flags);
  const int64_t words = nnz / 32 + 3;
  hipLaunchKernelGGL(flat_clear_kernel, dim3(capped_grid(ceil_div(words, kBlock))), dim3(kBlock), 0, s, flags, words, d_stat);
  SAGNN_LAUNCH_CHECK();
  if (rows > 0) {
    hipLaunchKernelGGL(flat_rowend_kernel, dim3(capped_grid(ceil_div(rows, kBlock))), dim3(kBlock), 0, s, d_rowptr, rows,
                       nnz, flags, d_stat);
    SAGNN_LAUNCH_CHECK();
  }
  if (rows > 0 && nchunks > 0) {
    hipLaunchKernelGGL(flat_chunks_kernel, dim3((unsigned)ceil_div(nchunks, kBlock)), dim3(kBlock), 0, s, d_rowptr, rows,
                       nnz, T, nchunks, reinterpret_cast<int4*>(ws + L.chunks), reinterpret_cast<int2*>(ws + L.fix_list),
                       L.max_chunks, d_stat);
    SAGNN_LAUNCH_CHECK();
  }
  return SAGNN_OK;
}

int flat_launch(const FlatArgs& a, int32_t col0, int32_t fw, hipStream_t s) {
  FlatDims d{};
  d.m = a.rows; d.nnz = a.nnz; d.nchunks = a.nchunks; d.ldb = a.ldb; d.ldc = a.ldc; d.carry_ld = a.carry_ld;
  d.generation = a.generation; d.kmax = a.kmax; d.f = fw; d.accumulate = a.accumulate;
  d.row_bytes = (uint32_t)(a.ldb * 4);
  const bool buf = buffer_addressable(a.kmax, a.ldb, fw, &d.b_bytes);
  d.parts = 1;
  const int64_t b_rows = (int64_t)a.kmax + 1;
  auto go = [&](auto kern, int lpe) -> int {
    const int64_t waves = ceil_div(a.nchunks, 64 / lpe);
    d.blocks = (int32_t)ceil_div(waves, kWaves);
    const int64_t grid = d.parts > 1 ? 8 * ceil_div(d.blocks, 8 / d.parts) : d.blocks;
    // An XCD takes a run of neighbouring chunks, so that where neighbouring rows want the same rows of B its L2 is asked for
    // an eighth of them; where they do not nothing changes.  At most as many at a time as the memory-side cache holds the rows
    // of, and in turn from 1200 MB on, where that is less than two neighbourhoods (one run, such runs: 1 M vertices of 6, f = 256
    // in turn 959, 1000, 957; 2 M, f = 128, 192, 256 989, 1451, 1945 and 976, 1462, 1976).  us in turn and so, 16 communities:
    // 20 k vertices of 12, f = 64, 128 9.6, 14.6 and 8.0, 13.5; 40 k of 24 f = 100, 192, 256 50, 91, 94 and 33, 50, 72; 100 k of
    // 12 f = 16, 64, 100, 256 20, 50, 85, 165 and 16, 28, 45, 138; 300 k of 8 f = 64, 128, 256 111, 200, 378 and 83, 163, 347;
    // random and power-law columns within 2 %.  And in turn where a row of B is hardly used twice (a rank's stage loop of
    // 190 k rows, eight blocks of 2 entries a row, f = 100, 128 515, 525 us in runs, 509, 526 in turn).
    const double bytes = (double)a.rows * fw * 4.0;
    d.window = d.blocks + 64;
    if (bytes > 256.0 * (1 << 20)) d.window = (int32_t)std::max(64.0, 256.0 * (1 << 20) / bytes * d.blocks) / 64 * 64;
    if (bytes > 1200.0 * (1 << 20) || a.nnz < 3 * b_rows) d.window = d.parts > 1 ? 8 / d.parts : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kBlock), 0, s, a.colidx, a.val, a.B + col0,
                       a.C + col0, a.hdr, a.chunks, a.flags, a.carry + col0, a.rowmap, d);
    SAGNN_LAUNCH_CHECK();
    return SAGNN_OK;
  };
#define SAGNN_FLAT(LPE_, NC_, FOLD_) \
  (buf ? go(spmm_flat_kernel<LPE_, NC_, FOLD_, false, true>, LPE_) : go(spmm_flat_kernel<LPE_, NC_, FOLD_, false, false>, LPE_))
#define SAGNN_FLAT_PARTS(LPE_) \
  (buf ? go(spmm_flat_kernel<LPE_, 2, 0, true, true>, LPE_) : go(spmm_flat_kernel<LPE_, 2, 0, true, false>, LPE_))
  // Column parts: each on a share of the XCDs, so that an L2 has to hold that share of the rows of B only, and is asked for
  // a line of it that many times as often; the sums are the same.  Parts of whole lines, where rows of B are used ten times or
  // more and B is larger than two L2s, with hubs, whose rows hit in any case, than more than eight.  Four parts without hubs at
  // 256 columns from 12 MB on.  us in runs whole, in two and in four parts:
  // - random columns, f = 128 16 k vertices of 11 (8 MB) 12.8, 12.1, 20 k of 40 48, 38, 60 k of 11 (29 MB) 53, 51; f = 256 10 k
  //   of 16, 40 (10 MB) 22, 45, 18, 33, 17, 31, 12 k of 24 (12 MB) 37, 28, 24, 20 k of 40 103, 85, 62, 50 k of 16 (49 MB) 121, -,
  //   104.
  // - communities, which in runs are better off whole (the launch does not know them); chunks in turn, whole, took longer than
  //   two parts from 8 MB, four from 12 MB on: f = 256 in turn, in two and in four parts 8.2 k of 16 13.6, 13.3, 14.6, 10 k of 40
  //   30, 29.5, 32.6, 12 k of 40 40, 34, 37, 20 k of 16 40, 26, 28; f = 128 16 k of 24 22.9, 21.3.
  // - 192 columns in parts of three lines, 10 to 28 MB: random columns, 14 k of 18 (10 MB) 25, 22, 30 k of 18 (22 MB) 58, 53; not
  //   42 k of 18 (31 MB) 82, 88, 70 k of 14 (51 MB) 115, 118; communities in turn and in two parts 11 k of 24 (8 MB) 21.2, 22.2,
  //   14 k of 24 25.7, 22.7.
  // - hubs, power-law, from 34 MB where rows of B are used 24 times or more, from 48 MB where less, at 192 columns from 64 MB under
  //   16 uses: f = 256 34 k of 24 (33 MB) 62, 63, 39 k of 24, 32 (38 MB) 72, 87, 70, 83, of 11, 14 42, 48, 44, 50, 52 k of 11 (51 MB)
  //   58, 54; f = 192 48 k of 24, 32 (35 MB) 69, 84, 65, 78, 62 k of 14 (45 MB) 61, 63, 75 k of 11, 14, 17 (55 MB) 64, 72, 86, 65, 72,
  //   79, 90 k of 11, 14 (66 MB) 76, 89, 75, 84; f = 128 30 k of 14 (15 MB) 25, 27, 62 k of 30 (30 MB) 71, 72, 78 k of 30 (38 MB) 90,
  //   86, 98 k of 11, 14 (48 MB) 59, 66, 56, 63; 170 k of 14 f = 128, 192, 256 (to 174 MB) 122, 193, 256, 111, 166, 231.
  // - not: 10 k random columns of 12 f = 128 (5 MB) 8.7, 8.3, 200 k of 4 f = 128 78, 81; in narrower parts 60 k of 12, f = 64 31, 30,
  //   170 k 64, 76; in parts of 13 lines or less that begin inside one, 30 k of 12 f = 100 27, 31.
  const bool lines = (a.ldb & 31) == 0 && (reinterpret_cast<uintptr_t>(a.B + col0) & 127) == 0;
  const int64_t mb = b_rows * fw * 4 >> 20;
  const int64_t from = !a.hubs ? (fw == 192 ? 10 : 8) : (a.nnz >= 24 * b_rows ? 34 : (fw == 192 && a.nnz < 16 * b_rows ? 64 : 48));
  const bool large = fw == 192 && !a.hubs && mb >= 28;
  if (fw >= 128 && (fw & 63) == 0 && lines && a.nnz >= 10 * b_rows && mb >= from && !large) {
    d.parts = fw == 256 && !a.hubs && mb >= 12 ? 4 : 2;
    d.part_cols = fw / d.parts;
    return d.part_cols <= 64 ? SAGNN_FLAT_PARTS(16) : SAGNN_FLAT_PARTS(32);
  }
  const bool brief = a.nnz < 64 * a.nchunks;
  // Up to 32 columns four groups of sixteen lanes a wavefront, most of them idle, where groups as narrow as a row would leave
  // SIMDs without a wavefront: with sixteen groups some row ends at nearly every step, and its wavefront stores what the
  // others wait for.  us of the kernel alone, f = 16, 32: 1 k rows of 8 8.7, 7.2 -> 5.9, 5.8; 4 k of 8 9.4, 7.5 -> 6.3, 6.1; 15 k of
  // 16 9.1, 8.5 -> 8.8, 8.8, 20 k of 12 9.8, 8.9 -> 8.8, 8.8 (both 15000 chunks); 5 k power-law rows of 19 11.6, 9.4 -> 8.3, 8.1;
  // beyond the line 20 k of 20 10.5, 11.4 and 12.9, 12.8, 30 k of 12 (22500 chunks) 10.5, 10.6 and 11.0, 11.4, power-law 20 k of 19
  // 12.8, 13.1 and 13.8, 13.8.
  const bool few = a.nchunks <= 16384;
  if (fw <= 16 && few) return SAGNN_FLAT(16, 2, 2);
  if (fw <= 32 && few) return SAGNN_FLAT(16, 2, 1);
  if (fw <= 16) return brief ? SAGNN_FLAT(4, 4, 2) : SAGNN_FLAT(4, 8, 2);
  if (fw <= 32) return brief ? SAGNN_FLAT(8, 4, 1) : SAGNN_FLAT(8, 8, 1);
  if (fw < 64) return SAGNN_FLAT(16, 2, 1);
  if (fw == 64) return SAGNN_FLAT(16, 2, 0);
  if (fw < 128) return SAGNN_FLAT(32, 2, 1);
  if (fw == 128) return SAGNN_FLAT(32, 2, 0);
  return SAGNN_FLAT(64, 2, 0);
#undef SAGNN_FLAT
#undef SAGNN_FLAT_PARTS
}

int flat_fixup(const FlatArgs& a, const int2* list, int64_t list_cap, int64_t n_small, int64_t n_big, int32_t f_total,
               hipStream_t s) {
  FixDims d{};
  d.nchunks = a.nchunks; d.m = a.rows; d.ldc = a.ldc; d.carry_ld = a.carry_ld; d.generation = a.generation;
  d.f_total = f_total;
  if (n_small + n_big <= 0) return SAGNN_OK;
  hipLaunchKernelGGL(flat_fixup_kernel, dim3((unsigned)(n_big + ceil_div(n_small, kWaves))), dim3(kBlock), 0, s, a.hdr, a.chunks,
                     list, n_small, list + (list_cap - n_big), n_big, a.carry, a.rowmap, a.C, d);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

}  // namespace sagnn
