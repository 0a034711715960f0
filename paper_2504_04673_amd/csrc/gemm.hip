// Dense transforms of the GCN layer on the matrix cores (MFMA), gfx950.
//   forward   Z = T W, H' = sigma(Z)                     (Sec. 2.1 forward equations; Alg. 1
//                                                          "H <- GEMM(Z, W)")
//   backward  G' = (S W^T) .* sigma'(Z')                  (Sec. 2.1 backward equation for G)
//             Y  = H'^T S                                  (Sec. 4.1, weight-gradient paragraph)
//
// Tall-skinny shapes: m is 10^5..10^7 rows, the feature widths are <= 256, so W fits in LDS
// and every kernel streams the tall operand from HBM exactly once.
//
// gemm_nn_kernel (gemm_nn.h, one source file per operand mode; Z = X op(W)): a workgroup stages its slab of W in LDS once and then walks
// row tiles persistently; each wavefront owns a 32-row tile and keeps NT 32x32 accumulator
// tiles in registers.  The A operand of the MFMA is read straight from global memory in
// operand layout: the k order inside an MFMA does not matter as long as both operands agree,
// so lane (row r, half h) takes the 16 (fp32) or 32 (bf16) contiguous bytes
// X[r][8j+4h..] / X[r][16j+8h..] and the matching rows of W are picked from LDS.
//   fp32: v_mfma_f32_32x32x2_f32;  bf16: operands rounded RNE, v_mfma_f32_32x32x16_bf16.
//   fp32 operands as three bfloat16 terms: the same bfloat16 instruction six times per product, W kept in
//   LDS as three packed planes, X split in registers (the accuracy of the fp32 instruction at 6/16 of its cost).
// The epilogue applies the optional mask and activation and stores from the accumulator
// layout (row = 8*(v/4) + 4*(lane/32) + v%4, col = lane%32 of each 32x32 tile).
//
// Y = X^T S: the reduction runs over the m rows, cut into slices whose partial results tn_reduce_kernel adds in a
// fixed order (reproducible, no atomics).  gemm_tn_direct_kernel takes its operands straight from memory, for every
// mode; gemm_tn_kernel stages 32 rows of X and S at a time in LDS transposed (k contiguous per column, so an operand is
// one LDS read) and holds a full f_in x f_out partial in registers (8 wavefronts x 2x4 tiles), for rounded operands
// whose result one workgroup of the other does not cover (see tn_staged).
#include <algorithm>
#include <type_traits>

#include "gemm.h"

namespace sagnn {
namespace {

// ------------------------------------------------------------------------------------------
// Y = X^T S.  KB rows per stage; LDS rows padded to KP elements (16-byte multiple).
constexpr int kTnWaves = 8;
constexpr int kTnThreads = kTnWaves * 64;
constexpr int KB = 32, KP = 40;

struct TnArgs {
  const float* X; int64_t ldx;
  const float* S; int64_t lds_;
  int64_t m; int32_t fi, fo;
  int64_t rows_per_wg;
  float* partial;  // [gridDim.x][fi][fo]
};

// operands rounded to bfloat16
__global__ __launch_bounds__(kTnThreads) void gemm_tn_kernel(const TnArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __bf16* Xs = reinterpret_cast<__bf16*>(smem);                    // [fi][KP]
  __bf16* Ss = Xs + (size_t)((g.fi + 31) / 32) * 32 * KP;         // [fo][KP], after the padded X part
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 31, h = lane >> 5;
  const int wa = wave >> 1, wb = wave & 1;  // wave tile: a-tiles {2wa,2wa+1}, b-tiles {4wb..4wb+3}
  const int TA = (g.fi + 31) / 32, TB = (g.fo + 31) / 32;
  // columns of the last tile that lie beyond fi / fo are never staged: keep them zero
  for (int idx = tid; idx < (TA + TB) * 32 * KP; idx += kTnThreads) Xs[idx] = (__bf16)0.f;
  __syncthreads();

  const int64_t r_begin = (int64_t)blockIdx.x * g.rows_per_wg;
  int64_t r_end = r_begin + g.rows_per_wg;
  if (r_end > g.m) r_end = g.m;

  floatx16 acc[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  // staging map: thread -> (column group cg of 4 columns, row pair kp); 64 groups x 8 pairs
  // per pass, two passes cover the KB = 32 rows of a stage
  const int cg = tid & 63, kp = tid >> 6;
  float4 xr[2][2], sr[2][2];
  auto load_stage = [&](int64_t r0) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int64_t row = r0 + (kp + 8 * p) * 2 + q;
        const bool ok = row < r_end;
        xr[p][q] = (ok && cg * 4 < g.fi) ? *reinterpret_cast<const float4*>(g.X + row * g.ldx + cg * 4)
                                         : make_float4(0.f, 0.f, 0.f, 0.f);
        sr[p][q] = (ok && cg * 4 < g.fo) ? *reinterpret_cast<const float4*>(g.S + row * g.lds_ + cg * 4)
                                         : make_float4(0.f, 0.f, 0.f, 0.f);
      }
  };
  // Transposing stores: column col = 4 cg + c of the stage goes to LDS row col, k contiguous, so a lane's two
  // rows (k, k + 1) of one column are one 4-byte store.  (Lanes that store the same c fall on two banks; taking
  // the columns in a rotated order spreads them over eight but lengthens the path from a load to its store, which
  // is what bounds a stage: 1.0 -> 1.2 ms at 2 M x 256 x 256.)
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto store_stage = [&]() {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int kk = (kp + 8 * p) * 2;
      const float xa[4] = {xr[p][0].x, xr[p][0].y, xr[p][0].z, xr[p][0].w};
      const float xb[4] = {xr[p][1].x, xr[p][1].y, xr[p][1].z, xr[p][1].w};
      const float sa[4] = {sr[p][0].x, sr[p][0].y, sr[p][0].z, sr[p][0].w};
      const float sb[4] = {sr[p][1].x, sr[p][1].y, sr[p][1].z, sr[p][1].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int col = cg * 4 + c;
        bf16x2 t;
        if (col < g.fi) {
          t[0] = (__bf16)xa[c]; t[1] = (__bf16)xb[c];
          *reinterpret_cast<bf16x2*>(Xs + col * KP + kk) = t;
        }
        if (col < g.fo) {
          t[0] = (__bf16)sa[c]; t[1] = (__bf16)sb[c];
          *reinterpret_cast<bf16x2*>(Ss + col * KP + kk) = t;
        }
      }
    }
  };

  if (r_begin < r_end) load_stage(r_begin);
  for (int64_t r0 = r_begin; r0 < r_end; r0 += KB) {
    __syncthreads();  // previous stage fully consumed
    store_stage();
    __syncthreads();
    if (r0 + KB < r_end) load_stage(r0 + KB);  // prefetch the next stage into registers
#pragma unroll
      for (int ks = 0; ks < KB / 16; ++ks) {
        bf16x8 av[2], bv[4];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const int ta = 2 * wa + a;
          av[a] = *reinterpret_cast<const bf16x8*>(
              Xs + ((ta < TA ? ta : 0) * 32 + i) * KP + ks * 16 + 8 * h);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int tb = 4 * wb + b;
          bv[b] = *reinterpret_cast<const bf16x8*>(
              Ss + ((tb < TB ? tb : 0) * 32 + i) * KP + ks * 16 + 8 * h);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (2 * wa + a < TA && 4 * wb + b < TB)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a], bv[b], acc[a][b], 0, 0, 0);
      }
  }

  float* __restrict__ P = g.partial + (int64_t)blockIdx.x * g.fi * g.fo;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int ta = 2 * wa + a, tb = 4 * wb + b;
      if (ta >= TA || tb >= TB) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ro = ta * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
        if (ro < g.fi && tb * 32 + i < g.fo) P[(int64_t)ro * g.fo + tb * 32 + i] = acc[a][b][v];
      }
    }
}

// Y = X^T S straight from registers.  In X^T S the reduction index is the row, so the lanes of an operand that
// hold one k hold one row of X: a lane loads V consecutive columns of a row (V = 1 to 4) and register c of
// those loads is the operand of the tile with columns V*i + c, i = 0..15.  No transpose, no LDS in the loop.
//   fp32                    16x16x4: a load brings 4 rows, one per 16 lanes
//   bfloat16, three terms   16x16x32: 8 loads bring 32 rows, lane group q the rows 8q..8q+7, packed in registers
// A wavefront owns a block of up to 64 x 64 of Y and a share of the rows of its workgroup's slice; the shares
// are summed through LDS, the slices by tn_reduce_kernel, both in a fixed order.
// It replaces a form that staged every slab transposed in LDS for all shapes (16 x 16 over 1 M rows took 1 ms:
// the staging work did not shrink with the width); that one is kept where it is faster (see launch_gemm_tn).
typedef float floatx4 __attribute__((ext_vector_type(4)));
// Wavefronts of a workgroup: sixteen where the sums and the rows on their way fit 128 registers, which takes loading the
// next rows into the registers that the matrix instructions have just read: with a second set of them two wavefronts per
// SIMD were resident (160 registers, workgroups of eight), the slices ran in two rounds, and the loads' latency showed.
// fp32, 170 k rows: 128 x 128 69 -> 59 us, 128 x 256 121 -> 113; 60 k x 128 x 128 36 -> 30; 1 M x 128 x 128 322 -> 282.
// (matrix instructions alone 213, reading the operands 213; their rates together are what is left)
constexpr int td_waves(int prec) { return prec == SAGNN_GEMM_FP32 ? 16 : 8; }

template <int V> struct ColVec;
template <> struct ColVec<1> { typedef float T; };
template <> struct ColVec<2> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct ColVec<4> { typedef float T __attribute__((ext_vector_type(4))); };
// three columns: 12 bytes at any multiple of 4 (a vector of three would be read as four)
template <> struct ColVec<3> {
  struct T {
    float v[3];
    __device__ T() {}
    __device__ explicit T(float a) : v{a, a, a} {}
    __device__ float operator[](int c) const { return v[c]; }
  };
};
template <int V>
__device__ __forceinline__ float comp(const typename ColVec<V>::T& v, int c) {
  if constexpr (V == 1) return v;
  else return v[c];
}

template <int PREC, int VA, int VB>
__global__ __launch_bounds__(td_waves(PREC) * 64) void gemm_tn_direct_kernel(const TnArgs g, int nbx, int nbs, int per,
                                                                             int kshare) {
  constexpr int KROWS = PREC == SAGNN_GEMM_FP32 ? 4 : 32;      // rows of one matrix instruction
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using xvec = typename ColVec<VA>::T;
  using svec = typename ColVec<VB>::T;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int i = lane & 15, q = lane >> 4;
  const int nb = nbx * nbs;
  const int first = (int)blockIdx.x * per;
  const int here = nb - first < per ? nb - first : per;             // blocks of Y in this workgroup
  const int blk = first + wave % here, share = wave / here;
  const bool busy = share < kshare;
  const int xb = blk / nbs * (16 * VA), sb = blk % nbs * (16 * VB);
  // a lane whose columns lie past the end reads column 0: its results are not stored
  const int xc = xb + VA * i < g.fi ? xb + VA * i : 0, sc = sb + VB * i < g.fo ? sb + VB * i : 0;
  const int64_t r0 = (int64_t)blockIdx.y * g.rows_per_wg;
  int64_t r_end = r0 + g.rows_per_wg;
  if (r_end > g.m) r_end = g.m;

  floatx4 acc[VA][VB];
#pragma unroll
  for (int a = 0; a < VA; ++a)
#pragma unroll
    for (int b = 0; b < VB; ++b) acc[a][b] = floatx4(0.f);

  if constexpr (PREC == SAGNN_GEMM_FP32) {
    constexpr int U = VA * VB >= 8 ? 4 : 8;                    // instructions' worth of rows in flight
    const int64_t step = (int64_t)kshare * (U * KROWS);
    int64_t r = r0 + (int64_t)share * (U * KROWS);
    const float* xp = g.X + (r + q) * g.ldx + xc;
    const float* sp = g.S + (r + q) * g.lds_ + sc;
    xvec x[U];
    svec s[U];
    // (three columns a lane may reach past a row's end, into the next row: the last row of all is read one by one)
    const int64_t whole = VA == 3 || VB == 3 ? (r_end < g.m ? r_end : g.m - 1) : r_end;
    auto full = [&](int64_t at) { return busy && at + U * KROWS <= whole; };
    auto load = [&](int u) {
      x[u] = *reinterpret_cast<const xvec*>(xp + (int64_t)(u * KROWS) * g.ldx);
      s[u] = *reinterpret_cast<const svec*>(sp + (int64_t)(u * KROWS) * g.lds_);
    };
    auto multiply = [&](int u) {
#pragma unroll
      for (int a = 0; a < VA; ++a)
#pragma unroll
        for (int b = 0; b < VB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp<VA>(x[u], a), comp<VB>(s[u], b), acc[a][b], 0, 0, 0);
    };
    if (full(r)) {
#pragma unroll
      for (int u = 0; u < U; ++u) load(u);
      for (r += step; full(r); r += step) {
        xp += step * g.ldx;
        sp += step * g.lds_;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          multiply(u);
          load(u);                                             // (the next step's rows, into the registers just read)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) multiply(u);
    }
    if (busy)
      for (int u = 0; u < U; ++u) {                            // the rows of the last, partial step
        const int64_t row = r + u * KROWS + q;
        if (r + u * KROWS >= r_end) break;
        xvec xt = xvec(0.f);
        svec st = svec(0.f);
        if (row < r_end) {
          const float* xr = g.X + row * g.ldx + xc;
          const float* sr = g.S + row * g.lds_ + sc;
          if constexpr (VA == 3) {
#pragma unroll
            for (int c = 0; c < 3; ++c) xt.v[c] = xr[xc + c < g.fi ? c : 0];
          } else {
            xt = *reinterpret_cast<const xvec*>(xr);
          }
          if constexpr (VB == 3) {
#pragma unroll
            for (int c = 0; c < 3; ++c) st.v[c] = sr[sc + c < g.fo ? c : 0];
          } else {
            st = *reinterpret_cast<const svec*>(sr);
          }
        }
#pragma unroll
        for (int a = 0; a < VA; ++a)
#pragma unroll
          for (int b = 0; b < VB; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp<VA>(xt, a), comp<VB>(st, b), acc[a][b], 0, 0, 0);
      }
  } else {
    constexpr int T = PREC == SAGNN_GEMM_BF16 ? 1 : 3;         // bfloat16 terms per element
    xvec x[8];
    svec s[8];
    auto load_x = [&](int64_t at) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int64_t row = at + 8 * q + t;
        x[t] = xvec(0.f);
        if (row < r_end) x[t] = *reinterpret_cast<const xvec*>(g.X + row * g.ldx + xc);
      }
    };
    auto load_s = [&](int64_t at) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int64_t row = at + 8 * q + t;
        s[t] = svec(0.f);
        if (row < r_end) s[t] = *reinterpret_cast<const svec*>(g.S + row * g.lds_ + sc);
      }
    };
    const int64_t step = (int64_t)kshare * KROWS;
    int64_t r = r0 + (int64_t)share * KROWS;
    if (busy && r < r_end) {
      load_x(r);
      load_s(r);
    }
    while (busy && r < r_end) {
      // the operands of S are packed first and their registers refilled under the matrix instructions, those of X
      // one column at a time (all at once, with three terms each, do not fit the registers beside the sums)
      bf16x8 sa[VB][T];
#pragma unroll
      for (int b = 0; b < VB; ++b)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          if constexpr (T == 1) {
            sa[b][0][t] = (__bf16)comp<VB>(s[t], b);
          } else {
            __bf16 t1, t2, t3;
            split3(comp<VB>(s[t], b), t1, t2, t3);
            sa[b][0][t] = t1; sa[b][1][t] = t2; sa[b][2][t] = t3;
          }
        }
      r += step;
      // (64 x 64 with three terms: only once half of X has been packed)
      constexpr int refill = T == 3 && VA * VB == 16 ? 2 : 0;
#pragma unroll
      for (int a = 0; a < VA; ++a) {
        if (a == refill && r < r_end) load_s(r);
        bf16x8 xa[T];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          if constexpr (T == 1) {
            xa[0][t] = (__bf16)comp<VA>(x[t], a);
          } else {
            __bf16 t1, t2, t3;
            split3(comp<VA>(x[t], a), t1, t2, t3);
            xa[0][t] = t1; xa[1][t] = t2; xa[2][t] = t3;
          }
        }
        if (a == VA - 1 && r < r_end) load_x(r);
#pragma unroll
        for (int b = 0; b < VB; ++b) {
          floatx4 z = acc[a][b];
          if constexpr (T == 3) {                              // smallest products first
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[2], sa[b][0], z, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[0], sa[b][2], z, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[1], sa[b][1], z, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[1], sa[b][0], z, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[0], sa[b][1], z, 0, 0, 0);
          }
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[0], sa[b][0], z, 0, 0, 0);
        }
        if constexpr (T == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // sum of the shares of a block: the upper half hands its sums to the lower half until one is left
  for (int n = kshare; n > 1;) {
    const int keep = (n + 1) / 2;
    floatx4* slot = reinterpret_cast<floatx4*>(smem) + ((size_t)(share - keep) * here + wave % here) * (VA * VB * 64) + lane;
    if (busy && share >= keep && share < n) {
#pragma unroll
      for (int a = 0; a < VA; ++a)
#pragma unroll
        for (int b = 0; b < VB; ++b) slot[(a * VB + b) * 64] = acc[a][b];
    }
    __syncthreads();
    if (busy && share + keep < n) {
      const floatx4* from = reinterpret_cast<const floatx4*>(smem) + ((size_t)share * here + wave % here) * (VA * VB * 64) + lane;
#pragma unroll
      for (int a = 0; a < VA; ++a)
#pragma unroll
        for (int b = 0; b < VB; ++b) acc[a][b] += from[(a * VB + b) * 64];
    }
    __syncthreads();
    n = keep;
  }
  if (share != 0) return;
  float* __restrict__ P = g.partial + (int64_t)blockIdx.y * g.fi * g.fo;
#pragma unroll
  for (int a = 0; a < VA; ++a)
#pragma unroll
    for (int b = 0; b < VB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ro = xb + VA * (4 * q + v) + a, co = sb + VB * i + b;
        if (ro < g.fi && co < g.fo) P[(int64_t)ro * g.fo + co] = acc[a][b][v];
      }
}

// Y[e] = sum of the slices' partials in a fixed order.  32 elements x 8 groups of slices per workgroup: enough
// loads in flight also for a small Y (one thread per element over 256 slices took 20 us whatever the size).
__global__ __launch_bounds__(256) void tn_reduce_kernel(const float* __restrict__ partial, int32_t nparts, int64_t elems,
                                                        float* __restrict__ Y) {
  __shared__ float red[8][33];
  const int e = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int64_t idx = (int64_t)blockIdx.x * 32 + e;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  if (idx < elems) {
    int p = grp;
    for (; p + 56 < nparts; p += 64) {
      float t[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = partial[(int64_t)(p + 8 * j) * elems + idx];
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j & 3] += t[j];
    }
    for (; p < nparts; p += 8) s[0] += partial[(int64_t)p * elems + idx];
  }
  red[grp][e] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (grp == 0 && idx < elems) {
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) t += red[j][e];
    Y[idx] = t;
  }
}

// Slices of rows, at least 128 rows each: two workgroups per CU, one where a partial result is large.
constexpr int64_t kTnSmall = 16384;   // elements of a result that is not large
inline int64_t tn_parts(int64_t m, int64_t elems) {
  return std::max<int64_t>(1, std::min<int64_t>(elems <= kTnSmall ? 512 : 256, ceil_div(m, 128)));
}
inline size_t tn_partial_bytes(int64_t m, int64_t elems) {
  return round_up(sizeof(float) * (size_t)(tn_parts(m, elems) * elems), 256);
}

// The LDS-staged form reads every row once per workgroup, the direct form once per 64 columns of the other
// operand (through L1 / L2).  With rounded operands, where the matrix instructions are too short to hide that,
// the staged form wins as soon as one workgroup does not cover Y (1 M rows: 462 against 773 us at 256 x 256, 320
// against 534 at 160 x 160, but 296 against 265 at 192 x 96).
inline bool tn_staged(int32_t fi, int32_t fo, int32_t prec) {
  return prec == SAGNN_GEMM_BF16 && ((fi + 63) / 64) * ((fo + 63) / 64) > td_waves(SAGNN_GEMM_BF16);
}

}  // namespace

// enough for narrower operands too: their result may be cut into more slices
size_t gemm_tn_ws_bytes(int64_t m, int32_t fi, int32_t fo) {
  const int64_t elems = (int64_t)fi * fo;
  return std::max(tn_partial_bytes(m, elems), tn_partial_bytes(m, std::min(elems, kTnSmall)));
}

int launch_gemm_tn(const float* X, int64_t ldx, const float* S, int64_t lds_, int64_t m,
                   int32_t fi, int32_t fo, int32_t prec, float* Y, void* yws, size_t yws_bytes,
                   hipStream_t s) {
  if (m < 0 || fi <= 0 || fo <= 0 || (fi & 3) || (fo & 3) || fi > 256 || fo > 256 ||
      ldx < fi || lds_ < fo || (ldx & 3) || (lds_ & 3))
    return SAGNN_EINVAL;
  if (prec != SAGNN_GEMM_FP32 && prec != SAGNN_GEMM_BF16 && prec != SAGNN_GEMM_FP32_BF16X3) return SAGNN_EINVAL;
  if (!Y || !yws || !aligned16(yws)) return SAGNN_EINVAL;
  if (m > 0 && (!X || !S || !aligned16(X) || !aligned16(S))) return SAGNN_EINVAL;
  if (yws_bytes < tn_partial_bytes(m, (int64_t)fi * fo)) return SAGNN_ECAPACITY;
  int32_t parts = (int32_t)tn_parts(m, (int64_t)fi * fo);
  if (td_waves(prec) == 16) parts = std::min(parts, 256);      // (one workgroup fills a CU)
  TnArgs g{};
  g.X = X; g.ldx = ldx; g.S = S; g.lds_ = lds_; g.m = m; g.fi = fi; g.fo = fo;
  g.rows_per_wg = ceil_div(ceil_div(m > 0 ? m : 1, parts), KB) * KB;
  g.partial = reinterpret_cast<float*>(yws);
  if (tn_staged(fi, fo, prec)) {
    const size_t lds = (size_t)(((fi + 31) / 32 + (fo + 31) / 32) * 32) * KP * 2;
    SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tn_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds));
    hipLaunchKernelGGL(gemm_tn_kernel, dim3(parts), dim3(kTnThreads), lds, s, g);
    SAGNN_LAUNCH_CHECK();
  } else {
    // Columns of a lane: four, but three where blocks of 48 waste less on columns that are not there (33 to 48, 65 to 96,
    // 129 to 144) and the matrix instructions bound it: fp32, 170 k x 96 x 96 57 -> 37 us, 256 x 40 63 -> 50, 48 x 48 23 -> 15.
    auto columns = [&](int32_t w) {
      if (w <= 16) return 1;
      if (w <= 32) return 2;
      return prec == SAGNN_GEMM_FP32 && (w + 47) / 48 * 3 < (w + 63) / 64 * 4 && (w + 47) / 48 == (w + 63) / 64 ? 3 : 4;
    };
    const int va = columns(fi), vb = columns(fo);
    const int nbx = (fi + 16 * va - 1) / (16 * va), nbs = (fo + 16 * vb - 1) / (16 * vb), nb = nbx * nbs;
    // Blocks of Y in a workgroup: one for each wavefront, but eight where sixteen would leave half of the CUs without a
    // workgroup (256 x 256 behind a product of one entry a row, 1000, 4000, 10000 rows 58, 62, 65 us with sixteen, 33, 39, 41
    // with eight; 20000 x 256 x 160 55, 59).
    const int waves = td_waves(prec), most = parts <= 128 ? std::min(waves, 8) : waves;
    const int nwg = (nb + most - 1) / most, per = (nb + nwg - 1) / nwg;
    // Shares of a slice's rows: one for each wavefront, but of eight where a slice has 128 rows, the fewest (30 k x 128 x
    // 128: 21 us with sixteen, 18 with eight).  Still fewer would take up to 2 us off such calls, but sums of 64 rows in a
    // chain are up to 1.4 times as far from exact as sums of 16.
    const int kshare = std::max(1, (g.rows_per_wg > 128 ? waves : std::min(waves, 8)) / per);
    const size_t lds = (size_t)(kshare / 2) * per * va * vb * 64 * 16;   // at most 8 KB a wavefront
    const dim3 grid((unsigned)nwg, (unsigned)parts);   // (workgroups that read the same rows run side by side)
    auto go = [&](auto kern) -> int {
      if (lds > 48 * 1024)
        SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(kern, grid, dim3((unsigned)(per * kshare * 64)), lds, s, g, nbx, nbs, per, kshare);
      SAGNN_LAUNCH_CHECK();
      return SAGNN_OK;
    };
    auto width = [&](auto p) -> int {
      constexpr int PREC = decltype(p)::value;
      auto with = [&](auto a) -> int {
        constexpr int VA = decltype(a)::value;
        if (vb == 1) return go(gemm_tn_direct_kernel<PREC, VA, 1>);
        if (vb == 2) return go(gemm_tn_direct_kernel<PREC, VA, 2>);
        if constexpr (PREC == SAGNN_GEMM_FP32)
          if (vb == 3) return go(gemm_tn_direct_kernel<PREC, VA, 3>);
        return go(gemm_tn_direct_kernel<PREC, VA, 4>);
      };
      if (va == 1) return with(std::integral_constant<int, 1>{});
      if (va == 2) return with(std::integral_constant<int, 2>{});
      if constexpr (PREC == SAGNN_GEMM_FP32)
        if (va == 3) return with(std::integral_constant<int, 3>{});
      return with(std::integral_constant<int, 4>{});
    };
    int rc;
    if (prec == SAGNN_GEMM_BF16) rc = width(std::integral_constant<int, SAGNN_GEMM_BF16>{});
    else if (prec == SAGNN_GEMM_FP32_BF16X3) rc = width(std::integral_constant<int, SAGNN_GEMM_FP32_BF16X3>{});
    else rc = width(std::integral_constant<int, SAGNN_GEMM_FP32>{});
    if (rc != SAGNN_OK) return rc;
  }
  const int64_t elems = (int64_t)fi * fo;
  hipLaunchKernelGGL(tn_reduce_kernel, dim3((unsigned)ceil_div(elems, 32)), dim3(256), 0, s,
                     g.partial, parts, elems, Y);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

int launch_gemm(const float* X, int64_t ldx, const float* W, int64_t ldw, int32_t transW,
                int64_t m, int32_t kdim, int32_t nout, int32_t prec, int32_t act,
                const float* mask, int64_t ldmask, float* Z, int64_t ldz, float* A, int64_t lda,
                hipStream_t s) {
  if (m < 0 || kdim <= 0 || nout <= 0 || (kdim & 3) || (nout & 3) || kdim > 256 || nout > 256)
    return SAGNN_EINVAL;
  if (prec != SAGNN_GEMM_FP32 && prec != SAGNN_GEMM_BF16 && prec != SAGNN_GEMM_FP32_BF16X3) return SAGNN_EINVAL;
  if (act != SAGNN_ACT_IDENTITY && act != SAGNN_ACT_RELU) return SAGNN_EINVAL;
  if (transW != 0 && transW != 1) return SAGNN_EINVAL;
  if (ldx < kdim || (ldx & 3) || ldw < (transW ? kdim : nout)) return SAGNN_EINVAL;
  if ((Z && ldz < nout) || (A && lda < nout) || (mask && ldmask < nout)) return SAGNN_EINVAL;
  if (!Z && !A) return SAGNN_EINVAL;
  if (!W) return SAGNN_EINVAL;
  if (m == 0) return SAGNN_OK;
  if (!X || !aligned16(X)) return SAGNN_EINVAL;

  GemmArgs g{};
  g.X = X; g.ldx = ldx; g.W = W; g.ldw = ldw; g.transW = transW; g.m = m; g.kdim = kdim;
  g.nout = nout; g.act = act; g.mask = mask; g.ldmask = ldmask; g.Z = Z; g.ldz = ldz; g.A = A;
  g.lda = lda;
  const int tiles = (nout + 31) / 32;
  // (fp32 is not run as three terms though these are faster from 50 k rows on, 170 k 128 x 256 135 us, 100: on an X with one
  // value in 32 not zero they are twice as far from 64 bits, 4.4e-8, 7.7e-8; one value of W that they do not hold makes it 330;
  // and a row's result would depend on how many rows there are and on those beside it)
  auto run = [&](int nt) {
    if (prec == SAGNN_GEMM_FP32) return gemm_nn_fp32(nt, g, s);
    return prec == SAGNN_GEMM_BF16 ? gemm_nn_bf16(nt, g, s) : gemm_nn_bf16x3(nt, g, s);
  };
  // 32-column tiles of the widest slab: all of W in one launch with rounded operands; 128 columns in fp32 and in three
  // terms, 64 where the three planes of 128 do not fit the LDS (beyond k = 128)
  const int widest = prec == SAGNN_GEMM_BF16 ? 8 : (prec == SAGNN_GEMM_FP32 || nn_slab_bytes(kdim, 4, prec) <= 160 * 1024 ? 4 : 2);
  int nt = 1;
  while (nt < widest && nt < tiles) nt *= 2;
  // Few rows: narrower slabs, side by side in one launch, until this many wavefronts have a tile.  A wide slab is a chain
  // on a few CUs there: staging W, then the matrix instructions of all its columns, and the slabs one after the other.
  // us before and so, fp32 4096 x 256 x 256 86, 13; 128 x 128 18, 10; 30 k 256 x 256 94, 53; 128 x 128 23, 21; 45 k
  // 256 x 256 98, 77; 200 x 100 48, 44; rounded 10 k 256 x 256 26, 17; three terms 10 k 256 x 256 65, 25.  The lines lie
  // where the wide form is as fast: rounded operands, whose matrix instructions cost little and whose workgroups have eight
  // wavefronts, 20 k x 128 x 128 15, with 1024 wavefronts 13, with 2048 17; three terms 45 k x 256 x 40 20 and 24, but where
  // the wide form is several launches 30 k x 256 x 256 73 and 53.  And from 1536 row tiles to 2048 the wide form is one round
  // of wavefronts that is nearly full, which narrow slabs cut in two: wide and narrow fp32 47 k rows (1469 row tiles) 100 x 64,
  // 256 x 40, 96 x 96, 200 x 100 16, 24, 22, 41 and 15, 20, 17, 37, 52 k (1625) 17, 25, 22, 42 and 21, 26, 25, 50; three terms
  // 48 x 200, 128 x 256 47 k 25, 38 and 20, 32, 52 k 24, 39 and 27, 41, and beyond k = 128 192 x 132 37 k
  // (1157) 34, 31, 42 k (1313) 35, 38.  In more than a round 128 columns of fp32 gain while its end is short: 67 k (2094)
  // 200 x 100 75, 61, 97 k 76, 71; 128 x 128, whose chains are short, 67 k 37, 34, 75 k (2344) 36, 36, 85 k 37, 39 and 52 k
  // 28, 26.  An output that overlaps X is written tile by tile behind the reads as before.
  const int64_t row_tiles = (m + 31) / 32;
  const int64_t enough = prec == SAGNN_GEMM_BF16 ? 1024 : (prec == SAGNN_GEMM_FP32 ? (tiles >= 4 ? 3072 : 2048) : (tiles > widest ? 4096 : 1024));
  int64_t most = INT64_MAX;   // row tiles up to which the slabs are narrow
  if (prec == SAGNN_GEMM_FP32) {
    if (tiles < 4 || (kdim > 128 && row_tiles <= 2048)) most = 1536;
    else if (kdim <= 128) most = 2560;
  } else if (prec == SAGNN_GEMM_FP32_BF16X3) {
    most = kdim > 128 ? 1200 : 1536;
  }
  auto apart = [&](const float* out, int64_t ld) {
    return !out || out + (m - 1) * ld + nout <= X || X + (m - 1) * ldx + kdim <= out;
  };
  if (row_tiles <= most && row_tiles * ((tiles + nt - 1) / nt) < enough && apart(Z, ldz) && apart(A, lda)) {
    while (nt > 1 && row_tiles * ((tiles + nt - 1) / nt) < enough) nt /= 2;
    g.slabs = (tiles + nt - 1) / nt;
    return run(nt);
  }
  g.slabs = 1;
  for (int32_t n0 = 0; n0 < nout; n0 += widest * 32) {
    g.n0 = n0;
    const int left = (nout - n0 + 31) / 32;
    for (nt = 1; nt < widest && nt < left;) nt *= 2;
    const int rc = run(nt);
    if (rc != SAGNN_OK) return rc;
  }
  return SAGNN_OK;
}

}  // namespace sagnn

SAGNN_EXPORT int dense_gemm_act(const float* d_X, int64_t ldx, const float* d_W, int64_t ldw,
                                int32_t transW, int64_t m, int32_t kdim, int32_t nout,
                                int32_t prec, int32_t act, const float* d_mask, int64_t ldmask,
                                float* d_Z, int64_t ldz, float* d_act, int64_t ldact,
                                void* stream) {
  return sagnn::launch_gemm(d_X, ldx, d_W, ldw, transW, m, kdim, nout, prec, act, d_mask, ldmask,
                            d_Z, ldz, d_act, ldact, (hipStream_t)stream);
}
