// Kernel of gemm.h and its launch, included by the source file of each operand mode.
#pragma once
#include <type_traits>

#include "gemm.h"

namespace sagnn {
namespace {

// ------------------------------------------------------------------------------------------
// W slab -> LDS: fp32 as Ws[k][n]; bf16 packed as Ws[k/8][n][k%8] (split mode: three such planes, one per term);
// zero outside W.  kdim is the zero-padded k extent, a multiple of 32.
// The chain of dependent round trips to L2 bounds this, not the bytes, and with few row tiles per wavefront it is
// the kernel: a thread has 16 loads in flight.  W as it lies: a thread takes 8 k of one column, the lanes of a
// load are 64 neighbouring columns.  W transposed: a thread takes 4 neighbouring k, eight lanes share a line of W (a
// lane per column touched 64 lines per load).  Loads outside W are clamped into it, so no branch stands between them.
// One element per thread and round trip before: 4096 x 256 x 256 bf16 40 -> 22 us as it lies, 44 -> 19 transposed;
// 125 k rows 131 -> 93 and 119 -> 89.
template <int NB, int PREC, int THREADS>
__device__ __forceinline__ void stage_w(const GemmArgs& g, int n0, char* smem, int kdim, int tid) {
  constexpr bool SPLIT = PREC == SAGNN_GEMM_FP32_BF16X3;
  const int kreal = g.kdim;
  float* __restrict__ Wf = reinterpret_cast<float*>(smem);
  __bf16* __restrict__ Wp = reinterpret_cast<__bf16*>(smem);
  if (!g.transW) {
    const int units = (kdim >> 3) * NB;      // a multiple of 128
    for (int u0 = tid; u0 < units; u0 += 2 * THREADS) {
      float w[2][8];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int u = u0 + b * THREADS;
        const int k0 = (u / NB) * 8;
        const int col = n0 + u % NB;
        const float* __restrict__ src = g.W + (col < g.nout ? col : g.nout - 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[b][i] = src[(int64_t)(k0 + i < kreal ? k0 + i : kreal - 1) * g.ldw];
      }
      __builtin_amdgcn_sched_barrier(0);     // all loads ahead of the first use
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int u = u0 + b * THREADS;
        if (u >= units) break;
        const int n = u % NB, k0 = (u / NB) * 8;
        const bool in = n0 + n < g.nout;
#pragma unroll
        for (int i = 0; i < 8; ++i) w[b][i] = in && k0 + i < kreal ? w[b][i] : 0.f;
        if constexpr (PREC == SAGNN_GEMM_FP32) {
#pragma unroll
          for (int i = 0; i < 8; ++i) Wf[(k0 + i) * NB + n] = w[b][i];
        } else {
          bf16x8 t1, t2, t3;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __bf16 a1 = (__bf16)w[b][i], a2 = a1, a3 = a1;
            if constexpr (SPLIT) split3(w[b][i], a1, a2, a3);
            t1[i] = a1; t2[i] = a2; t3[i] = a3;
          }
          bf16x8* __restrict__ Wv = reinterpret_cast<bf16x8*>(smem);
          Wv[u] = t1;
          if constexpr (SPLIT) {
            Wv[units + u] = t2;
            Wv[2 * units + u] = t3;
          }
        }
      }
    }
  } else {
    const int units = (kdim >> 2) * NB;      // (4 k of one column), a multiple of 256
    // any ldw and address is accepted: four single loads where a quad may straddle a 16-byte line
    const bool quads = (g.ldw & 3) == 0 && (reinterpret_cast<uintptr_t>(g.W) & 15) == 0;
    for (int u0 = tid; u0 < units; u0 += 4 * THREADS) {
      float4 w[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int u = u0 + b * THREADS;
        const int k0 = ((u / (8 * NB)) * 8 + (u & 7)) * 4;
        const int col = n0 + (u >> 3) % NB;
        // (kreal is a multiple of 4: a quad lies inside or outside as a whole)
        const float* __restrict__ src = g.W + (int64_t)(col < g.nout ? col : g.nout - 1) * g.ldw + (k0 < kreal ? k0 : kreal - 4);
        if (quads) w[b] = *reinterpret_cast<const float4*>(src);
        else w[b] = make_float4(src[0], src[1], src[2], src[3]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int u = u0 + b * THREADS;
        if (u >= units) break;
        const int n = (u >> 3) % NB, k0 = ((u / (8 * NB)) * 8 + (u & 7)) * 4;
        const bool in = n0 + n < g.nout && k0 < kreal;
        const float x[4] = {in ? w[b].x : 0.f, in ? w[b].y : 0.f, in ? w[b].z : 0.f, in ? w[b].w : 0.f};
        if constexpr (PREC == SAGNN_GEMM_FP32) {
#pragma unroll
          for (int i = 0; i < 4; ++i) Wf[(k0 + i) * NB + n] = x[i];
        } else {
          bf16x4 t1, t2, t3;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            __bf16 a1 = (__bf16)x[i], a2 = a1, a3 = a1;
            if constexpr (SPLIT) split3(x[i], a1, a2, a3);
            t1[i] = a1; t2[i] = a2; t3[i] = a3;
          }
          const int at = ((k0 >> 3) * NB + n) * 8 + (k0 & 4);
          *reinterpret_cast<bf16x4*>(Wp + at) = t1;
          if constexpr (SPLIT) {
            *reinterpret_cast<bf16x4*>(Wp + kdim * NB + at) = t2;
            *reinterpret_cast<bf16x4*>(Wp + 2 * kdim * NB + at) = t3;
          }
        }
      }
    }
  }
  (void)Wf; (void)Wp;
}

// KPAD: kdim need not be a multiple of 32, loads of X are clamped to the real k extent.
// RAG: the slab has fewer than NB columns (a form of its own: the guards cost the full one registers).
// NG > 0: the k loop has exactly NG groups of 32 and is fully unrolled.  In straight-line code the
// compiler counts outstanding loads exactly; around a loop back-edge it waits for ALL of them,
// which would make the prefetch of the next group useless.
template <int NT, int PREC, int WAVES, bool KPAD, int NG, bool RAG>
__global__ __launch_bounds__(WAVES * 64) void gemm_nn_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int NB = NT * 32;
  constexpr bool BF16 = PREC == SAGNN_GEMM_BF16;
  constexpr bool SPLIT = PREC == SAGNN_GEMM_FP32_BF16X3;
  const int tid = threadIdx.x;
  const int kreal = g.kdim;                  // any multiple of 4
  const int kdim = (kreal + 31) & ~31;       // the k loop runs over the zero-padded extent

  const int n0 = g.n0 + (int)blockIdx.y * NB;   // first column of this workgroup's slab
  stage_w<NB, PREC, WAVES * 64>(g, n0, smem, kdim, tid);
  __syncthreads();

  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int64_t ntiles = (g.m + 31) >> 5;
  // Full tiles reach mask and outputs by a row address in scalar registers and one 32-bit offset per lane and array
  // (1 M x 16 x 16, both outputs: 56 -> 41 us; 170 k x 256 x 40 with bf16 operands, masked: 76 -> 37).
  constexpr int64_t kNear = 1 << 26;
  const bool near = (!g.mask || g.ldmask < kNear) && (!g.Z || g.ldz < kNear) && (!g.A || g.lda < kNear);
  const uint32_t moff0 = (uint32_t)(h * 4 * (int)g.ldmask + r) * 4u, zoff0 = (uint32_t)(h * 4 * (int)g.ldz + r) * 4u,
                 aoff0 = (uint32_t)(h * 4 * (int)g.lda + r) * 4u;
  for (int64_t t = (int64_t)blockIdx.x * WAVES + wave; t < ntiles; t += (int64_t)gridDim.x * WAVES) {
    int64_t row = t * 32 + r;
    if (row >= g.m) row = g.m - 1;  // clamped read, result discarded at the store
    const float* __restrict__ xrow = g.X + row * g.ldx;
    auto ldx4 = [&](int col) {   // X[row][col..col+3], zero beyond the real k extent (clamped load: no branch)
      if constexpr (KPAD) {
        const bool in = col < kreal;
        const float4 x = *reinterpret_cast<const float4*>(xrow + (in ? col : kreal - 4));
        return make_float4(in ? x.x : 0.f, in ? x.y : 0.f, in ? x.z : 0.f, in ? x.w : 0.f);
      } else {
        return *reinterpret_cast<const float4*>(xrow + col);
      }
    };
    floatx16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nt][v] = 0.f;

    // The k loop runs in groups of JB steps; the A-operand loads of the next group are issued
    // before the MFMAs of the current one, so HBM latency hides behind matrix-core work.
    if (SPLIT) {
      const bf16x8* __restrict__ Ws = reinterpret_cast<const bf16x8*>(smem);
      const int plane = (kdim >> 3) * NB;      // bf16x8 elements per term plane
      constexpr int JB = 2;
      const int ngroups = NG > 0 ? NG : kdim / (16 * JB);
      float4 cur[JB][2], nxt[JB][2];
#pragma unroll
      for (int q = 0; q < JB; ++q) {
        cur[q][0] = ldx4(16 * q + 8 * h);
        cur[q][1] = ldx4(16 * q + 8 * h + 4);
      }
#pragma unroll
      for (int gi = 0; gi < (NG > 0 ? NG : ngroups); ++gi) {
        if (gi + 1 < ngroups) {
#pragma unroll
          for (int q = 0; q < JB; ++q) {
            nxt[q][0] = ldx4(16 * ((gi + 1) * JB + q) + 8 * h);
            nxt[q][1] = ldx4(16 * ((gi + 1) * JB + q) + 8 * h + 4);
          }
        }
        if constexpr (NG > 0) __builtin_amdgcn_sched_barrier(0);   // keep the prefetch ahead of this group's MFMAs
#pragma unroll
        for (int q = 0; q < JB; ++q) {
          const int j = gi * JB + q;
          const float xs[8] = {cur[q][0].x, cur[q][0].y, cur[q][0].z, cur[q][0].w,
                               cur[q][1].x, cur[q][1].y, cur[q][1].z, cur[q][1].w};
          bf16x8 a1, a2, a3;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __bf16 t1, t2, t3;
            split3(xs[i], t1, t2, t3);
            a1[i] = t1; a2[i] = t2; a3[i] = t3;
          }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const int at = (2 * j + h) * NB + nt * 32 + r;
            const bf16x8 b1 = Ws[at], b2 = Ws[plane + at], b3 = Ws[2 * plane + at];
            // the six products down to 2^-16 of the leading one, smallest first
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a3, b1, acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b3, acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b2, acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b1, acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b2, acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, acc[nt], 0, 0, 0);
          }
        }
#pragma unroll
        for (int q = 0; q < JB; ++q) {
          cur[q][0] = nxt[q][0];
          cur[q][1] = nxt[q][1];
        }
      }
    } else if (BF16) {
      const bf16x8* __restrict__ Ws = reinterpret_cast<const bf16x8*>(smem);
      constexpr int JB = 2;
      const int ngroups = NG > 0 ? NG : kdim / (16 * JB);
      float4 cur[JB][2], nxt[JB][2];
#pragma unroll
      for (int q = 0; q < JB; ++q) {
        cur[q][0] = ldx4(16 * q + 8 * h);
        cur[q][1] = ldx4(16 * q + 8 * h + 4);
      }
#pragma unroll
      for (int gi = 0; gi < (NG > 0 ? NG : ngroups); ++gi) {
        if (gi + 1 < ngroups) {
#pragma unroll
          for (int q = 0; q < JB; ++q) {
            nxt[q][0] = ldx4(16 * ((gi + 1) * JB + q) + 8 * h);
            nxt[q][1] = ldx4(16 * ((gi + 1) * JB + q) + 8 * h + 4);
          }
        }
        if constexpr (NG > 0) __builtin_amdgcn_sched_barrier(0);   // keep the prefetch ahead of this group's MFMAs
#pragma unroll
        for (int q = 0; q < JB; ++q) {
          const int j = gi * JB + q;
          const float4 x0 = cur[q][0], x1 = cur[q][1];
          bf16x8 a;
          a[0] = (__bf16)x0.x; a[1] = (__bf16)x0.y; a[2] = (__bf16)x0.z; a[3] = (__bf16)x0.w;
          a[4] = (__bf16)x1.x; a[5] = (__bf16)x1.y; a[6] = (__bf16)x1.z; a[7] = (__bf16)x1.w;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const bf16x8 b = Ws[(2 * j + h) * NB + nt * 32 + r];
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[nt], 0, 0, 0);
          }
        }
#pragma unroll
        for (int q = 0; q < JB; ++q) {
          cur[q][0] = nxt[q][0];
          cur[q][1] = nxt[q][1];
        }
      }
    } else {
      const float* __restrict__ Ws = reinterpret_cast<const float*>(smem);
      constexpr int JB = 4;
      const int ngroups = NG > 0 ? NG : kdim / (8 * JB);
      float4 cur[JB], nxt[JB];
#pragma unroll
      for (int q = 0; q < JB; ++q) cur[q] = ldx4(8 * q + 4 * h);
#pragma unroll
      for (int gi = 0; gi < (NG > 0 ? NG : ngroups); ++gi) {
        if (gi + 1 < ngroups) {
#pragma unroll
          for (int q = 0; q < JB; ++q)
            nxt[q] = ldx4(8 * ((gi + 1) * JB + q) + 4 * h);
        }
        if constexpr (NG > 0) __builtin_amdgcn_sched_barrier(0);   // keep the prefetch ahead of this group's MFMAs
#pragma unroll
        for (int q = 0; q < JB; ++q) {
          const int j = gi * JB + q;
          const float xs[4] = {cur[q].x, cur[q].y, cur[q].z, cur[q].w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float* wrow = Ws + (8 * j + 4 * h + i) * NB + r;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[i], wrow[nt * 32], acc[nt], 0, 0, 0);
          }
        }
#pragma unroll
        for (int q = 0; q < JB; ++q) cur[q] = nxt[q];
      }
    }

    // (opaque from here on: worked out ahead of the row loop, the addresses of a tile's stores took 32 to 190
    // registers and left one or two wavefronts per SIMD)
    int64_t ldmask = g.ldmask, ldz = g.ldz, lda = g.lda;
    uint32_t moff = moff0, zoff = zoff0, aoff = aoff0;
    asm volatile("" : "+s"(ldmask), "+s"(ldz), "+s"(lda));
    asm volatile("" : "+v"(moff), "+v"(zoff), "+v"(aoff));
    if (t * 32 + 32 <= g.m && near) {
      // full tile of rows (the 16 values of a lane are rows 8*(v/4) + 4*h + v%4)
      const int col0 = n0 + r;
      const char* mt = reinterpret_cast<const char*>(g.mask + (t * 32 * ldmask + n0));
      char* zt = reinterpret_cast<char*>(g.Z + (t * 32 * ldz + n0));
      char* at = reinterpret_cast<char*>(g.A + (t * 32 * lda + n0));
      const bool relu = g.act == SAGNN_ACT_RELU;
      if (g.mask) {
        // the mask is applied in a pass of its own: between the stores below its loads would each
        // have to wait for the store before them (the arrays may alias as far as the compiler
        // knows), one memory round trip per element
        // and its loads are issued a batch at a time (16 to 32 in flight) ahead of their uses
        constexpr int VB = NT >= 8 ? 2 : 4;
        uint32_t mc[NT];                         // (a column beyond the slab reads the last one's mask)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          mc[nt] = moff + (!RAG || col0 + nt * 32 < g.nout ? nt * 128 : (g.nout - 1 - col0) * 4);
#pragma unroll
        for (int v0 = 0; v0 < 16; v0 += VB) {
          float mv[VB][NT];
#pragma unroll
          for (int dv = 0; dv < VB; ++dv) {
            const int64_t dr = ((v0 + dv) >> 2) * 8 + ((v0 + dv) & 3);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              mv[dv][nt] = *reinterpret_cast<const float*>(mt + dr * ldmask * 4 + (uint64_t)mc[nt]);
          }
          __builtin_amdgcn_sched_barrier(0);   // keep the batch of loads together, ahead of the selects
#pragma unroll
          for (int dv = 0; dv < VB; ++dv)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              if (!(mv[dv][nt] > 0.f)) acc[nt][v0 + dv] = 0.f;
        }
      }
      if constexpr (!RAG && PREC == SAGNN_GEMM_FP32 && NT == 2) {
        // 64 columns in fp32: a pointer per lane.  With scalar row addresses one output of 64 columns takes longer than
        // two (2.45 M x 128 x 64: 502 us with one, 504 with both; 600 k: 142); this way 430 and 515 (600 k: 115).  The
        // other slabs are as fast or faster with scalars (128 columns, masked, 600 k: 223 against 235).
        float* zl = g.Z ? g.Z + (t * 32 + h * 4) * g.ldz + col0 : nullptr;
        float* al = g.A ? g.A + (t * 32 + h * 4) * g.lda + col0 : nullptr;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t dr = (v >> 2) * 8 + (v & 3);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const float z = acc[nt][v];
            if (zl) zl[dr * g.ldz + nt * 32] = z;
            if (al) al[dr * g.lda + nt * 32] = relu ? (z > 0.f ? z : 0.f) : z;
          }
        }
      } else if constexpr (!RAG) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t dr = (v >> 2) * 8 + (v & 3);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const float z = acc[nt][v];
            if (g.Z) reinterpret_cast<float*>(zt + dr * ldz * 4 + (uint64_t)zoff)[nt * 32] = z;
            if (g.A) reinterpret_cast<float*>(at + dr * lda * 4 + (uint64_t)aoff)[nt * 32] = relu ? (z > 0.f ? z : 0.f) : z;
          }
        }
      } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (col0 + nt * 32 >= g.nout) continue;   // one branch per 32 columns, none between their stores
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int64_t dr = (v >> 2) * 8 + (v & 3);
            const float z = acc[nt][v];
            if (g.Z) reinterpret_cast<float*>(zt + dr * ldz * 4 + (uint64_t)zoff)[nt * 32] = z;
            if (g.A) reinterpret_cast<float*>(at + dr * lda * 4 + (uint64_t)aoff)[nt * 32] = relu ? (z > 0.f ? z : 0.f) : z;
          }
        }
      }
    } else {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int col = n0 + nt * 32 + r;
        if (col >= g.nout) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t ro = t * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
          if (ro >= g.m) continue;
          float z = acc[nt][v];
          if (g.mask && !(g.mask[ro * ldmask + col] > 0.f)) z = 0.f;
          if (g.Z) g.Z[ro * ldz + col] = z;
          if (g.A) g.A[ro * lda + col] = (g.act == SAGNN_ACT_RELU) ? (z > 0.f ? z : 0.f) : z;
        }
      }
    }
  }
}

template <int NT, int PREC, int WAVES>
int launch_nn_waves(const GemmArgs& g, size_t lds, hipStream_t s) {
  // A k extent of up to 128, or 256, has its loop unrolled (see NG).  Whole groups take the form without guards in fp32
  // and three-term mode: on many rows the guards cost a quarter (2.45 M rows, fp32, activation only: 64 x 64 345 us with
  // and 309 without, 96 x 64 512 and 377).  A single group has nothing to prefetch and is not unrolled (32 x 64: 245 with
  // guards, 219 unrolled, 190 as a loop, the last two with the stores of 64 columns below).  With operands rounded to
  // bfloat16 the guarded forms are as fast or faster (96 x 64: 283 and 301).
  auto pick = [&](auto rag) -> void (*)(const GemmArgs) {
    constexpr bool RAG = decltype(rag)::value;
    const int ng = (g.kdim + 31) / 32;
    if constexpr (PREC != SAGNN_GEMM_BF16) {
      if (g.kdim == 32) return gemm_nn_kernel<NT, PREC, WAVES, false, 0, RAG>;
      if (g.kdim == 64) return gemm_nn_kernel<NT, PREC, WAVES, false, 2, RAG>;
      if (g.kdim == 96) return gemm_nn_kernel<NT, PREC, WAVES, false, 3, RAG>;
    }
    if (ng == 1) return gemm_nn_kernel<NT, PREC, WAVES, true, 1, RAG>;
    if (g.kdim == 128) return gemm_nn_kernel<NT, PREC, WAVES, false, 4, RAG>;
    if constexpr (NT < 8) {   // (256 columns leave no registers for the guards of an unrolled loop)
      if (ng == 2) return gemm_nn_kernel<NT, PREC, WAVES, true, 2, RAG>;
      if (ng == 3) return gemm_nn_kernel<NT, PREC, WAVES, true, 3, RAG>;
      if (ng == 4) return gemm_nn_kernel<NT, PREC, WAVES, true, 4, RAG>;
    }
    if (g.kdim == 256) return gemm_nn_kernel<NT, PREC, WAVES, false, 8, RAG>;
    return g.kdim & 31 ? gemm_nn_kernel<NT, PREC, WAVES, true, 0, RAG> : gemm_nn_kernel<NT, PREC, WAVES, false, 0, RAG>;
  };
  void (*kern)(const GemmArgs) = g.n0 + g.slabs * NT * 32 <= g.nout ? pick(std::false_type{}) : pick(std::true_type{});
  SAGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const int64_t ntiles = (g.m + 31) / 32;
  int64_t blocks = ceil_div(ntiles, WAVES);
  // (a narrow slab: as many wavefronts as the registers hold, its time is the chain load - multiply - store)
  const int64_t per_cu = lds > 80 * 1024 ? 1 : (lds > 40 * 1024 ? 2 : (lds > 18 * 1024 || NT > 1 ? 4 : (WAVES == 4 ? 5 : 3)));
  if (blocks > 256 * per_cu) blocks = 256 * per_cu;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)g.slabs), dim3(WAVES * 64), lds, s, g);
  SAGNN_LAUNCH_CHECK();
  return SAGNN_OK;
}

template <int NT, int PREC>
int launch_nn(const GemmArgs& g, hipStream_t s) {
  const size_t lds = nn_slab_bytes(g.kdim, NT, PREC);
  if (lds > 160 * 1024) return SAGNN_EINVAL;
  // fp32: 4 wavefronts per workgroup, two workgroups per CU while the W slab allows it; when the
  // slab is so large that only one workgroup fits a CU, 8 wavefronts keep two per SIMD
  if constexpr (PREC != SAGNN_GEMM_FP32) {
    return launch_nn_waves<NT, PREC, 8>(g, lds, s);
  } else {
    if constexpr (NT == 4)
      if (lds > 80 * 1024) return launch_nn_waves<NT, PREC, 8>(g, lds, s);
    return launch_nn_waves<NT, PREC, 4>(g, lds, s);
  }
}

}  // namespace
}  // namespace sagnn
