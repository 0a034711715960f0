// The tall-skinny dense transform on the matrix cores, Z = X op(W): arguments and launch by operand mode.
// One source file per mode instantiates the kernel: the forms of a mode take a minute to compile.
#pragma once
#include "common.h"

namespace sagnn {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Split mode: a finite fp32 number x is the exact sum of three bfloat16 numbers: t1 = x rounded to
// nearest, t2 = (x - t1) rounded, t3 = x - t1 - t2, which needs no rounding (8 + 8 + 8 significant
// bits); both subtractions are exact, |t2| <= 2^-8 |x| and |t3| <= 2^-16 |x|.
__device__ __forceinline__ void split3(float x, __bf16& t1, __bf16& t2, __bf16& t3) {
  t1 = (__bf16)x;
  const float r = x - (float)t1;
  t2 = (__bf16)r;
  t3 = (__bf16)(r - (float)t2);
}

struct GemmArgs {
  const float* X; int64_t ldx;
  const float* W; int64_t ldw; int32_t transW;
  int64_t m; int32_t kdim, nout;
  int32_t act;
  const float* mask; int64_t ldmask;
  float* Z; int64_t ldz;
  float* A; int64_t lda;
  int32_t n0;     // first output column of this launch
  int32_t slabs;  // column slabs of this launch
};

// bytes of LDS the W slab of NT*32 columns takes (split mode: three bfloat16 planes)
inline size_t nn_slab_bytes(int32_t kdim, int nt, int prec) {
  const size_t elems = (size_t)((kdim + 31) & ~31) * nt * 32;
  return prec == SAGNN_GEMM_FP32 ? elems * 4 : (prec == SAGNN_GEMM_BF16 ? elems * 2 : elems * 6);
}

// nt: 32-column tiles of the slab (1, 2, 4; bf16 also 8)
int gemm_nn_fp32(int nt, const GemmArgs& g, hipStream_t s);
int gemm_nn_bf16(int nt, const GemmArgs& g, hipStream_t s);
int gemm_nn_bf16x3(int nt, const GemmArgs& g, hipStream_t s);

}  // namespace sagnn
