#include "gemm_nn.h"

namespace sagnn {

int gemm_nn_fp32(int nt, const GemmArgs& g, hipStream_t s) {
  if (nt == 1) return launch_nn<1, SAGNN_GEMM_FP32>(g, s);
  if (nt == 2) return launch_nn<2, SAGNN_GEMM_FP32>(g, s);
  if (nt == 4) return launch_nn<4, SAGNN_GEMM_FP32>(g, s);
  return SAGNN_EINVAL;
}

}  // namespace sagnn
