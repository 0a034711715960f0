#include "gemm_nn.h"

namespace sagnn {

int gemm_nn_bf16(int nt, const GemmArgs& g, hipStream_t s) {
  if (nt == 1) return launch_nn<1, SAGNN_GEMM_BF16>(g, s);
  if (nt == 2) return launch_nn<2, SAGNN_GEMM_BF16>(g, s);
  if (nt == 4) return launch_nn<4, SAGNN_GEMM_BF16>(g, s);
  if (nt == 8) return launch_nn<8, SAGNN_GEMM_BF16>(g, s);
  return SAGNN_EINVAL;
}

}  // namespace sagnn
