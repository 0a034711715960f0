#include "gemm_nn.h"

namespace sagnn {

int gemm_nn_guarded(int nt, const GemmArgs& g, hipStream_t s) {
  if (nt == 1) return launch_nn<1, kGemmGuarded>(g, s);
  if (nt == 2) return launch_nn<2, kGemmGuarded>(g, s);
  if (nt == 4) return launch_nn<4, kGemmGuarded>(g, s);
  return SAGNN_EINVAL;
}

}  // namespace sagnn
