// Instances of the decompress-then-GEMM products' GEMM for FP32 plans.
#define TV_SPLIT_GEMM_KERNELS
#include "tv_dtg_gemm.h"

namespace tv {
split_gemm_fn split_gemm_pick_f32(bool adj, int mt, int ncol) {
  if (mt > 8) return nullptr;
  if (ncol == 256) return adj ? split_pick_w<3, true, 4>(mt) : split_pick_w<3, false, 4>(mt);
  return adj ? split_pick_w<3, true, 2>(mt) : split_pick_w<3, false, 2>(mt);
}
}  // namespace tv
