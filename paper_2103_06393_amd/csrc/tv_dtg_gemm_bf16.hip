// Instances of the decompress-then-GEMM products' GEMM for BF16X3 plans.
#define TV_SPLIT_GEMM_KERNELS
#include "tv_dtg_gemm.h"

namespace tv {
split_gemm_fn split_gemm_pick_bf16(bool adj, int mt, int ncol) {
  if (mt > 8) return ncol != 128 ? nullptr : adj ? split_pick_full<2, true>(mt) : split_pick_full<2, false>(mt);
  if (ncol == 256) return adj ? split_pick_w<2, true, 4>(mt) : split_pick_w<2, false, 4>(mt);
  return adj ? split_pick_w<2, true, 2>(mt) : split_pick_w<2, false, 2>(mt);
}
}  // namespace tv
