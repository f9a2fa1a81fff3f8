// The direct-to-LDS projection kernels for calls of few tiles a workgroup, in a translation unit of their own so that they build
// beside the others.
#include "ll_epilogue.h"
#include "ll_gemm_lds.h"

namespace ll {

GemmKernel short_topk_kernel(int k, bool bias, bool ragged) {
  return with_list_length(k, [&](auto kr) -> GemmKernel {
    constexpr int KR = decltype(kr)::value;
    // (the longer lists have no registers for the classes, nor has the next one beside a bias)
    if constexpr (KR <= 12) {
      if (bias) return ragged ? ll_lens_gemm_short_kernel<TopKEpilogue<KR, true, true>, true> : ll_lens_gemm_short_kernel<TopKEpilogue<KR, true, true>, false>;
    }
    if constexpr (KR <= 20) {
      if (!bias) return ragged ? ll_lens_gemm_short_kernel<TopKEpilogue<KR, false, true>, true> : ll_lens_gemm_short_kernel<TopKEpilogue<KR, false, true>, false>;
    }
    return nullptr;
  });
}

}  // namespace ll
