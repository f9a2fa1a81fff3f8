// The direct-to-LDS projection kernels for a hidden size that is not a multiple of 64, and the rarely taken form of the
// steering sweep, in a translation unit of their own so that they build beside the others.
#include "ll_epilogue.h"
#include "ll_epilogue_sweep.h"
#include "ll_gemm_lds.h"

namespace ll {

GemmKernel tail_topk_kernel(int k, bool bias) {
  return with_list_length(k, [&](auto kr) -> GemmKernel {
    constexpr int KR = decltype(kr)::value;
    if (!bias) return ll_lens_gemm_dma_tail_kernel<TopKEpilogue<KR, false>>;
    if constexpr (KR < 32)
      return ll_lens_gemm_dma_tail_kernel<TopKEpilogue<KR, true>>;
    else
      return nullptr;   // two registers too many
  });
}

GemmKernel tail_sweep_kernel(bool lists) {
  return lists ? ll_lens_gemm_dma_tail_kernel<SweepEpilogue<SWEEP_KS, false>> : ll_lens_gemm_dma_tail_kernel<SweepEpilogue<1, false>>;
}

GemmKernel general_sweep_kernel(bool lists) {
  return lists ? ll_lens_gemm_dma_tail_kernel<SweepEpilogue<SWEEP_KS, true>> : ll_lens_gemm_dma_tail_kernel<SweepEpilogue<1, true>>;
}

}  // namespace ll
