// The steering sweep's direct-to-LDS kernels that form u = W_U v themselves (see ll_epilogue_sweep.h), in a translation unit of their
// own so that they build beside the others.
#include "ll_epilogue.h"
#include "ll_epilogue_sweep.h"
#include "ll_gemm_lds.h"

namespace ll {

GemmKernel whole_sweep_kernel(bool lists, bool general, bool ragged) {
  if (general) return lists ? ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<SWEEP_KS, true>> : ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<1, true>>;
  if (lists) return ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<SWEEP_KS, false>>;   // (four registers too many in one of its own)
  return ragged ? ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<1, false>> : ll_lens_gemm_dma_kernel<WholeSweepEpilogue<1, false>>;
}

}  // namespace ll
