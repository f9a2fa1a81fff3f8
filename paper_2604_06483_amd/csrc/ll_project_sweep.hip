// The steering sweep's direct-to-LDS kernels that form u = W_U v themselves (see ll_epilogue_sweep.h), in a translation unit of their
// own so that they build beside the others.
#include "ll_epilogue.h"
#include "ll_epilogue_sweep.h"
#include "ll_gemm_lds.h"

namespace ll {

GemmKernel whole_sweep_kernel(bool lists, bool general, bool ragged) {
  if (general) return lists ? ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<SWEEP_KS, true>> : ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<1, true>>;
  // (Lists over whole K stages run in the ragged kernel: one of their own would have no register to spare; 500 rows, d = 2560, V = 151936 434 | 431 us,
  // 1500 x 4096 x 128256 1317 | 1303, 700 x 1024 x 50257 173.6 | 173.1.)
  if (lists) return ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<SWEEP_KS, false>>;
  return ragged ? ll_lens_gemm_dma_tail_kernel<WholeSweepEpilogue<1, false>> : ll_lens_gemm_dma_kernel<WholeSweepEpilogue<1, false>>;
}

}  // namespace ll
