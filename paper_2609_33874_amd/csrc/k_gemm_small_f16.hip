// Small-tile GEMMs (gemm_small.h): fp16 operands.
#include "gemm_small_tiles.h"

namespace jetk {

hipError_t small_gemm_f16(int epi, int cfg, const GemmArgs<f16> &g, hipStream_t st) {
  return run_small_tiles<f16, 1, 0>(epi, cfg, g, st);
}

}  // namespace jetk
