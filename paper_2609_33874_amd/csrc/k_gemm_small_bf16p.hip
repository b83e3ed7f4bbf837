// Small-tile GEMMs (gemm_small.h): (hi, lo) bf16 pairs.
#include "gemm_small_tiles.h"

namespace jetk {

hipError_t small_gemm_bf16p(int epi, int cfg, const GemmArgs<bf16> &g, hipStream_t st) {
  return run_small_tiles<bf16, 2, 0>(epi, cfg, g, st);
}

}  // namespace jetk
