// The tile kernel's LM-head forms on whole tiles.
#include "tiled_gemm_kernel.h"

namespace mrp {

hipError_t launch_tiled_lm(const TiledGemmArgs &a, int nb, int rem, hipStream_t st) { return launch_lm<false>(a, nb, rem, st); }

}  // namespace mrp
