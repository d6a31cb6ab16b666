// The tile kernel's LM-head forms whose left-over tiles are halved.
#include "tiled_gemm_kernel.h"

namespace mrp {

hipError_t launch_tiled_lm_halves(const TiledGemmArgs &a, int nb, int rem, hipStream_t st) { return launch_lm<true>(a, nb, rem, st); }

}  // namespace mrp
