// fp32 contractions of 3x3 convolutions (implicit GEMMs) on the bf16 matrix cores.

#include "gemm_split.h"

namespace opfuse {

hipError_t split_launch_conv(int kind, int tile, int S, int cz, int r_split, const GemmProblem& pr,
                             const EpiArgs& ea, void* ws, int vo, int ve, hipStream_t s) {
  return split_launch<true>(kind, tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
}

}  // namespace opfuse
