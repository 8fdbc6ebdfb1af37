// fp32 contractions of 3x3 convolutions (implicit GEMMs) on the bf16 matrix cores (gemm_split.h).

#include "gemm_split.h"

namespace opfuse {

template <int EPI>
static hipError_t launch_kind(int tile, int S, int cz, int r_split, const GemmProblem& pr,
                              const EpiArgs& ea, void* ws, int vo, int ve, hipStream_t s) {
  // the tiles a kind takes: see cheapest_split and gemm_launch
  if constexpr (EPI == EPI_FWD_FF) {
    if (tile == ST_64x32) return split_launch_t<S64x32, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32) return split_launch_t<S128x32, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32N) return split_launch_t<S128x32N, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32R) return split_launch_t<S128x32R, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  } else {
    if (tile == ST_64x64) return split_launch_t<S64x64, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x128) return split_launch_t<S128x128, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  if constexpr (EPI == EPI_FWD || EPI == EPI_DGRAD) {
    if (tile == ST_64x128) return split_launch_t<S64x128, EPI, true>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  return hipErrorInvalidValue;
}

hipError_t split_launch_conv(int kind, int tile, int S, int cz, int r_split, const GemmProblem& pr,
                               const EpiArgs& ea, void* ws, int vo, int ve, hipStream_t s) {
  switch (kind) {
    case EPI_FWD: return launch_kind<EPI_FWD>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_FWD_FF: return launch_kind<EPI_FWD_FF>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_DGRAD: return launch_kind<EPI_DGRAD>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_WGRAD: return launch_kind<EPI_WGRAD>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_WGRAD_BF: return launch_kind<EPI_WGRAD_BF>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace opfuse
