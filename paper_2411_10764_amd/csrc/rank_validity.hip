// The validity walks over the rank form (rank_walk.h).
#include "rank_walk.h"

namespace ml2 {

hipError_t launch_rank_validity_kernel(int depth, RankMode mode, int waves, const RankArgs &a,
                                       int grid, size_t lds, hipStream_t s) {
  return rank::launch<false>(depth, mode, waves, a, grid, lds, s);
}

}  // namespace ml2
