#include "fwd_block.h"

namespace fd {
template hipError_t launch_jvp_block_range<double, 1>(const Plan&, const DevPlan&, int, const LevelPtrs<double>&,
                                                  const cx<double>*, const cx<double>*, int, int64_t, hipStream_t);
}  // namespace fd
