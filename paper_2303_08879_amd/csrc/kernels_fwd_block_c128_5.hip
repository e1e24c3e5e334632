#include "fwd_block.h"

namespace fd {
template hipError_t launch_fwd_block_range<double, 5>(const Plan&, const DevPlan&, int, const LevelPtrs<double>&,
                                                  const cx<double>*, const cx<double>*, int, hipStream_t);
}  // namespace fd
