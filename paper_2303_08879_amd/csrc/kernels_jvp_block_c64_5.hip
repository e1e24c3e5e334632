#include "fwd_block.h"

namespace fd {
template hipError_t launch_jvp_block_range<float, 5>(const Plan&, const DevPlan&, int, const LevelPtrs<float>&,
                                                  const cx<float>*, const cx<float>*, int, int64_t, hipStream_t);
}  // namespace fd
