#include "vjp_block.h"

namespace fd {
template hipError_t launch_vjp_block_range<float, 1>(const Plan&, const DevPlan&, const VjpPtrs<float>&, const cx<float>*,
                                                   const cx<float>*, int, int, double2*, hipStream_t);
}  // namespace fd
