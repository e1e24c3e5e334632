#include "vjp_block.h"

namespace fd {
template hipError_t launch_vjp_block_range<double, 1>(const Plan&, const DevPlan&, const VjpPtrs<double>&, const cx<double>*,
                                                   const cx<double>*, int, int, double2*, hipStream_t);
}  // namespace fd
